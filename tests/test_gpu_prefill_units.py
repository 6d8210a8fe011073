"""Prefill down projection units (128 rows of d by a chunk of at most 256
tokens, 16-token tiles) at their edges: chunks and runs with remainders, a
last row block of 64 rows, one token per tile, every expert kept, and the
longest tile list.  Against the fp64 oracle, and for the largest layer
against the decode kernels."""
import numpy as np
import pytest

import paper_2605_28283_amd as pp
from paper_2605_28283_amd.workloads import make_layer, make_tokens
from gpu_helpers import DevLayer, parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    pp.load()
    torch.cuda.init()


# (64, 8): one half row block, chunks of 32 tokens; (576, 16) and (192, 20):
# a last block of 64 rows; (1024, 2), T = 8209: 8 row blocks by 64 chunks of
# 129 tokens, two rounds of the 256 CUs
@pytest.mark.parametrize("d,E,T", [(64, 8, 1), (64, 8, 65), (576, 16, 33), (576, 16, 257),
                                   (192, 20, 600), (1024, 2, 8209)])
def test_prefill_units(oracle_mod, d, E, T):
    L = make_layer(d, E * 128, E, 700 + d)
    x, _ = make_tokens(T, d, 701 + T)
    with DevLayer(L, T) as dl:
        for tau in (0.3, 0.9, 1.0):
            print("prefill units d=%d E=%d T=%d tau=%g" % (d, E, T, tau), flush=True)
            parity(oracle_mod, dl, "prefill", x, tau)


def test_prefill_longest_tile_list():
    """256 experts, all kept, 64 row blocks: chunks of 238 tokens, whose list of
    256 x 15 tiles shares the LDS with the outputs, and a last one of 236.
    Prefill and decode each lie within 2.6e-6 of the exact result (2-norm), so
    within 1e-5 of each other."""
    import torch
    d, E, T = 8192, 256, 950
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    W = [torch.randn(s, generator=g, device="cuda").mul_(std).bfloat16()
         for s, std in (((E, d), 0.03), ((E * 128, d), 0.02), ((E * 128, d), 0.02),
                        ((d, E * 128), 0.02))]
    x = torch.randn((T, d), generator=g, device="cuda").bfloat16()
    h = pp.prunepath_create(d, E * 128, E, T, *W)
    try:
        ys = []
        for call in (pp.prunepath_ffn_prefill, pp.prunepath_ffn_decode):
            y = torch.full((T, d), float("nan"), device="cuda")
            cnt = torch.empty((T,), dtype=torch.int32, device="cuda")
            idx = torch.empty((T, E), dtype=torch.int32, device="cuda")
            call(h, x, T, 1.0, None, y, idx, cnt)
            torch.cuda.synchronize()
            assert (cnt == E).all()
            ys.append(y.double())
    finally:
        pp.prunepath_destroy(h)
    assert ((ys[0] - ys[1]).norm() / ys[1].norm()).item() <= 1e-5


@pytest.mark.parametrize("E", [1, 2, 3, 4, 5, 6, 7])
def test_prefill_expert_rings(oracle_mod, E):
    """Units of one expert to seven, each with one tile and with three (the last
    of two tokens): rings of three experts, and none, one or two after them."""
    d = 128
    L = make_layer(d, E * 128, E, 720 + E)
    for T in (9, 34):
        x, _ = make_tokens(T, d, 730 + T)
        with DevLayer(L, T) as dl:
            print("prefill rings E=%d T=%d" % (E, T), flush=True)
            parity(oracle_mod, dl, "prefill", x, 1.0)
