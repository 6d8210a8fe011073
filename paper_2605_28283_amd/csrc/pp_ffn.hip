// Prefill expert evaluation: Eq. (ffn) restricted to the kept experts and
// summed per token, Eqs. (moefication_decomp) and (moe_output), for large T.
//
// Work is organised in "groups" listed by a plan: one expert with up to 128
// of the tokens that kept it.  dispatch_k buckets the tokens per expert and
// splits each bucket into groups of 128; each (token, expert) pair owns one
// row of the h scratch, rows numbered group by group, tokens ascending inside
// a group.
//
//   dispatch_k  : per expert, the ascending list of tokens that kept it
//                 (ballot prefix over blocks of 256 tokens + scatter), where
//                 each token chunk starts in it, and the plan,
//                 written by the last expert to finish.
//   gateup_pf_k : unit = one group, all of K, one workgroup per CU; the
//                 gate/up projections and the SiLU product (bf16 MFMA, each
//                 weight fragment read once per group).  The groups of a last,
//                 partial round are split along K into pieces whose partial
//                 sums the last piece adds in piece order.
//   down_rows_k : unit = (128 rows of d, a chunk of up to kPfChunk tokens);
//                 the chunk's y rows are summed in LDS over the experts in
//                 ascending order and written once -- no float atomics in
//                 memory, deterministic.
// Units sharing weights (an expert's groups; a row block's token chunks) are
// placed on one XCD, where they meet in L2.
#include "pp_gateup.h"

namespace pp {
namespace {

struct DNParams {
    int T, d, E;
    const uint16_t *Wd;
    const uint16_t *h_hi;
    const uint16_t *h_lo;
    float *y;
    const float *bproj;    // [d] output bias, or NULL (0)
    const int32_t *cut;    // [E][nC + 1]: expert e's tokens below token c * C
    int C, nC;             // tokens per chunk, chunks
    const int32_t *ebase;  // [E] first pair (h row) of each expert's bucket
    const int32_t *pair_tok;  // [pairs] token of each h row
};

// Gate/up of one group (one expert, up to kPfGroupTokens of its tokens) in
// one workgroup, all 256 gate/up columns and all of K: wavefront w owns the
// expert's neuron tile w (16 neurons, gate and up) for every token tile of
// the group, so each weight fragment is read once per group, by one
// wavefront, straight from HBM into registers kPfPF K-steps ahead.  The
// group's token rows are staged in LDS in B-fragment order, kPfXC K-steps at
// a time: wavefront w copies token tile w's fragments of the next sub-chunk
// straight into LDS (buffer loads to LDS, no registers) while the current
// one is multiplied -- two LDS buffers, separate arrays so that the
// compiler's waits for the copies into one do not hold up reads of the
// other, and one barrier per sub-chunk.  Token tiles are multiplied in
// pairs, the pairs past the group skipped.  One workgroup per CU; the groups
// of one expert are neighbouring units on one XCD, where they share the
// expert's weights in L2.  16384 tokens at tau 0.9 on the LLaMA-3-8B shape take
// 605 us with 8.3 GB requested of L2 (13.8 TB/s, half of what plain reads reach
// with more bytes in flight per CU), 700 us when a copy took 64-byte pieces of
// rows.  Left out one at a time, the token copies save 28 %, the weight loads
// 12 %, the products 7 % and the LDS reads nothing: waits for the copies weigh
// most, and no unit is at its rate.
constexpr int kPfXC = 8;                         // K-steps per staged token sub-chunk
constexpr int kPfPF = 4;                         // K-steps of weights in flight per wavefront
constexpr int kPfNT = kPfGroupTokens / 16;       // token tiles per group
static_assert(kPfXC % kPfPF == 0, "the weight ring restarts at every sub-chunk");
static_assert(kPfNT == kGuThreads / 64, "wavefront w stages token tile w");

// SiLU(a) * b with the hardware exp2 and reciprocal (about 1 ulp each):
// a / (1 + e^-a) = a * rcp(1 + 2^(-a log2 e)); a -> -inf gives 0, a -> +inf a.
__device__ __forceinline__ float silu_mul_fast(float a, float b) {
    const float t = __builtin_amdgcn_exp2f(-a * 1.44269504088896341f);
    return a * __builtin_amdgcn_rcpf(1.0f + t) * b;
}

// Copies 16 bytes per lane from the buffer into LDS: lane l's bytes land at
// dst + 16 l (dst wavefront-uniform).
__device__ __forceinline__ void lds_dma16(__amdgpu_buffer_rsrc_t r, uint4 *dst, unsigned off) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        r, (__attribute__((address_space(3))) void *)dst, 16, off, 0, 0, 0);
}

// A token sub-chunk in LDS: [K-step pair][token tile][8 rows][row, 16-byte
// chunk].  A copy instruction takes the 128 bytes that a pair of K-steps reads
// of eight rows, whole cache lines (one that took 64 bytes of sixteen rows
// fetched each line twice); chunk c of row r lies at place c ^ (r % 8), which
// spreads the 16 rows that a fragment read touches over all banks.
typedef uint4 PfTokens[kPfXC / 2][kPfNT][2][64];

// This lane's part of the B fragment of K-step k, token tile j: row lane %
// 16, chunk 4 (k % 2) + lane / 16 of the pair.
__device__ __forceinline__ uint4 pf_token_frag(const PfTokens &xs, int k, int j, int lane) {
    const int r = lane & 7, c = (4 * (k & 1) + (lane >> 4)) ^ r;
    return xs[k >> 1][j][(lane >> 3) & 1][8 * r + c];
}

template <bool GATED>
__device__ __forceinline__ float pf_act(const GUParams &P, int e, int r, float a, float b) {
    if (GATED) return silu_mul_fast(a, b);
    return act<false>(P, e, r, a, b);
}

// STREAM: a dense decode batch (every expert kept) streams the weights; a
// prefill group's weights are shared with the other groups of its expert in
// L2 and are read with plain loads.
template <bool GATED, bool STREAM>
__device__ __forceinline__ void pf_load_w(const uint16_t *wb, int s, uint4 &g, uint4 &u) {
    const uint16_t *p = wb + (size_t)s * kStepElems<GATED>;
    g = ldw16_if<STREAM>(p);
    if (GATED) u = ldw16_if<STREAM>(p + 512);
}

// Work list of gateup_pf_k with nG groups on nW workgroups: full rounds of
// whole groups (nW groups each), then the groups left over, each split into
// KS pieces along K (at most nW pieces in all, at most four per group), so
// that the last (or only) round uses more of the workgroups instead of
// leaving them idle.
struct PfSchedule {
    int full;    // groups run whole: [0, full)
    int KS;      // pieces per leftover group (1 when nothing is left over)
    int units;   // full + (nG - full) * KS
};

__device__ __forceinline__ PfSchedule pf_schedule(int nG, int nW, size_t part_rows) {
    PfSchedule S;
    S.full = nG - nG % nW;
    const int left = nG - S.full;
    S.KS = 1;
    if (left > 0) {
        S.KS = min(nW / left, 4);
        // each piece's partial rows (up to kPfGroupTokens per group) must fit
        while (S.KS > 1 && (size_t)left * S.KS * kPfGroupTokens > part_rows) --S.KS;
        if (S.KS < 1) S.KS = 1;
    }
    if (S.KS == 1) S.full = nG;
    S.units = S.full + (nG - S.full) * S.KS;
    return S;
}

// DEC: a decode batch whose groups come from the router's per-expert token
// masks (the decode plan, derived here in LDS as the decode gate/up kernel
// does; workgroup 0 stores it for the down projection).
template <bool GATED, bool DEC>
__global__ __launch_bounds__(kGuThreads, 1) void gateup_pf_k(GUParams P) {
    __shared__ PfTokens xs0, xs1;
    __shared__ int stok[kPfGroupTokens];
    __shared__ int s_flag;
    __shared__ DecodePlan D;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (DEC) decode_plan<true>(P, D, tid < P.E ? P.emask[tid] : 0ull);
    const int nG = DEC ? D.nG : P.plan.head[0];
    const int NS = P.NS, last = NS - 1;
    const int nsub = (NS + kPfXC - 1) / kPfXC;  // token sub-chunks over all of K
    const bool sig = (P.flags & PP_AGG_SIGMOID) != 0;
    const PfSchedule S = pf_schedule(nG, (int)gridDim.x, P.abpart_rows);
    const int slots_full = 8 * ((S.full + 7) / 8);
    for (int slot = blockIdx.x; slot < slots_full + (S.units - S.full); slot += gridDim.x) {
        // unit: a whole group (xcd-ordered, so an expert's groups share an
        // XCD), or piece `piece` of leftover group g (pieces of one group are
        // neighbouring slots)
        int g, piece = 0, KSg = 1;
        if (slot < slots_full) {
            g = xcd_order(slot, S.full);
            if (g >= S.full) continue;
        } else {
            const int v = slot - slots_full;
            g = S.full + v / S.KS;
            piece = v - (g - S.full) * S.KS;
            KSg = S.KS;
        }
        const int cA = piece * nsub / KSg, cB = (piece + 1) * nsub / KSg;
        const int sA = cA * kPfXC, sB = min(cB * kPfXC, NS);
        int e, n, p0;
        __syncthreads();  // the previous unit is done with stok and xs
        if (DEC) {
            const unsigned long long m = D.mask[g];
            e = D.e[g];
            n = __popcll(m);
            p0 = D.pair[g];
            if (tid < 64 && ((m >> tid) & 1ull)) stok[__popcll(m & ((1ull << tid) - 1ull))] = tid;
        } else {
            e = P.plan.grp_e[g];
            n = P.plan.grp_n[g];
            p0 = P.plan.grp_pair[g];
            if (tid < n) {
                const int t = P.plan.toklist[P.plan.grp_tok[g] + tid];
                stok[tid] = t;
                if (piece == 0) P.pair_tok[p0 + tid] = t;
            }
        }
        __syncthreads();
        const int nt = (n + 15) >> 4;
        const bool stager = wv < nt;
        // this lane's token rows while staging tile wv (slots past the group
        // read its last token: they only feed output columns never stored)
        unsigned xoff[2];
#pragma unroll
        for (int h = 0; h < 2; ++h)
            xoff[h] = (unsigned)stok[min(16 * wv + 8 * h + (lane >> 3), n - 1)] * (unsigned)P.d * 2u +
                      16u * ((lane & 7) ^ (lane >> 3));
        const auto rx = buf_rsrc(P.x, stager ? (unsigned)((size_t)P.T * P.d * 2u) : 0u);
        const uint16_t *wb =
            P.Wgu + (size_t)(e * 8 + wv) * NS * kStepElems<GATED> + lane * 8;
        uint4 G[kPfPF], U[kPfPF];
#pragma unroll
        for (int i = 0; i < kPfPF; ++i) pf_load_w<GATED, DEC>(wb, min(sA + i, last), G[i], U[i]);
        auto stage = [&](PfTokens &xs, int s0) {  // K-steps come in pairs (d is a multiple of 64)
#pragma unroll
            for (int k = 0; k < kPfXC; k += 2)
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    lds_dma16(rx, &xs[k >> 1][wv][h][0],
                              xoff[h] + (unsigned)min(s0 + k, last - 1) * kKStep * 2u);
        };
        stage(xs0, sA);
        {
            const uint4 own = xs0[kPfXC / 2 - 1][wv][1][lane];  // waits for this wavefront's copies
            asm volatile("" ::"v"(own.x));
        }
        __syncthreads();
        f32x4 ag[kPfNT], au[kPfNT];
#pragma unroll
        for (int j = 0; j < kPfNT; ++j) {
            ag[j] = f32x4{0.f, 0.f, 0.f, 0.f};
            au[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        auto sub = [&](const PfTokens &cur, PfTokens &nxt, int s0) {
            const bool more = s0 + kPfXC < sB;
            if (more) stage(nxt, s0 + kPfXC);
            // the token fragments of step k are read from LDS one step ahead
            uint4 b[kPfNT];
#pragma unroll
            for (int j = 0; j < kPfNT; ++j) b[j] = pf_token_frag(cur, 0, j, lane);
#pragma unroll
            for (int k = 0; k < kPfXC; ++k) {
                uint4 bn[kPfNT];
                if (k + 1 < kPfXC) {
#pragma unroll
                    for (int j = 0; j < kPfNT; ++j) bn[j] = pf_token_frag(cur, k + 1, j, lane);
                }
                if (s0 + k < sB) {
                    // token tiles in pairs: the pairs past the group are skipped
#pragma unroll
                    for (int j = 0; j < kPfNT; ++j) {
                        if (j < 2 || nt > (j & ~1)) {
                            ag[j] = mfma16(G[k % kPfPF], b[j], ag[j]);
                            if (GATED) au[j] = mfma16(U[k % kPfPF], b[j], au[j]);
                        }
                    }
                }
                pf_load_w<GATED, DEC>(wb, min(s0 + k + kPfPF, last), G[k % kPfPF], U[k % kPfPF]);
                if (k + 1 < kPfXC) {
#pragma unroll
                    for (int j = 0; j < kPfNT; ++j) b[j] = bn[j];
                }
            }
            if (more) {
                // this wavefront's copies into nxt have landed before the barrier
                const uint4 own = nxt[kPfXC / 2 - 1][wv][1][lane];
                asm volatile("" ::"v"(own.x));
            }
            __syncthreads();
        };
        for (int s0 = sA; s0 < sB; s0 += 2 * kPfXC) {
            sub(xs0, xs1, s0);
            if (s0 + kPfXC < sB) sub(xs1, xs0, s0 + kPfXC);
        }
        // lane holds neurons r0 .. r0 + 3 of token slot 16 j + lane % 16
        const int r0 = wv * 16 + 4 * (lane >> 4);
        if (KSg > 1) {
            // a piece of a split group: its partial (a, b) in fragment order,
            // [piece][token tile][wavefront][a, b][lane] float4 (one KiB per
            // wavefront store); the last piece to arrive adds the pieces in
            // piece order at its own fragments and goes on to the epilogue
            constexpr unsigned kPieceBytes = kPfNT * 8 * 2 * 64 * 16;
            const auto pr = buf_rsrc(P.abpart + (size_t)(g - S.full) * KSg * (kPieceBytes / 4),
                                     (unsigned)KSg * kPieceBytes);
            const unsigned lo = ((unsigned)wv * 2 * 64 + lane) * 16;
#pragma unroll
            for (int j = 0; j < kPfNT; ++j) {
                if (j < nt) {
                    const unsigned o = (unsigned)piece * kPieceBytes + j * (8 * 2 * 64 * 16) + lo;
                    st_dev16(pr, o, ag[j]);
                    if (GATED) st_dev16(pr, o + 64 * 16, au[j]);
                }
            }
            if (!arrive_last(&P.cnt[g], (unsigned)KSg, &s_flag)) continue;
            f32x4 sa[kPfNT], su[kPfNT];
            for (int k = 0; k < KSg; ++k) {
#pragma unroll
                for (int j = 0; j < kPfNT; ++j) {
                    f32x4 va = ag[j], vu = au[j];
                    if (k != piece && j < nt) {
                        const unsigned o = (unsigned)k * kPieceBytes + j * (8 * 2 * 64 * 16) + lo;
                        va = ld_dev16(pr, o);
                        if (GATED) vu = ld_dev16(pr, o + 64 * 16);
                    }
                    sa[j] = k == 0 ? va : sa[j] + va;
                    su[j] = k == 0 ? vu : su[j] + vu;
                }
            }
#pragma unroll
            for (int j = 0; j < kPfNT; ++j) {
                ag[j] = sa[j];
                au[j] = su[j];
            }
        }
#pragma unroll
        for (int j = 0; j < kPfNT; ++j) {
            const int q = 16 * j + (lane & 15);
            if (j < nt && q < n) {
                const float scl = sig ? P.gsig[(size_t)stok[q] * P.E + e] : 1.0f;
                uint16_t hi[4], lo[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    split_bf16(pf_act<GATED>(P, e, r0 + i, ag[j][i], au[j][i]) * scl, hi[i],
                               lo[i]);
                const size_t row = (size_t)(p0 + q) * kExpertWidth + r0;
                *reinterpret_cast<uint2 *>(P.h_hi + row) = make_uint2(
                    hi[0] | ((uint32_t)hi[1] << 16), hi[2] | ((uint32_t)hi[3] << 16));
                *reinterpret_cast<uint2 *>(P.h_lo + row) = make_uint2(
                    lo[0] | ((uint32_t)lo[1] << 16), lo[2] | ((uint32_t)lo[3] << 16));
            }
        }
    }
}

// ------------------------------------------------------------------ prefill

__global__ __launch_bounds__(256) void dispatch_k(const uint32_t *__restrict__ selmask, int T,
                                                  int E, int32_t *__restrict__ ecount,
                                                  int32_t *__restrict__ tokl, int stride,
                                                  int32_t *__restrict__ cut, PfChunks ck,
                                                  int32_t *__restrict__ ebase, uint32_t *cnt,
                                                  PlanView plan, int num_cu) {
    const int ncut = ck.n + 1;
    // t / C for t < 2^20 and C <= 256 (the quotient's error stays below 1 / C)
    const uint32_t rcpC = 0xFFFFFFFFu / (uint32_t)ck.C + 1u;
    constexpr int kBlocks = 8;  // blocks of 256 tokens whose flags are loaded at once
    __shared__ int scan[8];
    __shared__ __align__(16) int wc[2][kBlocks][4];  // per block and wavefront: tokens that kept e
    __shared__ int s_flag;
    const int e = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int w = e >> 5, b = e & 31;
    const unsigned long long below = (1ull << lane) - 1ull;
    int base = 0, par = 0;
    for (int T0 = 0; T0 < T; T0 += kBlocks * 256, par ^= 1) {
        uint32_t word[kBlocks];
#pragma unroll
        for (int j = 0; j < kBlocks; ++j) {
            const int t = T0 + 256 * j + tid;
            word[j] = t < T ? selmask[(size_t)t * 8 + w] : 0u;
        }
        unsigned long long bal[kBlocks];
#pragma unroll
        for (int j = 0; j < kBlocks; ++j) {
            bal[j] = __ballot((word[j] >> b) & 1u);
            if (lane == 0) wc[par][j][wv] = __popcll(bal[j]);
        }
        __syncthreads();
        // block j's tokens follow those of blocks 0 .. j - 1, in token order
#pragma unroll
        for (int j = 0; j < kBlocks; ++j) {
            const int t = T0 + 256 * j + tid;
            const int4 c = *reinterpret_cast<const int4 *>(wc[par][j]);
            const int before = (wv > 0 ? c.x : 0) + (wv > 1 ? c.y : 0) + (wv > 2 ? c.z : 0);
            const int pos = base + before + __popcll(bal[j] & below);
            const int ch = (int)__umulhi((uint32_t)t, rcpC);
            if (t < T && ch * ck.C == t) cut[(size_t)e * ncut + ch] = pos;
            if ((bal[j] >> lane) & 1ull) tokl[(size_t)e * stride + pos] = t;
            base += (c.x + c.y) + (c.z + c.w);
        }
    }
    if (tid == 0) {
        cut[(size_t)e * ncut + ck.n] = base;
        st_dev_u32(reinterpret_cast<uint32_t *>(ecount + e), (uint32_t)base);
    }
    if (!arrive_last(cnt, (unsigned)E, &s_flag)) return;
    // prefill plan: expert e's bucket becomes ceil(c_e / gs) groups of nearly
    // equal size (the first c_e % groups one token larger), so that the groups
    // of one expert stream its weights at the same pace and meet in L2.  The
    // group size gs is the smallest of 64, 80, 96, 112 whose groups all fit in
    // one round on the CUs (smaller groups stage fewer token rows and spread
    // over more CUs), else kPfGroupTokens.
    const int c = (tid < E) ? (int)ld_dev_u32(reinterpret_cast<uint32_t *>(ecount + tid)) : 0;
    int gs = kPfGroupTokens;
    if ((long)T * E / 64 + E < 65535) {
        // the four sizes' group counts, two to an int (each sum below 2^16): one scan
        int x0, x1, p0, p1;
        block_excl_scan2(((c + 63) / 64) | (((c + 79) / 80) << 16),
                         ((c + 95) / 96) | (((c + 111) / 112) << 16), &x0, &x1, &p0, &p1, scan);
        const int n64 = p0 & 0xFFFF, n80 = p0 >> 16, n96 = p1 & 0xFFFF, n112 = p1 >> 16;
        gs = n64 <= num_cu ? 64 : n80 <= num_cu ? 80 : n96 <= num_cu ? 96 : n112 <= num_cu ? 112 : gs;
    }
    const int nch = (c + gs - 1) / gs;
    int cb, off, nG, npairs;
    block_excl_scan2(nch, c, &cb, &off, &nG, &npairs, scan);
    if (tid < E) ebase[tid] = off;
    const int gbase = nch > 0 ? c / nch : 0, grem = nch > 0 ? c - gbase * nch : 0;
    for (int ch = 0, first = 0; ch < nch; ++ch) {
        const int g = cb + ch, n = gbase + (ch < grem ? 1 : 0);
        plan.grp_e[g] = tid;
        plan.grp_pair[g] = off + first;
        plan.grp_n[g] = n;
        plan.grp_tok[g] = tid * stride + first;
        first += n;
    }
    if (tid == 0) {
        plan.head[0] = nG;
        plan.head[1] = npairs;
    }
}

// Unit = (kRowBlock rows of d, a chunk of C consecutive tokens).  The chunk's
// outputs in those rows stay in LDS for the whole unit, starting from the
// output bias (or 0).  The experts are taken in ascending order; the tokens
// of the chunk that kept expert e are a contiguous run of its ascending
// bucket (positions cut[e][c] .. cut[e][c + 1]), so their h rows are
// consecutive.  A step is one 16-token tile of a run.  Wavefronts 0 - 3 each
// own 32 rows of the block for every token: they multiply the tile's h
// (bf16 MFMA 16x16x32, A = the tokens' h, hi then lo per K-step, B = the
// expert's down rows, held in registers and loaded two experts ahead) and add
// the products to the tokens' LDS rows.  No other wavefront touches those
// rows, so the experts' order is the wavefront's own program order: every
// output is the bias plus its token's pair contributions in ascending expert
// order, deterministic, with no atomics in memory and no per-pair rows.
// Wavefronts 4 - 7 carry the h tiles from memory through registers (loads
// kTileAhead steps ahead, which covers the Infinity Cache's latency) into one
// of two LDS slots; one barrier per step hands a slot over.
//
// What bounds it: the CU's LDS accesses (per step 32 KiB of h read by the four
// wavefronts, 8 KiB read and written of y, 8 KiB of h written: about 480
// cycles of 600 to 650; the products take 300, and without the weight loads a
// step is a tenth to a fifth shorter).  A block of 64 rows by 512 tokens, staged in LDS and
// multiplied by whichever wavefronts the run's tiles fill, with two barriers
// per expert, took (LLaMA-3-8B shape) 132 us for 2048 tokens at tau 0.7 and
// 1550 us for 16384 at tau 0.9; this takes 88 and 1070 (98 and 1150 with h
// carried as 64-byte pieces of sixteen rows).  For 777 tokens of a 1024-wide
// GELU layer (16-row blocks before): 51 and 21.
constexpr int kTileAhead = 8;      // tiles in flight per carrying wavefront
constexpr int kWAhead = 2;         // experts whose down rows are loaded ahead (2048 tokens at
                                   // tau 0.7, LLaMA-3-8B shape: 1 95 us, 2 88, 3 90)
constexpr int kRowThreads = 512;
static_assert(kTileAhead % 2 == 0, "tile k lies in slot k % 2");

// Rows of the LDS outputs: token t's kRowBlock values from t * kRowBlock on,
// each wavefront's 32 with rows r and r + 16 side by side (value 2 (r % 16) +
// r / 16).  A lane's products with its two row tiles then make one 8-byte
// access, and the 16 lanes of a token cover all banks once, whatever the
// tokens.
__device__ __forceinline__ int row_off(int t) { return t * (kRowBlock * 4); }

struct DownRowsLds {
    uint4 h[2][2][16][16];     // [slot][hi, lo][place]: the token's h, 16-byte piece c of
                               // place q at c ^ q (spreads a fragment's reads over all banks)
    int off[2][16];            // [slot][place]: the token's row_off
    uint16_t ent[kMaxExperts]; // experts with tokens in the chunk, ascending: e | tiles << 8
    int scan[2 * (kRowThreads / 64)];
    // followed by the tile list, one word per tile in order (first pair (h
    // row) | (tokens - 1) << 24), and the outputs y, whose last row (C) takes
    // the products of empty tile places
};
static_assert(sizeof(DownRowsLds) % 16 == 0, "y rows are read as float4");
static_assert(sizeof(DownRowsLds) == kRowLdsFixed, "pf_row_lds counts on it");

// A tile's fragments as held by a multiplying wavefront.
struct RowTile {
    uint4 hi[4], lo[4];
    int4 off;  // the lane's four tokens (places 4 (lane / 16) + i)
};

// The lane's 16 bytes of K-step s of a slot's hi or lo: place lane % 16, piece
// 4 s + lane / 16.
__device__ __forceinline__ uint4 rows_frag(const uint4 (&h)[16][16], int s, int lane) {
    const int q = lane & 15;
    return h[q][(4 * s + (lane >> 4)) ^ q];
}

__device__ __forceinline__ void rows_read(RowTile &t, const DownRowsLds &S, int slot, int lane) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        t.hi[s] = rows_frag(S.h[slot][0], s, lane);
        t.lo[s] = rows_frag(S.h[slot][1], s, lane);
    }
    t.off = *reinterpret_cast<const int4 *>(&S.off[slot][4 * (lane >> 4)]);
}

// The barrier after which tile k + 1 is in its slot and the carrying wavefronts
// may write to tile k's.  This wavefront has then read all of tile k (t): the
// barrier takes what it read as operands, so that the compiler waits for those
// reads, and for no later access.
__device__ __forceinline__ void rows_handover(const RowTile &t) {
    auto v = [](const uint4 &u) { return __builtin_bit_cast(u32x4_t, u); };
    asm volatile("s_barrier" ::"v"(v(t.hi[0])), "v"(v(t.lo[0])), "v"(v(t.hi[1])), "v"(v(t.lo[1])),
                 "v"(v(t.hi[2])), "v"(v(t.lo[2])), "v"(v(t.hi[3])), "v"(v(t.lo[3])),
                 "v"(__builtin_bit_cast(u32x4_t, t.off))
                 : "memory");
}

// A tile's products on their way to the LDS outputs.
struct RowSums {
    f32x4 a0, a1;
    int off[4];
};

__device__ __forceinline__ float2 sums_load(const char *yb, const RowSums &p, int i) {
    return *reinterpret_cast<const float2 *>(yb + p.off[i]);
}

// (read, add, write: an LDS float atomic took ten times as long)
__device__ __forceinline__ void sums_store(char *yb, float2 y, const RowSums &p, int i) {
    *reinterpret_cast<float2 *>(yb + p.off[i]) = make_float2(y.x + p.a0[i], y.y + p.a1[i]);
}

// One step of a multiplying wavefront: multiplies tile k, adds tile k - 1's
// products to its tokens' rows and fetches tile k + 1.  An LDS access holds up
// the wavefront's next instruction for longer than a product does, so the 17
// accesses are spread between the 16 products (left in a row before them,
// they added a third to the step).  So are the loads (LOAD) of a coming
// expert's down rows, from wn.
template <bool LOAD>
__device__ __forceinline__ void rows_step(const DownRowsLds &S, char *yb, const RowTile &cur,
                                          RowTile &nxt, RowSums &prev, int slot,
                                          const uint4 (&W)[8], int col, int lane, uint4 (&Wn)[8],
                                          const uint16_t *wn) {
    f32x4 a[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    float2 y[4];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const int s = j >> 2;
        a[j & 1] = mfma16((j & 2) ? cur.lo[s] : cur.hi[s], W[4 * (j & 1) + s], a[j & 1]);
        if (j < 4) y[j] = sums_load(yb, prev, j);
        if (j == 5) rows_handover(cur);
        if (j >= 6 && j < 10) {
            nxt.hi[j - 6] = rows_frag(S.h[slot][0], j - 6, lane);
            nxt.lo[j - 6] = rows_frag(S.h[slot][1], j - 6, lane);
        }
        if (j == 10) nxt.off = *reinterpret_cast<const int4 *>(&S.off[slot][4 * (lane >> 4)]);
        if (LOAD && (j & 1)) Wn[j >> 1] = ldg16(wn + (j >> 1) * 512);
        if (j >= 11 && j < 15) sums_store(yb, y[j - 11], prev, j - 11);
        __builtin_amdgcn_sched_barrier(0);
    }
    prev.a0 = a[0];
    prev.a1 = a[1];
    prev.off[0] = cur.off.x + col;
    prev.off[1] = cur.off.y + col;
    prev.off[2] = cur.off.z + col;
    prev.off[3] = cur.off.w + col;
}

// One expert's run of `tiles` tiles on a multiplying wavefront; k: index of
// its first tile, whose fragments are in A; leaves the next run's first tile
// in A.  Loads a coming expert's down rows into Wn on the way.
template <bool LOAD>
__device__ __forceinline__ void rows_expert(const DownRowsLds &S, char *yb, RowTile &A, RowTile &B,
                                            RowSums &prev, int k, int tiles, const uint4 (&W)[8],
                                            int col, int lane, uint4 (&Wn)[8],
                                            const uint16_t *wn) {
    rows_step<LOAD>(S, yb, A, B, prev, (k + 1) & 1, W, col, lane, Wn, wn);
    for (; tiles > 2; tiles -= 2) {
        rows_step<false>(S, yb, B, A, prev, k & 1, W, col, lane, Wn, wn);
        rows_step<false>(S, yb, A, B, prev, (k + 1) & 1, W, col, lane, Wn, wn);
    }
    if (tiles == 2)
        rows_step<false>(S, yb, B, A, prev, k & 1, W, col, lane, Wn, wn);
    else
        A = B;
}

// A tile on its way through a carrying wavefront's registers.  The wavefront
// carries hi or lo (src) of eight places, two loads of four whole rows each
// (1 KiB in a piece where the run fills them); places past the run repeat its
// last row.
struct Carry {
    u32x4_t v[2];
    int tok, last;  // last: the tile's last place with a token
};

// d: the tile's list word; q0: the wavefront's first place
__device__ __forceinline__ void carry_issue(Carry &c, unsigned d, const uint16_t *src,
                                            const int32_t *pair_tok, int q0, int lane) {
    c.last = (int)(d >> 24);
    const size_t r0 = d & 0xFFFFFFu;
    const char *row = reinterpret_cast<const char *>(src + r0 * kExpertWidth);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const unsigned q = (unsigned)min(q0 + 4 * i + (lane >> 4), c.last);
        c.v[i] = *reinterpret_cast<const u32x4_t *>(row + (q * (kExpertWidth * 2u) +
                                                           16u * (lane & 15)));
    }
    c.tok = *reinterpret_cast<const int32_t *>(reinterpret_cast<const char *>(pair_tok + r0) +
                                               4u * (unsigned)min(lane & 15, c.last));
}

// A unit's place: the row blocks in groups of kRowGroup, a group's token
// chunks one after another.  An XCD works on consecutive units, about 4 row
// blocks by 8 chunks at a time: each chunk's h rows and each row block's
// weights are then shared in its L2, and the fewest bytes come from the
// Infinity Cache (16384 tokens of 112 experts at tau 0.9: 2.1 GB, against
// 9.7 GB with one row block for all 32 CUs of an XCD).
constexpr int kRowGroup = 4;
__device__ __forceinline__ void rows_place(int unit, int nRB, int nC, int &rb, int &c) {
    const int g = unit / (kRowGroup * nC), r = unit - g * kRowGroup * nC;
    const int w = min(kRowGroup, nRB - g * kRowGroup);
    c = r / w;
    rb = g * kRowGroup + r - c * w;
}

// A multiplying wavefront's unit of m experts, in whole rings and what is left:
// with the loop's only exit at its bottom, every wait covers the loads of the
// expert that is multiplied and leaves the next one's in flight (an exit inside
// the ring joined the loop head with fewer loads in flight, and the first
// expert of every ring waited for both: 95 us for 2048 tokens of the shape
// above, 88 so).
__device__ __forceinline__ void rows_multiply(const DownRowsLds &S, char *yb, const DNParams &P,
                                              int C, int rb, int m, int wv, int lane) {
    constexpr int kRing = kWAhead + 1;
    const size_t estride = (size_t)(P.d / 16) * 4 * 512;
    const int rt = min(rb * (kRowBlock / 16) + 2 * wv, P.d / 16 - 2);
    const uint16_t *wd = P.Wd + (size_t)rt * 4 * 512 + lane * 8;
    const int col = wv * 128 + (lane & 15) * 8;
    auto ent = [&](int i) { return __builtin_amdgcn_readfirstlane((int)S.ent[min(i, m - 1)]); };
    uint4 W[kRing][8];  // the down rows' two 16-row tiles that the wavefront owns
#pragma unroll
    for (int i = 0; i < kWAhead; ++i) {
        const uint16_t *w = wd + (size_t)(ent(i) & 255) * estride;
#pragma unroll
        for (int j = 0; j < 8; ++j) W[i][j] = ldg16(w + j * 512);
    }
    __syncthreads();  // tile 0 is in its slot
    RowTile A, B;
    rows_read(A, S, 0, lane);
    RowSums prev;
    prev.a0 = prev.a1 = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i) prev.off[i] = row_off(C) + col;
    int k = 0, x = 0;
    for (; x + kRing <= m; x += kRing) {
#pragma unroll
        for (int i = 0; i < kRing; ++i) {
            const int tiles = ent(x + i) >> 8;
            rows_expert<true>(S, yb, A, B, prev, k, tiles, W[i], col, lane, W[(i + kWAhead) % kRing],
                              wd + (size_t)(ent(x + i + kWAhead) & 255) * estride);
            k += tiles;
        }
    }
    // the experts past the last whole ring, whose down rows it has loaded
#pragma unroll
    for (int i = 0; i < kWAhead; ++i) {
        if (x + i < m) {
            const int tiles = ent(x + i) >> 8;
            rows_expert<false>(S, yb, A, B, prev, k, tiles, W[i], col, lane, W[i], wd);
            k += tiles;
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) sums_store(yb, sums_load(yb, prev, j), prev, j);
    // the carrying wavefronts end on a whole ring
    for (; k % kTileAhead != 0; ++k) __syncthreads();
}

// A carrying wavefront's unit (p: which of the four), in whole rings of tiles
// with one wait each: past the last tile it carries that tile again.
__device__ __forceinline__ void rows_carry(DownRowsLds &S, const uint32_t *list, const DNParams &P,
                                           int C, int t0, int steps, int p, int lane) {
    const int part = p & 1, q0 = 8 * (p >> 1);
    const uint16_t *src = part ? P.h_lo : P.h_hi;
    auto word = [&](int k) { return (int)list[min(k, steps - 1)]; };
    Carry ring[kTileAhead];
#pragma unroll
    for (int i = 0; i < kTileAhead; ++i) {
        carry_issue(ring[i], (unsigned)__builtin_amdgcn_readfirstlane(word(i)), src, P.pair_tok,
                    q0, lane);
        __builtin_amdgcn_sched_barrier(0);  // issued in order: the loop's waits count on it
    }
    int next = word(kTileAhead);
    for (int k0 = 0; k0 < steps; k0 += kTileAhead) {
#pragma unroll
        for (int i = 0; i < kTileAhead; ++i) {
            const unsigned d = (unsigned)__builtin_amdgcn_readfirstlane(next);
            Carry &cr = ring[i];
            // nothing of a later tile is computed here: it would be waited for
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("" : "+v"(cr.tok));
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int q = q0 + 4 * u + (lane >> 4);
                *reinterpret_cast<u32x4_t *>(&S.h[i % 2][part][q][(lane & 15) ^ q]) = cr.v[u];
            }
            // (every 16 lanes of the four wavefronts store the same offsets)
            const int q = lane & 15;
            S.off[i % 2][q] = row_off(q <= cr.last ? cr.tok - t0 : C);
            next = word(k0 + i + kTileAhead + 1);
            carry_issue(ring[i], d, src, P.pair_tok, q0, lane);
            __syncthreads();  // tile k0 + i is in its slot; the one before has been read
        }
    }
    __syncthreads();  // the last step's barrier
}

__global__ __launch_bounds__(kRowThreads, 1) void down_rows_k(DNParams P) {
    __shared__ __align__(16) unsigned char lds[kRowLds];
    DownRowsLds &S = *reinterpret_cast<DownRowsLds *>(lds);
    uint32_t *list = reinterpret_cast<uint32_t *>(lds + sizeof(DownRowsLds));
    float *y = reinterpret_cast<float *>(lds + sizeof(DownRowsLds) + pf_list_bytes(P.E, P.C));
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nC = P.nC, nRB = (P.d + kRowBlock - 1) / kRowBlock, units = nRB * nC;
    const int slots = 8 * ((units + 7) / 8);
    for (int slot = blockIdx.x; slot < slots; slot += gridDim.x) {
        const int unit = xcd_order(slot, units);
        if (unit >= units) continue;
        int rb, c;
        rows_place(unit, nRB, nC, rb, c);
        const int t0 = c * P.C, nt = min(P.C, P.T - t0);
        int n = 0, p0 = 0;  // expert tid's tokens in the chunk and their first pair
        if (tid < P.E) {
            const int a = P.cut[(size_t)tid * (nC + 1) + c];
            n = P.cut[(size_t)tid * (nC + 1) + c + 1] - a;
            p0 = P.ebase[tid] + a;
        }
        // a thread's values: rows r .. r + 3 and r + 16 .. r + 19.  The block's
        // rows past d (d a multiple of 64) are computed from its last valid
        // rows and not stored.
        const int nr = min(kRowBlock, P.d - rb * kRowBlock);
        constexpr int kQ = kRowBlock / 8;
        for (int i = tid; i < nt * kQ; i += kRowThreads) {
            const int t = i / kQ, q = i - t * kQ, r = 32 * (q >> 2) + 4 * (q & 3);
            float4 v0 = make_float4(0.f, 0.f, 0.f, 0.f), v1 = v0;
            if (P.bproj && r < nr) {
                const float *b = P.bproj + rb * kRowBlock + r;
                v0 = *reinterpret_cast<const float4 *>(b);
                v1 = *reinterpret_cast<const float4 *>(b + 16);
            }
            float4 *o = reinterpret_cast<float4 *>(&y[t * kRowBlock + 8 * q]);
            o[0] = make_float4(v0.x, v1.x, v0.y, v1.y);
            o[1] = make_float4(v0.z, v1.z, v0.w, v1.w);
        }
        const int tiles = (n + 15) >> 4;
        int slot_e, slot_t, m, steps;
        block_excl_scan2(n > 0 ? 1 : 0, tiles, &slot_e, &slot_t, &m, &steps, S.scan);
        if (n > 0) S.ent[slot_e] = (uint16_t)(tid | (tiles << 8));
        for (int i = 0; i < tiles; ++i)
            list[slot_t + i] = (uint32_t)(p0 + 16 * i) | ((uint32_t)(min(16, n - 16 * i) - 1) << 24);
        __syncthreads();
        m = __builtin_amdgcn_readfirstlane(m);
        steps = __builtin_amdgcn_readfirstlane(steps);
        if (m > 0) {
            if (wv < 4)
                rows_multiply(S, reinterpret_cast<char *>(y), P, P.C, rb, m, wv, lane);
            else
                rows_carry(S, list, P, P.C, t0, steps, wv - 4, lane);
        }
        __syncthreads();
        for (int i = tid; i < nt * kQ; i += kRowThreads) {
            const int t = i / kQ, q = i - t * kQ, r = 32 * (q >> 2) + 4 * (q & 3);
            if (r < nr) {
                const float4 *v = reinterpret_cast<const float4 *>(&y[t * kRowBlock + 8 * q]);
                const float4 a = v[0], b = v[1];
                float *o = P.y + (size_t)(t0 + t) * P.d + rb * kRowBlock + r;
                *reinterpret_cast<float4 *>(o) = make_float4(a.x, a.z, b.x, b.z);
                *reinterpret_cast<float4 *>(o + 16) = make_float4(a.y, a.w, b.y, b.w);
            }
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------------ launchers

DNParams dn_params(pp_layer *L, int T, float *y) {
    DNParams P;
    P.T = T;
    P.d = L->dm.d;
    P.E = L->dm.E;
    P.Wd = L->Wd;
    P.h_hi = L->h_hi;
    P.h_lo = L->h_lo;
    P.y = y;
    P.bproj = L->bproj;
    P.cut = L->pf_cut;
    const PfChunks ck = pf_chunks(P.d, P.E, T, L->num_cu);
    P.C = ck.C;
    P.nC = ck.n;
    P.ebase = L->pf_ebase;
    P.pair_tok = L->pair_tok;
    return P;
}

}  // namespace

// Gate/up of a decode batch in which every token keeps every expert (dense):
// the grouped kernel above, its groups from the decode plan.
void launch_gateup_dense_dec(pp_layer *L, const uint16_t *x, int T, hipStream_t s) {
    const GUParams gp = gu_params(L, x, T, false);
    if (L->gated)
        hipLaunchKernelGGL((gateup_pf_k<true, true>), dim3(L->num_cu), dim3(kGuThreads), 0, s, gp);
    else
        hipLaunchKernelGGL((gateup_pf_k<false, true>), dim3(L->num_cu), dim3(kGuThreads), 0, s, gp);
}

counter_layout counters_for(const pp_dims &dm, int max_tokens) {
    counter_layout c;
    c.route = 0;
    c.gateup = (size_t)plan_max_groups(dm, max_tokens);
    c.down = (size_t)((dm.d + 127) / 128);
    c.dispatch = 1;
    c.total = c.route + c.gateup + c.down + c.dispatch;
    return c;
}

hipError_t launch_prefill_ffn(pp_layer *L, const uint16_t *x, int T, float *y, hipStream_t s) {
    const pp_dims &dm = L->dm;
    const counter_layout cl = counters_for(dm, L->max_tokens);
    prof_mark(L, PP_KERNEL_DISPATCH, s, true);
    hipLaunchKernelGGL(dispatch_k, dim3(dm.E), dim3(256), 0, s, L->selmask, T, dm.E, L->ecount,
                       L->tokl, L->max_tokens, L->pf_cut, pf_chunks(dm.d, dm.E, T, L->num_cu),
                       L->pf_ebase, L->counters + cl.dispatch_base(), plan_view(L, true), L->num_cu);
    prof_mark(L, PP_KERNEL_DISPATCH, s, false);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    const GUParams gp = gu_params(L, x, T, true);
    prof_mark(L, PP_KERNEL_GATEUP, s, true);
    // one workgroup per CU (the kernel's registers and LDS allow no more)
    if (L->gated)
        hipLaunchKernelGGL((gateup_pf_k<true, false>), dim3(L->num_cu), dim3(kGuThreads), 0, s, gp);
    else
        hipLaunchKernelGGL((gateup_pf_k<false, false>), dim3(L->num_cu), dim3(kGuThreads), 0, s, gp);
    prof_mark(L, PP_KERNEL_GATEUP, s, false);
    err = hipGetLastError();
    if (err != hipSuccess) return err;
    const DNParams dp = dn_params(L, T, y);
    prof_mark(L, PP_KERNEL_DOWN, s, true);
    hipLaunchKernelGGL(down_rows_k, dim3(L->num_cu), dim3(kRowThreads), 0, s, dp);
    prof_mark(L, PP_KERNEL_DOWN, s, false);
    return hipGetLastError();
}

}  // namespace pp
