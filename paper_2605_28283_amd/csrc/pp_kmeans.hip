// Balanced k-means of neuron feature rows: MoEfication's clustering step
// (Sec. 2.2), which groups the d_ff intermediate neurons into E experts of
// exactly d_ff / E neurons and so defines the permutation Pi of
// Eq. (permuted_weights).  Lloyd's iteration under the balance constraint
// (the constrained k-means the paper cites):
//
//   assignment  minimise sum_i ||x_i - mu_a(i)||^2 with every cluster holding
//               exactly m = n / k rows: a transportation problem, solved
//               exactly by an ascending-price auction on the k cluster prices
//               lambda (dual variables).  Each round every row takes its exact
//               argmax of -s_ij - lambda_j (s_ij = ||mu_j||^2 - 2 x_i . mu_j,
//               the row's own ||x_i||^2 does not change the choice); every
//               over-full cluster raises its price by the (m+1)-th largest
//               margin (best minus second-best value) of its rows plus eps.
//               When no cluster is over-full all hold exactly m rows, and an
//               argmax assignment that is balanced is optimal by LP duality,
//               whatever eps was; eps only ends price wars, so it decays
//               geometrically (0.3 scale * 0.9^r, floor 2^-22 scale).  Small
//               steps cannot move a price far, so after kKmAuctionRounds
//               rounds the rest of the excess is routed by successive
//               shortest paths on the k-node cluster graph (edge a -> b: the
//               cheapest move of one of a's rows to b, minus the price
//               difference, >= 0 since every row sits at its argmax); each
//               augmentation moves one unit from an over-full to an
//               under-full cluster and updates the prices by the Dijkstra
//               distances (Johnson potentials), which keeps every row at its
//               argmax -- so the result stays exactly optimal.
//   update      mu_j = mean of the rows of cluster j (ascending row order).
//   Pi          clusters in index order, rows ascending inside each.
//
// Kernels: km_xnorm_k (||x_i||^2, fp64), km_split_k (mu as three bf16 parts
// mu = h + m + l exactly, and ||mu_j||^2), km_dist_k (s = ||mu||^2 - 2 F mu^T
// with bf16 MFMA 16x16x32 on the exact bf16 features and the three parts:
// products exact, fp32 accumulation), km_bid_k / km_price_k (one auction round
// each), km_members_k / km_ssp_rows_k / km_ssp_k (the shortest-path finish:
// member lists, edge rows, and the search in one workgroup), km_objective_k,
// km_perm_k, km_update_k.
#include <algorithm>
#include <cmath>
#include <utility>

#include "pp_internal.h"

namespace pp {
namespace {

constexpr int kKmMaxK = 256;
constexpr int kKmMaxN = 65536;
constexpr int kKmMaxD = 16384;
constexpr int kKmCols = 64;            // columns of mu staged in LDS per chunk
constexpr int kKmDistWaves = 4;        // km_dist_k: 4 wavefronts x 16 rows
constexpr int kKmBidRows = 64;         // rows per bid workgroup, one per lane
constexpr int kKmBidWaves = 8;         // its wavefronts, each an eighth of the clusters
constexpr int kKmPriceThreads = 1024;
constexpr int kKmAuctionRounds = 128;  // price rounds before the shortest-path finish
// eps of round 0, in units of the rows' mean spread of s.  The steps of all
// rounds together (ten times eps0) are about as far as a price moves, and rows
// of unequal norm need prices far apart: from 0.05 on, rows scaled by
// LogNormal(0, 0.2) leave 108 to 376 of the excess to the shortest-path finish
// (0.04 - 0.2 ms a unit), 0.3 leaves 3 to 11 (8192 x 64 and 14336 x 112,
// planted groups or none).  On rows of one norm 0.05 ends up to 20 rounds (0.2
// ms) earlier.  Steps that follow the excess instead end in price wars.
constexpr double kKmEps0 = 0.3;
constexpr int kKmBatch = 64;           // rounds enqueued between convergence checks
constexpr int kKmSspThreads = 1024;

struct KmWork {
    float *S;            // [k][n] s_ij, for the bids (lanes over rows)
    float *St;           // [n][k] the same, for the shortest-path finish (lanes over clusters)
    double *xnorm;       // [n]
    float *margin;       // [n] best minus second-best value of each row, rounded up to fp32
    int32_t *memb;       // [k][n] shortest-path finish: the rows of each cluster
    double *lam;         // [k] cluster prices
    double *part;        // [bid workgroups] spread sums, then [bid workgroups] = the eps scale
    float *cn;           // [k] ||mu_j||^2
    uint16_t *mu3;       // [3][k][D] bf16 parts of mu
    int32_t *count;      // [k] shortest-path finish: rows of each cluster
    double *base;        // [k][k] shortest-path finish: min over a's rows of s_ib - s_ia
    int32_t *bidx;       // [k][k] the row attaining it (lowest index on ties)
    int32_t *pos;        // [n] a row's place in its cluster's member list
    int32_t *flags;      // [0..1] over-full clusters of round r (by parity), [2] done,
                         // [3] rounds the step took
};

inline int bid_blocks(int n) { return (n + kKmBidRows - 1) / kKmBidRows; }

size_t align_up(size_t v) { return (v + 255) & ~(size_t)255; }

// Workspace carving (every region 256-byte aligned).
size_t km_layout(int n, int D, int k, KmWork *w, char *base) {
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char *p = base ? base + off : nullptr;
        off += align_up(bytes);
        return p;
    };
    KmWork t;
    t.S = reinterpret_cast<float *>(take(sizeof(float) * (size_t)k * n));
    t.St = reinterpret_cast<float *>(take(sizeof(float) * (size_t)k * n));
    t.xnorm = reinterpret_cast<double *>(take(sizeof(double) * n));
    t.margin = reinterpret_cast<float *>(take(sizeof(float) * (size_t)n));
    t.memb = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * (size_t)k * n));
    t.lam = reinterpret_cast<double *>(take(sizeof(double) * k));
    t.part = reinterpret_cast<double *>(take(sizeof(double) * (bid_blocks(n) + 1)));
    t.cn = reinterpret_cast<float *>(take(sizeof(float) * k));
    t.mu3 = reinterpret_cast<uint16_t *>(take(sizeof(uint16_t) * 3 * (size_t)k * D));
    t.count = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * k));
    t.base = reinterpret_cast<double *>(take(sizeof(double) * (size_t)k * k));
    t.bidx = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * (size_t)k * k));
    t.pos = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * n));
    t.flags = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * 4));
    if (w) *w = t;
    return off;
}

// ||x_i||^2 in fp64, one wavefront per row, lanes over 8-column groups in
// order, then a fixed butterfly.
__global__ __launch_bounds__(256) void km_xnorm_k(const uint16_t *__restrict__ F, int n, int D,
                                                  double *__restrict__ xnorm) {
    const int lane = threadIdx.x & 63;
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= n) return;
    const uint16_t *row = F + (size_t)i * D;
    double acc = 0.0;
    for (int c = 8 * lane; c < D; c += 512) {
        const uint4 v = ldg16(row + c);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double a = bf16_to_f32((uint16_t)(w[q] & 0xFFFFu));
            const double b = bf16_to_f32((uint16_t)(w[q] >> 16));
            acc += a * a + b * b;
        }
    }
#pragma unroll
    for (int st = 32; st >= 1; st >>= 1) acc += __shfl_xor(acc, st, 64);
    if (lane == 0) xnorm[i] = acc;
}

// mu_j as three bf16 parts (h = bf16(mu), m = bf16(mu - h), l = bf16(mu - h - m),
// each difference exact in fp32) and ||mu_j||^2 (fp64 in a fixed order,
// stored fp32).  One workgroup per centroid.
__global__ __launch_bounds__(256) void km_split_k(const float *__restrict__ mu, int k, int D,
                                                  uint16_t *__restrict__ mu3,
                                                  float *__restrict__ cn) {
    __shared__ double red[256];
    const int j = blockIdx.x, tid = threadIdx.x;
    double acc = 0.0;
    for (int c = tid; c < D; c += 256) {
        const float v = mu[(size_t)j * D + c];
        const uint16_t h = f32_to_bf16(v);
        const float r1 = v - bf16_to_f32(h);
        const uint16_t m = f32_to_bf16(r1);
        const uint16_t l = f32_to_bf16(r1 - bf16_to_f32(m));
        const size_t o = (size_t)j * D + c;
        mu3[o] = h;
        mu3[(size_t)k * D + o] = m;
        mu3[2 * (size_t)k * D + o] = l;
        acc += (double)v * v;
    }
    red[tid] = acc;
    __syncthreads();
    for (int s = 128; s >= 1; s >>= 1) {
        if (tid < s) red[tid] += red[tid + s];
        __syncthreads();
    }
    if (tid == 0) cn[j] = (float)red[0];
}

// s[j][i] = ||mu_j||^2 - 2 x_i . mu_j.  A workgroup owns 64 rows (16 per
// wavefront, the MFMA A operand straight from HBM, prefetched one chunk
// ahead; 14336 rows then fill 224 of the CUs); the three bf16 parts of mu,
// kKmCols columns at a time, are staged in LDS and shared by the wavefronts.
// A chunk is fetched into registers while the one before it is multiplied
// (fetched behind the barrier, 128 rows a workgroup, the kernel took 257 us
// for 14336 x 4096 x 112; now 113, where F alone is 25 at the copy rate.  Left
// out one at a time, the products save 30 %, the fetches of mu 14 %, F 11 % and
// the stores 4 %: one workgroup per CU chains them).  A fetch takes 128 bytes of eight rows of mu, whole
// cache lines; 16-byte piece c of row r lies at place c ^ (r % 8), so that a
// fragment's reads spread over all banks.  NT = ceil(k/16) cluster tiles per
// wavefront.
template <int NT>
__global__ __launch_bounds__(64 * kKmDistWaves, 1) void km_dist_k(const uint16_t *__restrict__ F,
                                                                 int n, int D, int k,
                                                                 const uint16_t *__restrict__ mu3,
                                                                 const float *__restrict__ cn,
                                                                 float *__restrict__ S,
                                                                 float *__restrict__ St) {
    // bs[part][tile][8 rows][row, piece]: 16 bytes each
    __shared__ u32x4_t bs[3][NT][2][64];
    static_assert(kKmCols == 64, "eight 16-byte pieces per row and chunk");
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int p = lane & 15, g = lane >> 4;
    const int i0 = blockIdx.x * (16 * kKmDistWaves) + wv * 16;
    const int row = min(i0 + p, n - 1);
    const uint16_t *frow = F + (size_t)row * D + 8 * g;
    f32x4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    constexpr int kSteps = kKmCols / 32;
    const size_t plane = (size_t)k * D;
    // the workgroup's 6 NT pieces of 64 x 16 bytes of a chunk, wavefront w
    // taking w, w + 4, ...
    constexpr int kPieces = 6 * NT, kPer = (kPieces + kKmDistWaves - 1) / kKmDistWaves;
    u32x4_t m[kPer];
    auto fetch = [&](int c0) {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int e = min(wv + u * kKmDistWaves, kPieces - 1);
            const int part = e / (2 * NT), th = e - part * (2 * NT);
            const int j = min(8 * th + (lane >> 3), k - 1);  // past k: columns never stored
            m[u] = *reinterpret_cast<const u32x4_t *>(mu3 + part * plane + (size_t)j * D + c0 +
                                                      8 * ((lane & 7) ^ (lane >> 3)));
        }
    };
    u32x4_t a[kSteps];
    fetch(0);
#pragma unroll
    for (int s = 0; s < kSteps; ++s) a[s] = *reinterpret_cast<const u32x4_t *>(frow + 32 * s);
    u32x4_t *flat = &bs[0][0][0][0];
    const int r = lane & 7;
    for (int c0 = 0; c0 < D; c0 += kKmCols) {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int e = wv + u * kKmDistWaves;
            if (e < kPieces) flat[e * 64 + lane] = m[u];
        }
        __syncthreads();
        // the next chunk (the last one again at the end)
        const int cn0 = min(c0 + kKmCols, D - kKmCols);
        fetch(cn0);
        u32x4_t an[kSteps];
#pragma unroll
        for (int s = 0; s < kSteps; ++s)
            an[s] = *reinterpret_cast<const u32x4_t *>(frow + cn0 + 32 * s);
#pragma unroll
        for (int s = 0; s < kSteps; ++s)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int part = 0; part < 3; ++part)
                    acc[t] = mfma16(__builtin_bit_cast(uint4, a[s]),
                                    __builtin_bit_cast(
                                        uint4, bs[part][t][(lane >> 3) & 1][8 * r + ((4 * s + g) ^ r)]),
                                    acc[t]);
        __syncthreads();
#pragma unroll
        for (int s = 0; s < kSteps; ++s) a[s] = an[s];
    }
    // lane holds rows i0 + 4 g + q (q < 4) of cluster t * 16 + p
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int j = t * 16 + p;
        if (j >= k) continue;
        const float c = cn[j];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = i0 + 4 * g + q;
            if (i < n) {
                const float v = c - 2.0f * acc[t][q];
                S[(size_t)j * n + i] = v;
                St[(size_t)i * k + j] = v;
            }
        }
    }
}

// Auction state for one assignment step: prices 0, flags clear.
__global__ void km_auction_init_k(int k, double *lam, int32_t *flags) {
    const int t = threadIdx.x;
    for (int j = t; j < k; j += blockDim.x) lam[j] = 0.0;
    if (t < 4) flags[t] = 0;
}

// (best, its cluster, second best) of part of a row's clusters; merging two
// parts gives the same result in any order: the better best wins (lower
// cluster on equal values), the second is the larger of the kept second and
// the other best.
struct Best2 {
    double w1, w2;
    int j1;
    float smin, smax;
};
__device__ __forceinline__ Best2 merge_best2(Best2 a, Best2 b) {
    if (b.w1 > a.w1 || (b.w1 == a.w1 && b.j1 < a.j1)) {
        const Best2 t = a;
        a = b;
        b = t;
    }
    a.w2 = fmax(a.w2, b.w1);
    a.smin = fminf(a.smin, b.smin);
    a.smax = fmaxf(a.smax, b.smax);
    return a;
}

// Round r, bids: every row's argmax j1 of w_ij = -s_ij - lambda_j (first
// index on ties) and its margin w1 - w2 (w2 the best over the other
// clusters), rounded up to fp32.  A lane owns a row, a wavefront an eighth of
// the clusters (its loads 16 at a time in flight, 256 contiguous bytes each),
// and the wavefronts' partial results are merged through LDS.  Latency-bound
// (6.4 MB of s for 14336 x 112): the row is only written down here -- the
// price kernel sorts the rows by cluster itself, which costs it less than
// lists appended through device-wide counters cost this kernel (LLaMA-3-8B
// layer, a round of both kernels: 16.6 us with the lists).  Exits at once when
// the previous round left no cluster over-full (the assignment then stands).
__global__ __launch_bounds__(64 * kKmBidWaves) void km_bid_k(const float *__restrict__ S, int n,
                                                             int k, int r, KmWork W,
                                                             int32_t *__restrict__ assign) {
    constexpr int kBatch = 16;  // a lane's clusters in flight at once (k <= 128: all of them)
    __shared__ Best2 part[kKmBidWaves][kKmBidRows];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (W.flags[2]) return;
    if (r > 0 && W.flags[(r - 1) & 1] == 0) {
        if (blockIdx.x == 0 && tid == 0) {
            W.flags[2] = 1;
            W.flags[3] = r;
        }
        return;
    }
    if (blockIdx.x == 0 && tid == 0) W.flags[r & 1] = 0;
    const int i = blockIdx.x * kKmBidRows + lane;
    const bool valid = i < n;
    const int ii = min(i, n - 1);
    const int per = (k + kKmBidWaves - 1) / kKmBidWaves;
    const int jA = wv * per, jB = min(jA + per, k);
    Best2 v{-INFINITY, -INFINITY, 0x7FFFFFFF, INFINITY, -INFINITY};
    for (int j0 = jA; j0 < jB; j0 += kBatch) {
        float sv[kBatch];
        double lam[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int j = min(j0 + u, k - 1);
            sv[u] = S[(size_t)j * n + ii];
            lam[u] = W.lam[j];
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int j = j0 + u;
            if (j < jB) {
                const double w = -(double)sv[u] - lam[u];
                const bool b1 = w > v.w1;  // ascending j: the first wins ties
                v.w2 = b1 ? v.w1 : fmax(v.w2, w);
                v.w1 = b1 ? w : v.w1;
                v.j1 = b1 ? j : v.j1;
                v.smin = fminf(v.smin, sv[u]);
                v.smax = fmaxf(v.smax, sv[u]);
            }
        }
    }
    part[wv][lane] = v;
    __syncthreads();
    if (wv != 0) return;
#pragma unroll
    for (int w = 1; w < kKmBidWaves; ++w) v = merge_best2(v, part[w][lane]);
    if (valid) {
        const double mg = v.w1 - v.w2;  // +inf when k == 1
        assign[i] = min(v.j1, k - 1);  // (NaN features choose no cluster)
        W.margin[i] = isinf(mg) ? 3.0e38f : __double2float_ru(mg);
    }
    if (r == 0) {  // eps scale: sum of per-row spreads, fixed order
        // (a row of NaNs has none)
        double sp = valid && v.smin <= v.smax ? (double)v.smax - (double)v.smin : 0.0;
#pragma unroll
        for (int st = 32; st >= 1; st >>= 1) sp += __shfl_xor(sp, st, 64);
        if (lane == 0) W.part[blockIdx.x] = sp;
    }
}

// Round r, prices: one workgroup per cluster.  It gathers the margins of its
// rows in LDS (reading every row's cluster, 16 rows a thread at once), and an
// over-full cluster finds the (m+1)-th largest of them by a radix select on
// the fp32 bits in three passes of 11, 11 and 10 bits (margins are >= 0, so
// bit order is value order; the order they were gathered in does not matter)
// and raises its price by that margin plus eps (the round's, in units of the
// eps scale); it also counts itself in flags[r & 1].  More than kKmPriceLds
// rows are read again from memory by every pass.  The eps scale (the round-0
// spread sums, in a fixed order) is formed in round 0 and kept in part[nbid].
constexpr int kKmPriceLds = 8192;
constexpr int kKmDigits = 2048;

__global__ __launch_bounds__(kKmPriceThreads) void km_price_k(int n, int m, int r, int nbid,
                                                              double eps, KmWork W,
                                                              const int32_t *__restrict__ assign) {
    constexpr int kBatch = 16;
    static_assert(kKmDigits == 2 * kKmPriceThreads, "two digits per thread");
    __shared__ int hist[kKmDigits];
    __shared__ int scan[2 * (kKmPriceThreads / 64)];
    __shared__ uint32_t s_pref;
    __shared__ int s_rank, s_c;
    __shared__ uint32_t sl[kKmPriceLds];
    const int j = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    auto rows = [&](int i0, int (&a)[kBatch], uint32_t (&v)[kBatch]) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int i = min(i0 + u * kKmPriceThreads + tid, n - 1);
            a[u] = assign[i];
            v[u] = __float_as_uint(W.margin[i]);
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
            if (i0 + u * kKmPriceThreads + tid >= n) a[u] = -1;
    };
    const int done = W.flags[2];
    int a[kBatch];  // the first rows' loads do not wait for the flag
    uint32_t v[kBatch];
    rows(0, a, v);
    if (done) return;
    if (tid == 0) {
        s_c = 0;
        s_pref = 0u;
        s_rank = m;  // 0-based rank from the top
    }
    hist[tid] = 0;
    hist[tid + kKmPriceThreads] = 0;
    __syncthreads();
    for (int i0 = 0;;) {
        // one counter update per wavefront
        unsigned long long mine[kBatch];
        int total = 0;
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            mine[u] = __ballot(a[u] == j);
            total += __popcll(mine[u]);
        }
        if (total) {
            int at = 0;
            if (lane == 0) at = atomicAdd(&s_c, total);
            at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                if (a[u] == j) {
                    const int o = at + __popcll(mine[u] & ((1ull << lane) - 1ull));
                    if (o < kKmPriceLds) sl[o] = v[u];
                    atomicAdd(&hist[v[u] >> 21], 1);  // the first pass's digits
                }
                at += __popcll(mine[u]);
            }
        }
        i0 += kBatch * kKmPriceThreads;
        if (i0 >= n) break;
        rows(i0, a, v);
    }
    __syncthreads();
    const int c = s_c;
    if (c <= m) return;
    const bool inl = c <= kKmPriceLds;  // workgroup-uniform
    uint32_t mask = 0u;
#pragma unroll
    for (int pass = 0; pass < 3; ++pass) {
        const int shift = pass == 0 ? 21 : (pass == 1 ? 10 : 0);
        const uint32_t digits = pass == 2 ? 1023u : 2047u;
        if (pass > 0) {
            hist[tid] = 0;
            hist[tid + kKmPriceThreads] = 0;
            __syncthreads();
            const uint32_t pref = s_pref;
            if (inl) {
                for (int i = tid; i < c; i += kKmPriceThreads)
                    if ((sl[i] & mask) == pref) atomicAdd(&hist[(sl[i] >> shift) & digits], 1);
            } else {
                for (int i0 = 0; i0 < n; i0 += kBatch * kKmPriceThreads) {
                    rows(i0, a, v);
#pragma unroll
                    for (int u = 0; u < kBatch; ++u)
                        if (a[u] == j && (v[u] & mask) == pref)
                            atomicAdd(&hist[(v[u] >> shift) & digits], 1);
                }
            }
            __syncthreads();
        }
        // digits from the top, two to a thread; the selected digit is where
        // the running count first exceeds the rank
        const int d0 = kKmDigits - 1 - 2 * tid, h0 = hist[d0], h1 = hist[d0 - 1];
        const int rank = s_rank;
        const uint32_t pref = s_pref;
        int ex, ex1, tot, tot1;
        block_excl_scan2(h0 + h1, 0, &ex, &ex1, &tot, &tot1, scan);
        if (ex <= rank && rank < ex + h0 + h1) {
            const bool first = rank < ex + h0;
            s_rank = rank - ex - (first ? 0 : h0);
            s_pref = pref | ((uint32_t)(first ? d0 : d0 - 1) << shift);
        }
        mask |= digits << shift;
        __syncthreads();
    }
    if (tid < 64) {
        double scale = 0.0;
        if (r == 0) {  // every over-full cluster forms the same value
            for (int b = lane; b < nbid; b += 64) scale += W.part[b];
#pragma unroll
            for (int st = 32; st >= 1; st >>= 1) scale += __shfl_xor(scale, st, 64);
            scale /= (double)n;
            if (lane == 0) W.part[nbid] = scale;
        } else {
            scale = W.part[nbid];
        }
        if (lane == 0) {
            W.lam[j] += (double)__uint_as_float(s_pref) + eps * scale;
            atomicAdd(&W.flags[r & 1], 1);
        }
    }
}

// The members of every cluster after a bid round, ascending, for the
// shortest-path finish: one workgroup per cluster.
__global__ __launch_bounds__(1024) void km_members_k(const int32_t *__restrict__ assign, int n,
                                                     KmWork W) {
    __shared__ int scan[32];
    const int j = blockIdx.x, tid = threadIdx.x;
    int base = 0;
    for (int i0 = 0; i0 < n; i0 += 1024) {
        const int i = i0 + tid;
        const int f = (i < n && assign[i] == j) ? 1 : 0;
        int ex, ex1, tot, tot1;
        block_excl_scan2(f, 0, &ex, &ex1, &tot, &tot1, scan);
        if (f) {
            W.memb[(size_t)j * n + base + ex] = i;
            W.pos[i] = base + ex;
        }
        base += tot;
    }
    if (tid == 0) W.count[j] = base;
}

// LDS of one edge row: a batch of the cluster's rows, and the wavefronts'
// minima.
struct SspRowLds {
    int row[kKmSspThreads];
    double best[kKmSspThreads / 64][kKmMaxK / 2];
    int bi[kKmSspThreads / 64][kKmMaxK / 2];
};

// Edge row a of the shortest-path finish: base[b] = min over a's rows i of
// s_bi - s_ai and bidx[b] the row attaining it (lowest index on ties, so the
// member-list order does not matter); b = a and empty clusters give +inf.
// Called by the whole workgroup: wavefront w takes rows w, w + 16, ..., its
// lanes the clusters, so a row is read as its k consecutive values of St (with
// lanes over rows instead, each value was a cache line of its own and an edge
// row took 14 us, 128 rows of 112 clusters).
__device__ __forceinline__ void ssp_row(const float *__restrict__ St, int n, int k, int a, int na,
                                        const int32_t *memb, double *base, int32_t *bidx,
                                        SspRowLds &R) {
    constexpr int kWaves = kKmSspThreads / 64, kV = kKmMaxK / 64, kB = 8;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    double best[kV];
    int bi[kV];
#pragma unroll
    for (int q = 0; q < kV; ++q) {
        best[q] = INFINITY;
        bi[q] = 0x7FFFFFFF;
    }
    for (int t0 = 0; t0 < na; t0 += kKmSspThreads) {
        const int nt = min(kKmSspThreads, na - t0);
        if (tid < nt) R.row[tid] = memb[(size_t)a * n + t0 + tid];
        __syncthreads();
        for (int u0 = wv; u0 < nt; u0 += kB * kWaves) {
            int row[kB];
            float sv[kB][kV];
#pragma unroll
            for (int u = 0; u < kB; ++u) {
                // past the batch: its last row again
                row[u] = __builtin_amdgcn_readfirstlane(R.row[min(u0 + u * kWaves, nt - 1)]);
                const float *p = St + (size_t)row[u] * k;
#pragma unroll
                for (int q = 0; q < kV; ++q) sv[u][q] = 64 * q < k ? p[min(lane + 64 * q, k - 1)] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < kB; ++u) {
                float own = sv[u][0];
#pragma unroll
                for (int q = 1; q < kV; ++q) own = a >> 6 == q ? sv[u][q] : own;
                own = lane_value(own, a & 63);
#pragma unroll
                for (int q = 0; q < kV; ++q) {
                    const double v = (double)sv[u][q] - (double)own;
                    if (v < best[q] || (v == best[q] && row[u] < bi[q])) {
                        best[q] = v;
                        bi[q] = row[u];
                    }
                }
            }
        }
        __syncthreads();
    }
    // the wavefronts' minima, half of the clusters at a time
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if (128 * h >= k) break;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            R.best[wv][lane + 64 * q] = best[2 * h + q];
            R.bi[wv][lane + 64 * q] = bi[2 * h + q];
        }
        __syncthreads();
        const int b = 128 * h + tid;
        if (tid < 128 && b < k) {
            double v = R.best[0][tid];
            int i = R.bi[0][tid];
#pragma unroll
            for (int w = 1; w < kWaves; ++w) {
                const double o = R.best[w][tid];
                const int oi = R.bi[w][tid];
                if (o < v || (o == v && oi < i)) {
                    v = o;
                    i = oi;
                }
            }
            base[b] = b == a ? (double)INFINITY : v;
            bidx[b] = b == a ? 0x7FFFFFFF : i;
        }
        __syncthreads();
    }
}

// All edge rows at once, one workgroup per cluster, from the member lists of
// the bid round that precedes the finish (its argmax matches the prices).
__global__ __launch_bounds__(kKmSspThreads) void km_ssp_rows_k(int n, int k, KmWork W) {
    __shared__ SspRowLds R;
    const int a = blockIdx.x;
    ssp_row(W.St, n, k, a, W.count[a], W.memb, W.base + (size_t)a * k, W.bidx + (size_t)a * k, R);
}

// The smallest (value, index) over the wavefront, lower index on equal values.
template <int ST>
__device__ __forceinline__ void wave_min_step(double &d, int &v, int lane) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(d);
    const uint32_t lo = xor_lane<ST>((uint32_t)u, lane), hi = xor_lane<ST>((uint32_t)(u >> 32), lane);
    const double od = __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
    const int ov = (int)xor_lane<ST>((uint32_t)v, lane);
    if (od < d || (od == d && ov < v)) {
        d = od;
        v = ov;
    }
}
__device__ __forceinline__ void wave_min(double &d, int &v, int lane) {
    wave_min_step<1>(d, v, lane);
    wave_min_step<2>(d, v, lane);
    wave_min_step<4>(d, v, lane);
    wave_min_step<8>(d, v, lane);
    wave_min_step<16>(d, v, lane);
    wave_min_step<32>(d, v, lane);
}

// Shortest-path finish of an assignment step (one workgroup; every loop is
// bounded by n, the largest possible excess).  Starts from the bid round's
// argmax assignment, counts and member lists, then per augmentation:
// multi-source Dijkstra from the over-full clusters over reduced costs
// max(0, base[u][v] + lambda_v - lambda_u) until the first under-full
// cluster t is settled; the path's rows move one edge each; lambda_v -=
// min(dist_v, dist_t); the edge rows of the clusters on the path are
// recomputed.  Sets flags[2] when balanced, flags[3] = augmentations.
// An edge without a row (base = +inf: u is empty, or its rows' values at v are
// not numbers) is never taken, whatever the prices make of its cost, as
// bidx[u][v] then names no row; prices that are not finite (features or
// centroids were not) end the step unbalanced, for they order nothing.
// A chain of latencies: the search runs in one wavefront, its labels in
// registers, and with LDS the edge costs lie in LDS, so a step costs no barrier
// and no memory round trip: whenever the k x k of them fit beside the rest
// (k <= 126: 127 units of excess among 126 clusters of 128 rows of 512, a whole
// call: 19.3 ms, 21.7 ms with the costs in memory).  16: the two ints behind the
// arrays, and padding.
constexpr int kKmSspFixed = 2 * kKmMaxK * sizeof(double) + 3 * kKmMaxK * sizeof(int) +
                            sizeof(SspRowLds) + 16;
constexpr int kKmSspEdges = (160 * 1024 - kKmSspFixed) / 16 * 2;
static_assert(kKmSspEdges >= 126 * 126, "edge costs of 126 clusters");

template <bool LDS>
__global__ __launch_bounds__(kKmSspThreads) void km_ssp_k(int n, int k, int m, KmWork W,
                                                          int32_t *__restrict__ assign) {
    constexpr int kV = kKmMaxK / 64;  // clusters per lane
    __shared__ double lam[kKmMaxK], dist[kKmMaxK];
    __shared__ int cnt[kKmMaxK], pred[kKmMaxK], chg[kKmMaxK];
    __shared__ int s_t, s_excess;
    __shared__ SspRowLds R;
    __shared__ double edges[LDS ? kKmSspEdges : 1];
    double *base = LDS ? edges : W.base;
    int32_t *memb = W.memb;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    for (int j = tid; j < k; j += kKmSspThreads) {
        lam[j] = W.lam[j];
        cnt[j] = W.count[j];
    }
    if (LDS)
        for (int i = tid; i < k * k; i += kKmSspThreads) edges[i] = W.base[i];
    __syncthreads();
    int aug = 0;
    for (; aug <= n; ++aug) {
        for (int v = tid; v < k; v += kKmSspThreads) chg[v] = 0;
        if (wv == 0) {
            double d[kV], lv[kV];
            int pr[kV];
            bool open[kV];
            int ex = 0;
            bool finite = true;
#pragma unroll
            for (int q = 0; q < kV; ++q) {
                const int v = lane + 64 * q, c = v < k ? cnt[v] : m;
                open[q] = v < k;
                d[q] = c > m ? 0.0 : INFINITY;
                lv[q] = v < k ? lam[v] : 0.0;
                pr[q] = -1;
                finite = finite && isfinite(lv[q]);
                ex += c > m ? c - m : 0;
            }
#pragma unroll
            for (int st = 32; st >= 1; st >>= 1) ex += __shfl_xor(ex, st, 64);
            int t = -1;
            if (ex > 0 && __all(finite)) {
                // Dijkstra until the first under-full cluster is settled
                for (int step = 0; step < k; ++step) {
                    double bd = INFINITY;
                    int bu = 0x7FFFFFFF;
#pragma unroll
                    for (int q = 0; q < kV; ++q)
                        if (open[q] && d[q] < bd) {  // ascending clusters: the first wins ties
                            bd = d[q];
                            bu = lane + 64 * q;
                        }
                    wave_min(bd, bu, lane);
                    const int u = __builtin_amdgcn_readfirstlane(bu);
                    if (u >= k) break;  // nothing within reach
                    if (cnt[u] < m) {
                        t = u;
                        break;
                    }
                    const double lu = lam[u];
#pragma unroll
                    for (int q = 0; q < kV; ++q) {
                        const int v = lane + 64 * q;
                        if (v == u) open[q] = false;
                        if (open[q]) {
                            const double c = base[(size_t)u * k + v];
                            const double nd = bd + fmax(0.0, c + lv[q] - lu);
                            if (c < INFINITY && nd < d[q]) {
                                d[q] = nd;
                                pr[q] = u;
                            }
                        }
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < kV; ++q) {
                const int v = lane + 64 * q;
                if (v < k) {
                    dist[v] = d[q];
                    pred[v] = pr[q];
                }
            }
            if (lane == 0) {
                s_excess = ex;
                s_t = t;
            }
        }
        __syncthreads();
        if (s_excess == 0) break;
        const int t = s_t;
        if (t < 0) break;  // no path: leaves flags[2] clear
        if (tid == 0) {  // move one row along each edge of the path, t back to its source
            for (int v = t, guard = 0; pred[v] >= 0 && guard < k; ++guard) {
                const int u = pred[v];
                const int p = W.bidx[(size_t)u * k + v];
                const int pu = W.pos[p], last = memb[(size_t)u * n + cnt[u] - 1];
                memb[(size_t)u * n + pu] = last;
                W.pos[last] = pu;
                memb[(size_t)v * n + cnt[v]] = p;
                W.pos[p] = cnt[v];
                --cnt[u];
                ++cnt[v];
                assign[p] = v;
                chg[u] = chg[v] = 1;
                v = u;
            }
        }
        const double dt = dist[t];
        for (int v = tid; v < k; v += kKmSspThreads) lam[v] -= fmin(dist[v], dt);
        __syncthreads();
        for (int a = 0; a < k; ++a)
            if (chg[a])
                ssp_row(W.St, n, k, a, cnt[a], memb, base + (size_t)a * k, W.bidx + (size_t)a * k, R);
        __syncthreads();
    }
    for (int j = tid; j < k; j += kKmSspThreads) W.lam[j] = lam[j];
    if (tid == 0) {
        W.flags[2] = s_excess == 0 ? 1 : 0;
        W.flags[3] = aug;
    }
}

// sum_i ||x_i - mu_a(i)||^2 = sum_i (||x_i||^2 + s_{a(i), i}), fp64, one
// workgroup, thread t takes rows t, t + 1024, ... then a fixed tree.
__global__ __launch_bounds__(1024) void km_objective_k(const float *__restrict__ S,
                                                       const double *__restrict__ xnorm,
                                                       const int32_t *__restrict__ assign, int n,
                                                       float *__restrict__ out) {
    __shared__ double red[1024];
    const int tid = threadIdx.x;
    double acc = 0.0;
#pragma unroll 8
    for (int i = tid; i < n; i += 1024) acc += xnorm[i] + (double)S[(size_t)assign[i] * n + i];
    red[tid] = acc;
    __syncthreads();
    for (int s = 512; s >= 1; s >>= 1) {
        if (tid < s) red[tid] += red[tid + s];
        __syncthreads();
    }
    if (tid == 0) *out = (float)red[0];
}

// Pi: cluster j's rows, ascending, at perm[j m ..].  One workgroup per
// cluster, a block scan over the rows in order.
__global__ __launch_bounds__(1024) void km_perm_k(const int32_t *__restrict__ assign, int n, int m,
                                                  int32_t *__restrict__ perm) {
    __shared__ int scan[32];
    const int j = blockIdx.x, tid = threadIdx.x;
    int base = 0;
    for (int i0 = 0; i0 < n; i0 += 1024) {
        const int i = i0 + tid;
        const int f = (i < n && assign[i] == j) ? 1 : 0;
        int ex, ex1, tot, tot1;
        block_excl_scan2(f, 0, &ex, &ex1, &tot, &tot1, scan);
        if (f && base + ex < m) perm[(size_t)j * m + base + ex] = i;
        base += tot;
    }
}

// mu_j[c] = mean over cluster j's rows (Pi order, fp64 sum), grid (k, D/256).
__global__ __launch_bounds__(256) void km_update_k(const uint16_t *__restrict__ F, int D, int m,
                                                   const int32_t *__restrict__ perm,
                                                   float *__restrict__ mu) {
    const int j = blockIdx.x, c = blockIdx.y * 256 + threadIdx.x;
    if (c >= D) return;
    double acc = 0.0;
#pragma unroll 8
    for (int t = 0; t < m; ++t) acc += bf16_to_f32(F[(size_t)perm[(size_t)j * m + t] * D + c]);
    mu[(size_t)j * D + c] = (float)(acc / (double)m);
}

__global__ void km_prices_out_k(const double *__restrict__ lam, int k, float *__restrict__ out) {
    for (int j = threadIdx.x; j < k; j += blockDim.x) out[j] = (float)lam[j];
}

template <int NT>
void launch_dist_nt(const uint16_t *F, int n, int D, int k, const KmWork &W, hipStream_t s) {
    const int blocks = (n + 16 * kKmDistWaves - 1) / (16 * kKmDistWaves);
    hipLaunchKernelGGL(km_dist_k<NT>, dim3(blocks), dim3(64 * kKmDistWaves), 0, s, F, n, D, k,
                       W.mu3, W.cn, W.S, W.St);
}

template <int... Q>
void launch_dist(int nt, const uint16_t *F, int n, int D, int k, const KmWork &W, hipStream_t s,
                 std::integer_sequence<int, Q...>) {
    ((nt == Q + 1 ? launch_dist_nt<Q + 1>(F, n, D, k, W, s) : void()), ...);
}

}  // namespace
}  // namespace pp

extern "C" size_t prunepath_kmeans_workspace(int32_t n, int32_t D, int32_t k) {
    if (k < 1 || k > pp::kKmMaxK || n < k || n > pp::kKmMaxN || n % k != 0) return 0;
    if (D < 64 || D > pp::kKmMaxD || D % 64 != 0) return 0;
    return pp::km_layout(n, D, k, nullptr, nullptr);
}

extern "C" pp_status prunepath_balanced_kmeans(const uint16_t *F, int32_t n, int32_t D, int32_t k,
                                               const float *init_centroids, int32_t iters,
                                               int32_t *assign, int32_t *perm, float *centroids,
                                               float *objective, float *prices, int32_t *rounds,
                                               void *workspace, void *hip_stream) {
    using namespace pp;
    if (!F || !init_centroids || !assign || !perm || !centroids || !workspace) return PP_EINVAL;
    if (prunepath_kmeans_workspace(n, D, k) == 0 || iters < 1 || iters > 1000) return PP_EINVAL;
    if ((reinterpret_cast<uintptr_t>(F) | reinterpret_cast<uintptr_t>(workspace)) & 15)
        return PP_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    KmWork W;
    km_layout(n, D, k, &W, static_cast<char *>(workspace));
    const int m = n / k, nbid = bid_blocks(n), nt = (k + 15) / 16;
    hipError_t e = hipSuccess;
    if (centroids != init_centroids)
        e = hipMemcpyAsync(centroids, init_centroids, sizeof(float) * (size_t)k * D,
                           hipMemcpyDeviceToDevice, s);
    if (e != hipSuccess) return PP_EHIP;
    hipLaunchKernelGGL(km_xnorm_k, dim3((n + 3) / 4), dim3(256), 0, s, F, n, D, W.xnorm);
    pp_status status = PP_OK;
    for (int it = 0; it < iters && status == PP_OK; ++it) {
        hipLaunchKernelGGL(km_split_k, dim3(k), dim3(256), 0, s, centroids, k, D, W.mu3, W.cn);
        launch_dist(nt, F, n, D, k, W, s, std::make_integer_sequence<int, kKmMaxK / 16>{});
        hipLaunchKernelGGL(km_auction_init_k, dim3(1), dim3(256), 0, s, k, W.lam, W.flags);
        int r = 0, used = 0;
        bool done = false;
        while (!done && r < kKmAuctionRounds) {
            const int r1 = r + kKmBatch;
            for (; r < r1; ++r) {
                hipLaunchKernelGGL(km_bid_k, dim3(nbid), dim3(64 * kKmBidWaves), 0, s, W.S, n, k,
                                   r, W, assign);
                hipLaunchKernelGGL(km_price_k, dim3(k), dim3(kKmPriceThreads), 0, s, n, m, r, nbid,
                                   std::max(kKmEps0 * std::pow(0.9, r), 0x1p-22), W, assign);
            }
            int32_t fl[4];
            if (hipMemcpyAsync(fl, W.flags, sizeof fl, hipMemcpyDeviceToHost, s) != hipSuccess ||
                hipStreamSynchronize(s) != hipSuccess)
                return PP_EHIP;
            // converged when a round left no cluster over-full: either a later
            // bid round saw it (done flag) or it was the last round enqueued
            done = fl[2] != 0 || fl[(r - 1) & 1] == 0;
            used = fl[2] != 0 ? fl[3] : r;
        }
        if (!done) {  // route the remaining excess by shortest paths
            // one more bid round: the argmax of the current prices (no price
            // round follows it), and the clusters' member lists
            hipLaunchKernelGGL(km_bid_k, dim3(nbid), dim3(64 * kKmBidWaves), 0, s, W.S, n, k, r, W,
                               assign);
            hipLaunchKernelGGL(km_members_k, dim3(k), dim3(1024), 0, s, assign, n, W);
            hipLaunchKernelGGL(km_ssp_rows_k, dim3(k), dim3(kKmSspThreads), 0, s, n, k, W);
            if (k * k <= kKmSspEdges)
                hipLaunchKernelGGL(km_ssp_k<true>, dim3(1), dim3(kKmSspThreads), 0, s, n, k, m, W,
                                   assign);
            else
                hipLaunchKernelGGL(km_ssp_k<false>, dim3(1), dim3(kKmSspThreads), 0, s, n, k, m,
                                   W, assign);
            int32_t fl[4];
            if (hipMemcpyAsync(fl, W.flags, sizeof fl, hipMemcpyDeviceToHost, s) != hipSuccess ||
                hipStreamSynchronize(s) != hipSuccess)
                return PP_EHIP;
            done = fl[2] != 0;
            used = r + fl[3];
        }
        if (rounds) rounds[it] = done ? used : -1;
        if (!done) {
            status = PP_ENOTCONVERGED;
            break;
        }
        if (objective)
            hipLaunchKernelGGL(km_objective_k, dim3(1), dim3(1024), 0, s, W.S, W.xnorm, assign, n,
                               objective + it);
        hipLaunchKernelGGL(km_perm_k, dim3(k), dim3(1024), 0, s, assign, n, m, perm);
        hipLaunchKernelGGL(km_update_k, dim3(k, (D + 255) / 256), dim3(256), 0, s, F, D, m, perm,
                           centroids);
    }
    if (prices) hipLaunchKernelGGL(km_prices_out_k, dim3(1), dim3(256), 0, s, W.lam, k, prices);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess) return PP_EHIP;
    return status;
}
