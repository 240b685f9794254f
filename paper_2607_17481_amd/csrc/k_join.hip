// k_join.hip -- the certificate's exact threshold join, as MFMA tiles.
//
// After the one pass the profile is a sound upper bound (Prop. 1); let T be
// the k-th value the greedy accepts on it.  A pair at distance d <= T has, by
// Lemma 2, true features within T sqrt(m/2) of each other, hence working
// vectors G (the stored features rounded to fp16) within
//   R = T sqrt(m/2) + e'_i + e'_j,     e' >= ||G - F||
// (the record's bound, the FP32 rounding and the fp16 rounding itself, which
// k_join_ops measures window by window; features off by more than their range
// give way to G = 0, which is within the largest possible norm of any F).  The
// join finds every such pair:
//
//  * grid: each length's windows get coordinates, the projections of their
//    FP32 feature copies f on the leading principal directions of that
//    length's features (orthonormal, so a coordinate moves by at most
//    ||df|| <= R_f = T sqrt(m/2) + e_i + e_j + u32 (|F~_i| + |F~_j|)); two of
//    them, in cells of width h >= R_f, place a pair within R_f in adjacent
//    cells (or one, in finer cells, when R_f is below the two-coordinate
//    grid's resolution), and all three must differ by at most R_f;
//  * tiles: windows sorted by (length, cell) are cut into blocks of 128
//    queries, one wavefront each; its candidates are the windows of the cells
//    next to its queries' cells (each a contiguous run of the order), taken 32
//    at a time against the four query tiles of 32;
//  * filter: for a 32 x 32 tile, <G_q, G_c> comes from two fp16 MFMA products
//    (the products are exact in FP32, which also accumulates them), and
//      ||dG||^2 = |G_q|^2 + |G_c|^2 - 2 <G_q, G_c>
//    is bounded below with a rigorous rounding margin; a pair is kept unless
//    that bound exceeds R^2.  It is a prefilter only: what it rejects provably
//    lies past T, and what it keeps is decided on the stored records and the
//    FP64 distance, so its 16 bits touch no result;
//  * exact: kept pairs pass the exclusion test, the certified Parseval bound
//    from the stored records (<= T and below one of the two cells) and are
//    verified with the canonical FP64 distance, lowering both cells.  The
//    tiles hand their kept pairs to a buffer, and the exact stage runs as a
//    kernel of its own (k_join_verify) after each chunk of tiles.
//
// Every unordered pair is examined once: a pair whose other end is itself a
// query and comes earlier in the order is left to that end's block (both ends
// see each other, since cell adjacency is symmetric and the filter is
// conservative on both sides).  At a length where every window is a query (no
// cell at 0: the usual case while T > 0) a block skips the candidates before
// its own first query altogether.
#include "pmp_dev.h"
#include "quant.h"

#include <algorithm>

namespace pmp {

namespace {

constexpr int kJT = kJoinTile;                // queries / candidates per tile
constexpr int kQueueCap = 512;                // group hits buffered before they are resolved
constexpr int kOutCap = 192;                  // kept pairs buffered before they are handed on
constexpr int kCovSample = 1024;              // windows per length for the directions
constexpr int kCovRows = 72;                  // of them per block of k_join_cov
constexpr int kCovParts = (kCovSample + kCovRows - 1) / kCovRows;
constexpr int kCovLd = 32 + 528;              // one block's sums and products (a <= b)

typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

__device__ __forceinline__ f16x8 as_f16x8(uint4 v) {
    union {
        uint4 u;
        f16x8 h;
    } c;
    c.u = v;
    return c.h;
}

// First position of the sorted keys[lo, hi) with key >= v (incl) or > v, by a
// 64-ary search of the whole wavefront (uniform arguments and result).
__device__ __forceinline__ uint32_t wave_first(const uint32_t *__restrict__ keys, uint32_t lo,
                                               uint32_t hi, uint32_t v, bool incl) {
    const uint32_t lane = (uint32_t)lane_id();
    while (hi > lo) {
        const uint32_t step = (hi - lo + kWave - 1) / kWave;
        const uint32_t idx = lo + lane * step;
        const uint32_t key = idx < hi ? keys[idx] : 0xFFFFFFFFu;
        const bool below = idx < hi && (incl ? key < v : key <= v);
        const uint32_t cnt = (uint32_t)__popcll(__ballot(below));
        if (cnt == 0) return lo;
        // keys[lo + (cnt - 1) step] is below, keys[lo + cnt step] is not
        const uint32_t end = lo + cnt * step;
        lo += (cnt - 1) * step + 1;
        hi = end < hi ? end : hi;
    }
    return lo;
}

__device__ __forceinline__ int wave_min_i(int v) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) v = min(v, __shfl_xor(v, off, kWave));
    return v;
}
__device__ __forceinline__ int wave_max_i(int v) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) v = max(v, __shfl_xor(v, off, kWave));
    return v;
}

}  // namespace

// ------------------------------------------------- principal directions

// Sums and second moments of the FP32 feature copies over an even sample of
// each length's windows, kCovRows windows a block: {sum[32], products[528]}, the
// products a <= b row by row.  A length's blocks write their sums one after
// the other from cov_base() on: a block's 4480 bytes lie in the 64 bytes that
// each of its 72 windows has in the sorted operands (filled later), and one
// block's more per length for the remainder.
//
// One block per length took 190 us whatever the request (1024 samples in turn,
// five FP64 sums a thread); fifteen blocks take 15 us, and k_pca adds them up.
__host__ __device__ inline int64_t cov_base(int64_t kbase, int l) {
    return kbase * (int64_t)(kJoinOp * sizeof(uint4) / sizeof(double)) + (int64_t)l * kCovLd;
}
static_assert(kCovRows * kJoinOp * sizeof(uint4) >= kCovLd * sizeof(double), "block sums fit");

template <typename FT>
__global__ __launch_bounds__(kBlock) void k_join_cov(Req q, double *__restrict__ out) {
    __shared__ float rows[kCovRows][2 * kMaxK + 1];
    const int l = blockIdx.y, part = blockIdx.x;
    const LenInfo &L = q.len[l];
    const int64_t n = L.n_index, kbase = L.kbase;
    const int S = (int)min<int64_t>(n, kCovSample);
    const int s0 = part * kCovRows, rn = min(kCovRows, S - s0);
    if (rn <= 0) return;
    double *o = out + cov_base(kbase, l) + (int64_t)part * kCovLd;
    for (int x = threadIdx.x; x < kCovRows * 32; x += kBlock) {
        const int r = x / 32, c = x % 32;
        float v = 0.0f;
        if (r < rn && c < 2 * (kMaxK - 1)) {
            const int64_t k = kbase + (int64_t)(((double)(s0 + r) + 0.5) * (double)n / (double)S);
            v = (float)((const FT *)q.F)[k * kRec + c];
        }
        rows[r][c] = v;
    }
    if (threadIdx.x < kCovRows) rows[threadIdx.x][32] = 1.0f;
    // thread -> pairs (a <= b < 32) of the upper triangle, or a sum entry
    double acc[3] = {0, 0, 0};
    int pa[3], pb[3];
#pragma unroll
    for (int x = 0; x < 3; ++x) {
        int p = threadIdx.x + x * kBlock;           // 528 pairs, then 32 sums
        pa[x] = 0;
        pb[x] = -1;
        if (p < 528) {
            int a = 0;
            while (p >= 32 - a) { p -= 32 - a; ++a; }
            pa[x] = a;
            pb[x] = a + p;
        } else if (p < 528 + 32) {
            pa[x] = p - 528;
            pb[x] = 32;                              // the sum entry
        }
    }
    __syncthreads();
    for (int r = 0; r < rn; ++r) {
#pragma unroll
        for (int x = 0; x < 3; ++x)
            acc[x] = fma((double)rows[r][pa[x]], (double)rows[r][max(pb[x], 0)], acc[x]);
    }
#pragma unroll
    for (int x = 0; x < 3; ++x) {
        const int p = threadIdx.x + x * kBlock;
        if (p < 528) o[32 + p] = acc[x];
        else if (p < 528 + 32) o[p - 528] = acc[x];
    }
}

namespace {
// Sum over the wavefront, in every lane (all 64 lanes active), by shifts within
// rows of 16 and row broadcasts.
template <int kCtrl, int kRows>
__device__ __forceinline__ void sum_step(double &v) {
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), kCtrl, kRows, 0xF, false);
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), kCtrl, kRows, 0xF, false);
    v += __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_sum_d(double v) {
    sum_step<0x111, 0xF>(v);
    sum_step<0x112, 0xF>(v);
    sum_step<0x114, 0xF>(v);
    sum_step<0x118, 0xF>(v);
    sum_step<0x142, 0xA>(v);
    sum_step<0x143, 0xC>(v);
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63),
                            __builtin_amdgcn_readlane(__double2loint(v), 63));
}
}  // namespace

// The kJoinDirs leading principal directions of each length's sample, made
// orthonormal in FP64; one block per length.  The covariance over its trace is
// squared twice by the whole block, then one wavefront (lane i holds component
// i of every direction) iterates all directions together, 16 products with the
// fourth power, set apart after every second and made orthonormal at the end.  Any orthonormal set
// keeps the threshold join exact; the leading directions make its cells
// selective.  udir[l][v][0..31] (components 30, 31 are 0).
//
// A serial chain: 64 products per direction in turn, with sums over the
// wavefront by general shuffles in each, took 180 us; this takes 55.
__global__ __launch_bounds__(kBlock) void k_pca(Req q, const double *__restrict__ cov, int L,
                                                double *__restrict__ udir) {
    constexpr int D = 2 * (kMaxK - 1);
    __shared__ double A[2][D][D + 1];
    __shared__ double sums[32];
    __shared__ double xs[kJoinDirs][32];
    __shared__ double trace;
    const int l = blockIdx.x;
    if (l >= L) return;
    const int tid = threadIdx.x;
    const double *c = cov + cov_base(q.len[l].kbase, l);
    const int n = (int)min<int64_t>(q.len[l].n_index, kCovSample);
    const int parts = (n + kCovRows - 1) / kCovRows;
    auto total = [&](int x) {
        double v[kCovParts], s = 0.0;
#pragma unroll
        for (int p = 0; p < kCovParts; ++p) v[p] = p < parts ? c[p * kCovLd + x] : 0.0;
#pragma unroll
        for (int p = 0; p < kCovParts; ++p) s += v[p];
        return s;
    };
    if (tid < 32) sums[tid] = total(tid);
    __syncthreads();
    const double S = (double)n;
    for (int x = tid; x < D * D; x += kBlock) {
        const int i = x / D, b = x % D, lo = min(i, b), hi = max(i, b);
        const double s = total(32 + lo * 32 - lo * (lo - 1) / 2 + hi - lo);
        A[0][i][b] = n >= 2 ? s / S - (sums[i] / S) * (sums[b] / S) : 0.0;
    }
    __syncthreads();
    if (tid < kWave) {
        const double t = wave_sum_d(tid < D ? A[0][tid][tid] : 0.0);
        if (tid == 0) trace = t;
    }
    __syncthreads();
    const double inv = trace > 1e-300 ? 1.0 / trace : 0.0;
    for (int x = tid; x < D * D; x += kBlock) A[0][x / D][x % D] *= inv;
    __syncthreads();
    for (int sq = 0; sq < 2; ++sq) {
        for (int x = tid; x < D * D; x += kBlock) {
            const int i = x / D, b = x % D;
            double s0 = 0.0, s1 = 0.0;
#pragma unroll
            for (int j = 0; j < D; j += 2) {               // (symmetric: row b is column b)
                s0 = fma(A[sq][i][j], A[sq][b][j], s0);
                s1 = fma(A[sq][i][j + 1], A[sq][b][j + 1], s1);
            }
            A[sq ^ 1][i][b] = s0 + s1;
        }
        __syncthreads();
    }
    if (tid >= kWave) return;
    // ---- one wavefront; A[0] holds the fourth power
    const int i = tid;
    double row[D];
#pragma unroll
    for (int j = 0; j < D; ++j) row[j] = i < D ? A[0][i][j] : 0.0;
    double u[kJoinDirs];
#pragma unroll
    for (int v = 0; v < kJoinDirs; ++v)
        u[v] = i < D ? 1.0 + 0.37 * ((i * (v + 3)) % 7) - 0.5 * (i % (v + 2)) : 0.0;
    // each direction against the ones before (twice, for rounding), then to
    // length 1; a degenerate one falls back to a unit vector
    auto orthonormal = [&]() {
#pragma unroll
        for (int v = 0; v < kJoinDirs; ++v) {
            double x = u[v];
            for (int e = 0;; ++e) {
                const double n0 = sqrt(wave_sum_d(x * x));
                if (n0 > 1e-300) {
                    x /= n0;
#pragma unroll
                    for (int w = 0; w < 2 * v; ++w) x -= wave_sum_d(x * u[w % v]) * u[w % v];
                    // (what is left of a dependent vector is rounding)
                    const double n1 = sqrt(wave_sum_d(x * x));
                    if (n1 > 1e-12) { x /= n1; break; }
                }
                x = i == e ? 1.0 : 0.0;
            }
#pragma unroll
            for (int w = 0; w < 2 * v; ++w) x -= wave_sum_d(x * u[w % v]) * u[w % v];
            x /= sqrt(wave_sum_d(x * x));
            u[v] = i < D ? x : 0.0;
        }
    };
    // between the products: once against the ones before, and to length 1
    // (what vanishes stays 0, for the last pass to replace)
    auto separate = [&]() {
#pragma unroll
        for (int v = 0; v < kJoinDirs; ++v) {
#pragma unroll
            for (int w = 0; w < v; ++w) u[v] -= wave_sum_d(u[v] * u[w]) * u[w];
            const double n2 = wave_sum_d(u[v] * u[v]);
            u[v] = n2 > 1e-280 ? u[v] * rsqrt(n2) : 0.0;
        }
    };
    separate();
    for (int it = 0; it < 16; ++it) {
        if (i < 32)
#pragma unroll
            for (int v = 0; v < kJoinDirs; ++v) xs[v][i] = u[v];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int v = 0; v < kJoinDirs; ++v) {
            double y0 = 0.0, y1 = 0.0;
#pragma unroll
            for (int j = 0; j < D; j += 2) {
                y0 = fma(row[j], xs[v][j], y0);
                y1 = fma(row[j + 1], xs[v][j + 1], y1);
            }
            u[v] = y0 + y1;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (it & 1) separate();
    }
    orthonormal();
    if (i < 32)
#pragma unroll
        for (int v = 0; v < kJoinDirs; ++v) udir[((int64_t)l * kJoinDirs + v) * 32 + i] = u[v];
}

// ------------------------------------------------------------ grid keys

// Sort key (length, cell1, cell2) and value k of every indexed window (from
// its principal coordinates, computed by k_keys), and its query flag (cell
// not yet at 0) for this round.  With cb2 = 0 the grid
// has one coordinate only, in finer cells (a band), for radii below the
// resolution of the two-coordinate grid.
__global__ __launch_bounds__(kBlock) void k_grid_keys(Req q, const GridLen *__restrict__ gl,
                                                      int64_t N, int cb1, int cb2, int cb3,
                                                      int l_lim, int64_t i_lim,
                                                      uint32_t *__restrict__ gkey,
                                                      uint32_t *__restrict__ gval,
                                                      uint8_t *__restrict__ qf,
                                                      float4 *__restrict__ gp,
                                                      uint32_t *__restrict__ nonq) {
    const int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k >= N) return;
    const int64_t k_first = (int64_t)blockIdx.x * kBlock + (threadIdx.x & ~(kWave - 1));
    const int l = find_len_k_wave(q.len, q.L, k_first, k);
    const GridLen &G = gl[l];
    const float4 c = gp[k];
    const double p1 = c.x, p2 = c.y, p3 = c.z;
    auto cell = [&](double p, int bits, double hinv) -> uint32_t {
        const uint32_t top = (1u << bits) - 1u;
        const double x = (p - G.qlo) * hinv;
        if (!(x > 0.0)) return 0u;
        if (x >= (double)top) return top;
        return (uint32_t)x;
    };
    gkey[k] = ((uint32_t)l << (cb1 + cb2 + cb3)) | (cell(p1, cb1, G.hinv) << (cb2 + cb3)) |
              (cb2 ? cell(p2, cb2, G.hinv2) << cb3 : 0u) | (cb3 ? cell(p3, cb3, G.hinv2) : 0u);
    gval[k] = (uint32_t)k;
    // a query: a cell not yet at 0 whose (length, start) lies at or before
    // the bound (the bound is the last length when it does not apply)
    const int64_t i = (int64_t)q.cell[k] - q.len[l].cell_base;
    const bool f = q.P[k] != 0ull && (l < l_lim || (l == l_lim && i <= i_lim));
    qf[k] = f;
    if (!f) nonq[l] = 1u;                         // (every writer stores the same value)
    // the same flag in the sign of the candidate's Gram term, so that a
    // candidate tile reads one 16-byte word per window besides its operands
    gp[k].w = f ? -fabsf(c.w) : fabsf(c.w);
}

// The join operands and coordinates in sorted (grid) order, so that a tile
// of the order reads contiguous blocks, with no index load before them: the
// operands as two arrays of half rows (32 bytes each, one per matrix product),
// the Gram terms again on their own.
__global__ __launch_bounds__(kBlock) void k_join_gather(const uint32_t *__restrict__ gval,
                                                        const uint4 *__restrict__ jop,
                                                        const float4 *__restrict__ gp, int64_t n,
                                                        uint4 *__restrict__ jop_s,
                                                        float4 *__restrict__ gp_s,
                                                        float *__restrict__ gw_s) {
    // four threads per window: one 16-byte part of its operands each
    const int64_t x = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t pos = x >> 2;
    const int part = (int)(x & 3);
    if (pos >= n) return;
    const uint32_t k = gval[pos];
    jop_s[(part >> 1) * 2 * n + pos * 2 + (part & 1)] = jop[(int64_t)k * kJoinOp + part];
    if (part == 0) {
        const float4 g = gp[k];
        gp_s[pos] = g;
        gw_s[pos] = g.w;
    }
}

// ------------------------------------------------------------ the tiles

// The exact stage of kept pairs, one pair (ki, kc) of indexed windows of one
// length per lane (whole wavefront; `valid` false on lanes without one).  A
// pair outside the exclusion zone gets the certified Parseval bound from the
// stored records, and if the bound leaves it able to lower one of its cells
// below T, the canonical FP64 distance, which lowers both cells.  The
// window's loads are issued together (one memory latency before the tests).
// Returns the distances this lane's pair needed (0 or 1).  kLean: the form
// with the fewest registers (no record bound, one term per lane per load):
// a pair the bound would have skipped then has its distance computed and
// discarded at the exit bound, which leaves every cell as the full form does.
template <typename FT, bool kLaneForm, bool kLean = false>
__device__ __forceinline__ uint32_t join_exact(const Req &q, bool valid, uint32_t ki, uint32_t kc,
                                               int m, int64_t cell_base, float sqrt2m, double T) {
    bool has = false;
    int64_t si = 0, sc = 0;
    double Pi = 0.0, Pc = 0.0, mui = 0.0, isi = 0.0, muc = 0.0, isc = 0.0, lim = INFINITY;
    if (valid) {
        si = (int64_t)q.cell[ki] - cell_base;
        sc = (int64_t)q.cell[kc] - cell_base;
        Pi = bitsd(q.P[ki]);
        Pc = bitsd(q.P[kc]);
        mui = q.mu[ki];
        isi = q.isig[ki];
        muc = q.mu[kc];
        isc = q.isig[kc];
        const int64_t gap = si > sc ? si - sc : sc - si;
        const double thr = fmin(T, fmax(Pi, Pc));
        if (gap >= q.excl && thr > 0.0) {
            const float lb = kLean ? 0.0f
                                   : lb_mem<FT>((const FT *)q.F + (int64_t)ki * kRec,
                                                (const FT *)q.F + (int64_t)kc * kRec, sqrt2m);
            if ((double)lb <= T && ((double)lb < Pi || (double)lb < Pc)) {
                has = true;
                lim = exit_bound(thr);
            }
        }
    }
    uint32_t n_ver = 0;
    const uint64_t mask = __ballot(has);
    if (mask) {
        uint64_t *P = q.P;
        verify_proposals<kLaneForm, kLean ? 1 : kZBatch>(mask, SeriesA{q.t}, q.t, si, mui, isi, sc,
                                                         muc, isc, m,
                                    [&](double dd) {
            ++n_ver;
            const unsigned long long db = (unsigned long long)dbits(dd);
            if (dd < Pi) atomicMin((unsigned long long *)&P[ki], db);
            if (dd < Pc) atomicMin((unsigned long long *)&P[kc], db);
        }, lim);
    }
    return n_ver;
}

// One wavefront per block of 128 sorted queries of one length (four tiles of
// 32, their fp16 operands in registers).  It lists the runs of candidates
// next to its queries' cells, 64 grid rows at a time: one lane per row finds
// the row's range of cells and, by binary search in the sorted keys, its run.
// Then it walks the runs 32 candidates at a time: two 16-byte operand words
// and one Gram term per lane (the next tile's loads in flight through the
// current one's products), two products per query tile.  The query's filter
// term rides in the two operand slots past the features and the accumulators
// start at minus the candidate's Gram term, so a pair is kept iff its
// accumulator's sign is clear: one shift per row packs a lane's 64 signs into
// two words.  The passing pairs (about five of a step's 4096 at noisy data) go to
// a queue in LDS, less those of a candidate that is a query earlier in the order
// (its own block has them).  A full queue is tested one pair per lane on the
// stored coordinates; the pairs left become window indices and go to the pair
// buffer, whose pairs k_join_verify takes after the launch.  A wavefront that finds the buffer
// full puts its block on the list of overflowed blocks and stops; those are
// taken again from their start with an emptied buffer (the pairs of the first
// attempt that reached the buffer are then verified twice, which changes no
// minimum), or, should one alone overflow it, by the kRedo form, which
// verifies its pairs in place.  Keeping the exact stage out of the main form
// keeps the walk in registers.  The main form covers the blocks [blk0, blk0 +
// gridDim.x) of the round, or those of a list.
//
// Wavefronts share nothing and meet no barrier.  The form before shared
// candidate tiles through LDS among four wavefronts of one query tile each and
// took six bf16 products a tile; it was bound by its barriers, by a row filter
// of about 100 VALU instructions a tile and by the mirror image of every pair.
// Measured (FP32 form, ECG-like, 51 lengths of 100..400): 250,000 samples 27 ->
// 5.8 ms for all tiles, 1,000,000 samples 280 -> 64 ms; with rows tested four at
// a time against the term, and the row found again by the pair's own product
// (gathers of both operands: four fifths of the cache accesses) 47 in FP64; with
// the signs 38.
constexpr int kJB = kJoinBlock;               // query tiles per wavefront
constexpr int kJQ = kJB * kJT;                // queries per wavefront
constexpr int kJWaves = 4;                    // wavefronts per SIMD the registers are held to

struct JoinSmem {
    uint2 queue[kQueueCap];                   // passing pairs (positions of query, candidate)
    uint2 outq[kOutCap];                      // kept pairs (k_q, k_c)
    uint32_t qkey[kJQ];                       // the queries' cells (kNone: not a query)
    uint32_t rbeg[kWave], rend[kWave];        // the non-empty runs of 64 grid rows
};

template <typename FT, bool kRedo>
__device__ __forceinline__ void join_block(const Req &q, const GridLen *__restrict__ gl,
                                           const uint32_t *__restrict__ gkey,
                                           const uint32_t *__restrict__ gval,
                                           const uint8_t *__restrict__ qf,
                                           const uint4 *__restrict__ jop_s,
                                           const float4 *__restrict__ jmeta,
                                           const float4 *__restrict__ gp_s,
                                           const float *__restrict__ gw_s, int64_t nwin,
                                           const uint32_t *__restrict__ nonq, int cb1, int cb2,
                                           int cb3, double T, int64_t gb, const JoinOut &out,
                                           JoinSmem &sm, uint32_t part = 0, uint32_t parts = 1) {
    uint2 *const queue = sm.queue, *const outq = sm.outq;
    uint32_t *const qkey = sm.qkey, *const rbeg = sm.rbeg, *const rend = sm.rend;
    const int lane = lane_id();
    int l;
    {
        int lo = 0, hi = q.L - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (gl[mid].blk_base <= gb) lo = mid; else hi = mid - 1;
        }
        l = lo;
    }
    const GridLen &G = gl[l];
    const int m = q.len[l].m;
    const int64_t cell_base = q.len[l].cell_base;
    // positions of the sorted order fit 32 bits (at most 2^31 - 1 cells)
    const uint32_t pbeg = (uint32_t)q.len[l].kbase;
    const uint32_t pend = pbeg + (uint32_t)q.len[l].n_index;
    const uint32_t p0 = pbeg + (uint32_t)((gb - G.blk_base) * kJQ);
    const int i = lane % kJT, hh = lane / kJT;
    const float scale = join_scale(m);
    // the largest e' of the length, over the sets
    static_assert((kJeSets & (kJeSets - 1)) == 0 && kJeSets <= kWave, "a set per lane");
    float je = q.jemax[(int64_t)(lane % kJeSets) * je_pitch(q.L) + l];
#pragma unroll
    for (int off = kJeSets / 2; off > 0; off >>= 1) je = fmaxf(je, __shfl_xor(je, off, kWave));

    const uint4 *const op0 = jop_s, *const op1 = jop_s + 2 * nwin;

    // ---- query operands (A), their filter terms in slots 30 and 31
    f16x8 a0[kJB], a1[kJB];
    const uint32_t kmask = (1u << (cb1 + cb2 + cb3)) - 1u;
    bool any = false;
#pragma unroll
    for (int t = 0; t < kJB; ++t) {
        const uint32_t pq = p0 + (uint32_t)(t * kJT + i);
        const bool validq = pq < pend;
        const uint32_t kq = validq ? gval[pq] : 0u;
        const bool isq = validq && qf[kq];
        any |= __ballot(isq) != 0ull;
        const uint4 z = make_uint4(0, 0, 0, 0);
        uint4 w0 = isq ? op0[(int64_t)pq * 2 + hh] : z, w1 = isq ? op1[(int64_t)pq * 2 + hh] : z;
        if (hh == 1) {
            float hi = -65504.0f, lo = 0.0f;
            if (isq) {
                const float4 mt = jmeta[kq];              // |G|^2, e', |G| bound, 0
                const double v = join_filter_term(G.Tr, G.eps_c, G.nmax2, mt.x, mt.y, mt.z, je, scale);
                // (past the range every pair passes: |v| / scale is below
                // 32768 wherever the test decides anything)
                const float x = (float)fmin(fmax(v / (double)scale, -60000.0), 60000.0);
                hi = half_float(half_bits(x));
                lo = x - hi;
                if (fabsf(hi) < 0x1.0p-14f) hi = 0.0f;
                if (fabsf(lo) < 0x1.0p-14f) lo = 0.0f;
            }
            w1.w = half_bits(hi) | (half_bits(lo) << 16);
        }
        a0[t] = as_f16x8(w0);
        a1[t] = as_f16x8(w1);
        if (hh == 0) qkey[t * kJT + i] = isq ? (gkey[pq] & kmask) : kNone;
    }
    if (!any) return;                                     // uniform
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();

    unsigned long long n_tiles = 0, n_kept = 0, n_ver = 0;
    int qn = 0, on = 0;                                   // queued groups, kept pairs (uniform)
    bool over = false;                                    // the buffer ran full (uniform)

    auto lds_sync = [] {
        // LDS is written and read by this wavefront only
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    // hand the kept pairs to the pair buffer (or, kRedo, verify them here)
    auto hand_on = [&]() {
        lds_sync();
        n_kept += (unsigned long long)on;
        if (kRedo) {
            for (int b = 0; b < on; b += kWave) {
                const int e = b + lane;
                const uint2 pr = e < on ? outq[e] : make_uint2(0u, 0u);
                n_ver += join_exact<FT, false, true>(q, e < on, pr.x, pr.y, m, cell_base,
                                                     G.sqrt2m, T);
            }
        } else {
            unsigned long long base = 0;
            const int seg = (int)(blockIdx.x % kCtrSlots);
            if (lane == 0) base = atomicAdd(&out.pcount[seg * kCtrStride], (unsigned long long)on);
            base = (unsigned long long)__builtin_amdgcn_readfirstlane((uint32_t)base) |
                   (unsigned long long)__builtin_amdgcn_readfirstlane((uint32_t)(base >> 32)) << 32;
            const unsigned long long cap = (unsigned long long)out.segcap;
            const int fit = base >= cap ? 0 : (int)min((unsigned long long)on, cap - base);
            for (int e = lane; e < fit; e += kWave) out.pairs[seg * out.segcap + (int64_t)base + e] = outq[e];
            over |= __builtin_amdgcn_readfirstlane(fit < on ? 1 : 0) != 0;
        }
        lds_sync();
        on = 0;
    };
    // test the queued pairs on their coordinates
    auto resolve = [&]() {
        lds_sync();
        for (int b = 0; b < qn; b += kWave) {
            const int e = b + lane;
            bool keep = false;
            uint2 pr = make_uint2(0u, 0u);
            if (e < qn) {
                pr = queue[e];
                const float4 gq = gp_s[pr.x], gc = gp_s[pr.y];
                // (all three at once: one wait)
                keep = fmaxf(fmaxf(fabsf(gq.x - gc.x), fabsf(gq.y - gc.y)), fabsf(gq.z - gc.z)) <=
                       G.rp;
            }
            const uint64_t mk = __ballot(keep);
            if (mk == 0ull) continue;
            if (keep) outq[on + __popcll(mk & lanemask_lt())] = make_uint2(gval[pr.x], gval[pr.y]);
            on += __popcll(mk);
            if (on > kOutCap - kWave) hand_on();
        }
        lds_sync();
        qn = 0;
    };

    // ---- the grid rows next to the queries' cells
    const uint32_t mask1 = (1u << cb1) - 1u, mask2 = (1u << cb2) - 1u, mask3 = (1u << cb3) - 1u;
    const uint32_t lbits = (uint32_t)l << (cb1 + cb2 + cb3);
    // rows are c1 cells with one or two coordinates (one coordinate: a single
    // row, the whole range), (c1, c2) pairs with three
    int r1lo, r1hi, r2lo = 0, r2n = 1;
    {
        int lo1 = INT_MAX, hi1 = -1, lo2 = INT_MAX, hi2 = -1;
        for (int x = lane; x < kJQ; x += kWave) {
            const uint32_t key = qkey[x];
            if (key == kNone) continue;
            const int c1 = (int)(key >> (cb2 + cb3)), c2 = (int)((key >> cb3) & mask2);
            lo1 = min(lo1, c1);
            hi1 = max(hi1, c1);
            lo2 = min(lo2, c2);
            hi2 = max(hi2, c2);
        }
        lo1 = wave_min_i(lo1);
        hi1 = wave_max_i(hi1);
        lo2 = wave_min_i(lo2);
        hi2 = wave_max_i(hi2);
        r1lo = max(lo1 - kJoinNb, 0);
        r1hi = min(hi1, (int)mask1 - kJoinNb) + kJoinNb;
        if (cb3 > 0) {
            r2lo = max(lo2 - kJoinNb, 0);
            r2n = min(hi2 + kJoinNb, (int)mask2) - r2lo + 1;
        }
    }
    // every window of the length a query: the candidates before this block's
    // first query see this block's queries themselves
    const uint32_t first = nonq[l] ? pbeg : p0;
    const int nrows = cb2 == 0 ? 1 : (r1hi - r1lo + 1) * r2n;

    for (int row0 = 0; row0 < nrows && !over; row0 += kWave) {
        // ---- one lane per row: its range of keys, then its run
        const int row = row0 + lane;
        uint32_t beg = 0, end = 0;
        uint32_t klo = 1u, khi = 0u;
        if (row < nrows) {
            if (cb2 == 0) {
                klo = lbits | (uint32_t)r1lo;
                khi = lbits | (uint32_t)r1hi;
            } else {
                const int c1 = r1lo + row / r2n, c2 = r2lo + row % r2n;
                int lo = INT_MAX, hi = -1;
#pragma unroll 8
                for (int x = 0; x < kJQ; ++x) {
                    const uint32_t key = qkey[x];
                    const int q1 = (int)(key >> (cb2 + cb3)), q2 = (int)((key >> cb3) & mask2);
                    const int qx = cb3 > 0 ? (int)(key & mask3) : q2;
                    const bool near = key != kNone && abs(q1 - c1) <= kJoinNb &&
                                      (cb3 == 0 || abs(q2 - c2) <= kJoinNb);
                    lo = near ? min(lo, qx) : lo;
                    hi = near ? max(hi, qx) : hi;
                }
                if (hi >= 0) {
                    const uint32_t rk = cb3 > 0
                        ? lbits | ((uint32_t)c1 << (cb2 + cb3)) | ((uint32_t)c2 << cb3)
                        : lbits | ((uint32_t)c1 << cb2);
                    klo = rk | (uint32_t)max(lo - kJoinNb, 0);
                    khi = rk | (uint32_t)min(hi + kJoinNb, (int)(cb3 > 0 ? mask3 : mask2));
                }
            }
        }
        if (nrows == 1) {
            // one row: the whole wavefront searches for it
            klo = __builtin_amdgcn_readfirstlane(klo);
            khi = __builtin_amdgcn_readfirstlane(khi);
            const uint32_t b0 = wave_first(gkey, first, pend, klo, true);
            const uint32_t e0 = wave_first(gkey, b0, pend, khi, false);
            if (lane == 0) {
                beg = b0;
                end = e0;
            }
        } else if (klo <= khi) {
            // first positions with key >= klo and key > khi, together
            uint32_t lo1 = first, hi1 = pend, lo2 = first, hi2 = pend;
            while (lo1 < hi1 || lo2 < hi2) {
                const uint32_t m1 = lo1 + ((hi1 - lo1) >> 1), m2 = lo2 + ((hi2 - lo2) >> 1);
                const uint32_t v1 = gkey[min(m1, pend - 1u)], v2 = gkey[min(m2, pend - 1u)];
                if (lo1 < hi1) {
                    if (v1 < klo) lo1 = m1 + 1u; else hi1 = m1;
                }
                if (lo2 < hi2) {
                    if (v2 <= khi) lo2 = m2 + 1u; else hi2 = m2;
                }
            }
            beg = lo1;
            end = lo2;
        }
        const uint64_t live = __ballot(beg < end);
        const int nrun = __popcll(live);
        if (beg < end) {
            const int at = __popcll(live & lanemask_lt());
            rbeg[at] = beg;
            rend[at] = end;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (nrun == 0) continue;

        // ---- the runs, 32 candidates at a time
        auto load_tile = [&](uint32_t c, uint4 &b0, uint4 &b1, float &w) {
            const uint32_t pc = min(c + (uint32_t)i, pend - 1u);
            b0 = op0[(int64_t)pc * 2 + hh];
            b1 = op1[(int64_t)pc * 2 + hh];
            w = gw_s[pc];
        };
        int run = 0;
        uint32_t c = __builtin_amdgcn_readfirstlane(rbeg[0]);
        uint32_t e = __builtin_amdgcn_readfirstlane(rend[0]);
        uint4 nb0, nb1;
        float nw;
        bool more = true;
        // one tile on (all uniform)
        auto next = [&]() {
            c += kJT;
            if (c >= e) {
                if (++run < nrun) {
                    c = __builtin_amdgcn_readfirstlane(rbeg[run]);
                    e = __builtin_amdgcn_readfirstlane(rend[run]);
                } else {
                    more = false;
                }
            }
        };
        if (kRedo) {
            // this part's tiles: every parts-th from the part-th on
            for (uint32_t x = 0; x < part && more; ++x) next();
        }
        load_tile(c, nb0, nb1, nw);
        while (more) {
            const f16x8 b0 = as_f16x8(nb0), b1 = as_f16x8(nb1);
            // the candidate's Gram term (its sign is the query flag), negative;
            // +0 for a term of 0, and -inf past the run's end
            const float term = c + (uint32_t)i < e ? 0.0f - fabsf(nw) : -INFINITY;
            const bool cq = signbit(nw);
            const uint32_t tc = c;
            next();
            if (kRedo) {
                for (uint32_t x = 1; x < parts && more; ++x) next();
            }
            load_tile(c, nb0, nb1, nw);                   // (past the last: read and dropped)
            n_tiles += kJB;
            f32x16 z;
#pragma unroll
            for (int r = 0; r < 16; ++r) z[r] = term;
            // two query tiles at a time; bit 16 t + r of a word: row r of tile
            // t fails (the accumulator's sign)
            uint32_t pass[kJB / 2];
#pragma unroll
            for (int u = 0; u < kJB / 2; ++u) {
                f32x16 acc[2];
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a0[2 * u + t], b0, z, 0, 0, 0);
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1[2 * u + t], b1, acc[t], 0, 0, 0);
                uint32_t fail = 0;
#pragma unroll
                for (int t = 1; t >= 0; --t)
#pragma unroll
                    for (int r = 15; r >= 0; --r)
                        fail = __builtin_amdgcn_alignbit(fail, (uint32_t)__float_as_int(acc[t][r]), 31);
                pass[u] = ~fail;
            }
#pragma unroll
            for (int u = 0; u < kJB / 2; ++u) {
                uint32_t hit = pass[u];
                uint64_t mk = __ballot(hit != 0u);
                while (mk) {
                    if (qn > kQueueCap - kWave) resolve();
                    bool put = false;
                    uint32_t pq = 0;
                    const uint32_t pc = tc + (uint32_t)i;
                    if (hit) {
                        // row r of tile t: 32 t + 8 (r / 4) + 4 hh + r % 4
                        const uint32_t x = (uint32_t)__builtin_ctz(hit);
                        pq = p0 + 64u * u + 32u * (x >> 4) + 8u * ((x >> 2) & 3u) + 4u * (uint32_t)hh +
                             (x & 3u);
                        hit &= hit - 1u;
                        put = pq != pc && !(cq && pc < pq);
                    }
                    const uint64_t pm = __ballot(put);
                    if (put) queue[qn + __popcll(pm & lanemask_lt())] = make_uint2(pq, pc);
                    qn += __popcll(pm);
                    mk = __ballot(hit != 0u);
                }
            }
            if (over) break;
        }
        // (the next rows' runs overwrite rbeg and rend)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    if (qn > 0 && !over) resolve();
    if (on > 0 && !over) hand_on();
    if (over) {
        // (its counts come from the second attempt)
        if (lane == 0) out.redo[atomicAdd(out.nredo, 1u)] = (uint32_t)gb;
        return;
    }
    // statistics: one atomic per wavefront
    for (int off = kWave / 2; off > 0; off >>= 1) n_ver += __shfl_xor(n_ver, off, kWave);
    if (lane == 0) {
        count_add(q.counters, C_JOIN_PAIRS, n_tiles * (unsigned long long)(kJT * kJT));
        if (n_kept) count_add(q.counters, C_JOIN_CAND, n_kept);
        if (n_ver) count_add(q.counters, C_JOIN_VER, n_ver);
    }
}

template <typename FT>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(kJWaves)))
void k_join_tiles(Req q, const GridLen *__restrict__ gl, const uint32_t *__restrict__ gkey,
                  const uint32_t *__restrict__ gval, const uint8_t *__restrict__ qf,
                  const uint4 *__restrict__ jop_s, const float4 *__restrict__ jmeta,
                  const float4 *__restrict__ gp_s, const float *__restrict__ gw_s, int64_t nwin,
                  const uint32_t *__restrict__ nonq, int cb1, int cb2, int cb3, double T,
                  int64_t blk0, int64_t nblocks, const uint32_t *__restrict__ list, int run,
                  JoinOut out) {
    __shared__ JoinSmem sm;
    const int64_t b = join_block_of((int64_t)blockIdx.x, run);
    if (b >= nblocks) return;
    const int64_t gb = list ? (int64_t)list[b] : blk0 + b;
    join_block<FT, false>(q, gl, gkey, gval, qf, jop_s, jmeta, gp_s, gw_s, nwin, nonq, cb1, cb2,
                          cb3, T, gb, out, sm);
}

// Blocks that overflow a segment of the buffer to themselves: their pairs are
// verified in place.  Each block's tiles go to `parts` wavefronts in turn: one
// wavefront took 3.2 ms for the few hundred thousand pairs of such a block (random
// walk, 4,443 samples at 259..396), 1.0 with up to 32.
template <typename FT>
__global__ __launch_bounds__(kWave)
void k_join_redo(Req q, const GridLen *__restrict__ gl, const uint32_t *__restrict__ gkey,
                 const uint32_t *__restrict__ gval, const uint8_t *__restrict__ qf,
                 const uint4 *__restrict__ jop_s, const float4 *__restrict__ jmeta,
                 const float4 *__restrict__ gp_s, const float *__restrict__ gw_s, int64_t nwin,
                 const uint32_t *__restrict__ nonq, int cb1, int cb2, int cb3, double T,
                 const uint32_t *__restrict__ list, uint32_t n, uint32_t parts, JoinOut out) {
    __shared__ JoinSmem sm;
    for (uint32_t x = blockIdx.x; x < n * parts; x += gridDim.x)
        join_block<FT, true>(q, gl, gkey, gval, qf, jop_s, jmeta, gp_s, gw_s, nwin, nonq, cb1, cb2,
                             cb3, T, (int64_t)list[x / parts], out, sm, x % parts, parts);
}

// The exact stage of the pairs in the buffer, one pair per lane, each block
// striding over one segment.  Pairs of one length sit together in the buffer (a
// queue holds one length), so a wavefront's pairs mostly share their window
// length.
template <typename FT>
__global__ __launch_bounds__(kBlock) void k_join_verify(Req q, const GridLen *__restrict__ gl,
                                                        JoinOut out, double T) {
    const int seg = (int)(blockIdx.x % kCtrSlots);
    const int64_t n = min((int64_t)out.pcount[seg * kCtrStride], out.segcap);
    const uint2 *const pairs = out.pairs + seg * out.segcap;
    const int lane = lane_id();
    const int64_t stride = (int64_t)(gridDim.x / kCtrSlots) * kBlock;
    uint32_t n_ver = 0;
    for (int64_t base = (int64_t)(blockIdx.x / kCtrSlots) * kBlock + (threadIdx.x & ~(kWave - 1));
         base < n; base += stride) {
        const int64_t e = base + lane;
        const bool valid = e < n;
        const uint2 pr = valid ? pairs[e] : make_uint2(0u, 0u);
        const int l = valid ? find_len_k(q.len, q.L, (int64_t)pr.x) : 0;
        const LenInfo &L = q.len[l];
        n_ver += join_exact<FT, true>(q, valid, pr.x, pr.y, L.m, L.cell_base, gl[l].sqrt2m, T);
    }
    unsigned long long v = n_ver;
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    if (lane == 0 && v) count_add(q.counters, C_JOIN_VER, v);
}

// ------------------------------------------- the exact stage's prefilter (quant.h)

// Ordered bits of a finite double: unsigned order is numeric order.
__device__ __forceinline__ unsigned long long order_bits(double x) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(x);
    return (u >> 63) ? ~u : u | 0x8000000000000000ull;
}
__device__ __forceinline__ double order_value(unsigned long long u) {
    return __longlong_as_double((long long)((u >> 63) ? u & 0x7FFFFFFFFFFFFFFFull : ~u));
}

// mm[0] = smallest, mm[1] = largest sample (ordered bits; mm starts as all
// ones and 0).
__global__ __launch_bounds__(kBlock) void k_quant_range(const double *__restrict__ t, int64_t n,
                                                        unsigned long long *__restrict__ mm) {
    __shared__ unsigned long long lo[kBlock / kWave], hi[kBlock / kWave];
    unsigned long long a = ~0ull, b = 0ull;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock) {
        const unsigned long long u = order_bits(t[i]);
        a = u < a ? u : a;
        b = u > b ? u : b;
    }
    for (int off = kWave / 2; off > 0; off >>= 1) {
        const unsigned long long x = __shfl_xor(a, off, kWave), y = __shfl_xor(b, off, kWave);
        a = x < a ? x : a;
        b = y > b ? y : b;
    }
    if (lane_id() == 0) {
        lo[threadIdx.x / kWave] = a;
        hi[threadIdx.x / kWave] = b;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / kWave; ++w) {
            a = lo[w] < a ? lo[w] : a;
            b = hi[w] > b ? hi[w] : b;
        }
        atomicMin(&mm[0], a);
        atomicMax(&mm[1], b);
    }
}

// The series' centre c and half range from k_quant_range's result.
__device__ __forceinline__ double2 quant_scale(const unsigned long long *__restrict__ mm) {
    const double lo = order_value(mm[0]), hi = order_value(mm[1]);
    const double c = 0.5 * lo + 0.5 * hi;
    return make_double2(c, fmax(hi - c, c - lo) * (1.0 + 1e-12));
}

// The 16-bit series, twice: x[r] and, for windows at odd starts, x[r + 1], so
// that every window begins on a 4-byte boundary (16-byte loads need that).
// Entries past the series are 0.
__global__ __launch_bounds__(kBlock) void k_quantize(const double *__restrict__ t, int64_t n,
                                                     const unsigned long long *__restrict__ mm,
                                                     int16_t *__restrict__ x16, int64_t pitch) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= pitch) return;
    const double2 cs = quant_scale(mm);
    const int16_t v = i < n ? (int16_t)rint((t[i] - cs.x) / cs.y * 32767.0) : (int16_t)0;
    x16[i] = v;
    if (i > 0) x16[pitch + i - 1] = v;
    if (i == pitch - 1) x16[pitch + i] = 0;
}

// Per indexed window: its start, s / sigma, (c - mu) / sigma and delta.
__global__ __launch_bounds__(kBlock) void k_quant_windows(Req q, int64_t k0, int64_t k1,
                                                          const unsigned long long *__restrict__ mm,
                                                          float4 *__restrict__ xw) {
    const int64_t k = k0 + (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k >= k1) return;
    const int64_t k_first = k0 + (int64_t)blockIdx.x * kBlock + (threadIdx.x & ~(kWave - 1));
    const int l = find_len_k_wave(q.len, q.L, k_first, k);
    const double2 cs = quant_scale(mm);
    const double is = q.isig[k];
    const uint32_t start = (uint32_t)((int64_t)q.cell[k] - q.len[l].cell_base);
    const double delta = (0x1.0p-16 * (1.0 + 1e-4) + 0x1.0p-21) * cs.y * is;
    xw[k] = make_float4(__uint_as_float(start), (float)(cs.y * is / 32767.0),
                        (float)((cs.x - q.mu[k]) * is), (float)(delta * (1.0 + 1e-6)));
}

// The exact stage with the prefilter in front: one pair per lane for the
// pairs' data, four lanes per pair for the 16-bit sums (64 bytes of each
// window per load), then join_exact for the survivors.
template <typename FT>
__global__ __launch_bounds__(kBlock) void k_join_verify_q(Req q, const GridLen *__restrict__ gl,
                                                          JoinOut out, double T,
                                                          const int16_t *__restrict__ x16,
                                                          int64_t pitch,
                                                          const float4 *__restrict__ xw) {
    const int seg = (int)(blockIdx.x % kCtrSlots);
    const int64_t n = min((int64_t)out.pcount[seg * kCtrStride], out.segcap);
    const uint2 *const pairs = out.pairs + seg * out.segcap;
    const int lane = lane_id();
    const int g = lane & 3;
    const int64_t stride = (int64_t)(gridDim.x / kCtrSlots) * kBlock;
    uint32_t n_ver = 0;
    for (int64_t base = (int64_t)(blockIdx.x / kCtrSlots) * kBlock + (threadIdx.x & ~(kWave - 1));
         base < n; base += stride) {
        const int64_t e = base + lane;
        const bool valid = e < n;
        const uint2 pr = valid ? pairs[e] : make_uint2(0u, 0u);
        int l = 0, m = 0;
        uint32_t si = 0, sj = 0;
        float ai = 0.0f, aj = 0.0f, b = 0.0f, lim = 0.0f;
        bool live = false, pass = false;      // needs the sums; goes on to the exact stage
        if (valid) {
            l = find_len_k(q.len, q.L, (int64_t)pr.x);
            m = q.len[l].m;
            const float4 wi = xw[pr.x], wj = xw[pr.y];
            si = __float_as_uint(wi.x);
            sj = __float_as_uint(wj.x);
            ai = wi.y;
            aj = wj.y;
            b = wi.z - wj.z;
            const uint32_t gap = si > sj ? si - sj : sj - si;
            if (gap >= (uint32_t)q.excl) {
                live = quant_limit(wi, wj, m, T, lim);
                pass = !live;
            }
        }
#pragma unroll 1
        for (int rnd = 0; rnd < 4; ++rnd) {
            // lanes 4 p .. 4 p + 3 take the pair of lane 16 rnd + p
            const int src = 16 * rnd + (lane >> 2);
            const bool go = __shfl(live ? 1 : 0, src, kWave) != 0;
            if (__ballot(go) == 0) continue;
            const uint32_t gi = (uint32_t)__shfl((int)si, src, kWave);
            const uint32_t gj = (uint32_t)__shfl((int)sj, src, kWave);
            const float gai = __shfl(ai, src, kWave), gaj = __shfl(aj, src, kWave);
            const float gb = __shfl(b, src, kWave), glim = __shfl(lim, src, kWave);
            const int gm = __shfl(m, src, kWave);
            const bool in = go && quant_below<4>(x16, pitch, gi, gj, gai, gaj, gb, gm, glim, g);
            const uint64_t mk = __ballot(in);
            if ((lane >> 4) == rnd && live) pass = (mk >> (4 * (lane & 15))) & 1ull;
        }
        if (__ballot(pass) == 0) continue;
        n_ver += join_exact<FT, true>(q, pass, pr.x, pr.y, m, q.len[l].cell_base, gl[l].sqrt2m, T);
    }
    unsigned long long v = n_ver;
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    if (lane == 0 && v) count_add(q.counters, C_JOIN_VER, v);
}

// ------------------------------------------------------------ launchers

static inline unsigned nblk(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

size_t join_sorted_bytes(int64_t N, int L) { return (size_t)cov_base(N, L) * sizeof(double); }

void launch_join_dirs(int precision, const Req &q, int nlen, double *cov, double *udir,
                      hipStream_t s) {
    if (nlen <= 0) return;
    if (precision == 0)
        hipLaunchKernelGGL(k_join_cov<double>, dim3(kCovParts, (unsigned)nlen), dim3(kBlock), 0, s, q, cov);
    else
        hipLaunchKernelGGL(k_join_cov<float>, dim3(kCovParts, (unsigned)nlen), dim3(kBlock), 0, s, q, cov);
    hipLaunchKernelGGL(k_pca, dim3((unsigned)nlen), dim3(kBlock), 0, s, q, cov, nlen, udir);
}

void launch_grid_keys(const Req &q, const GridLen *gl, int64_t N, int cb1, int cb2, int cb3,
                      int l_lim, int64_t i_lim, uint32_t *gkey, uint32_t *gval, uint8_t *qf,
                      float4 *gp, uint32_t *nonq, hipStream_t s) {
    if (N <= 0) return;
    hipLaunchKernelGGL(k_grid_keys, dim3(nblk(N)), dim3(kBlock), 0, s, q, gl, N, cb1, cb2, cb3,
                       l_lim, i_lim, gkey, gval, qf, gp, nonq);
}

void launch_join_gather(const uint32_t *gval, const uint4 *jop, const float4 *gp, int64_t n,
                        uint4 *jop_s, float4 *gp_s, float *gw_s, hipStream_t s) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_join_gather, dim3((unsigned)((n * kJoinOp + kBlock - 1) / kBlock)),
                       dim3(kBlock), 0, s, gval, jop, gp, n, jop_s, gp_s, gw_s);
}

void launch_join_tiles(const JoinIn &in, int64_t blk0, int64_t nblocks, const uint32_t *list,
                       const JoinOut &out, hipStream_t s) {
    if (nblocks <= 0) return;
    const int run = join_run(nblocks);
    const dim3 grid((unsigned)join_workgroups(nblocks));
    if (in.precision == 0)
        hipLaunchKernelGGL(k_join_tiles<double>, grid, dim3(kWave), 0, s, in.q, in.gl, in.gkey,
                           in.gval, in.qf, in.jop_s, in.jmeta, in.gp_s, in.gw_s, in.nwin, in.nonq,
                           in.cb1, in.cb2, in.cb3, in.T, blk0, nblocks, list, run, out);
    else
        hipLaunchKernelGGL(k_join_tiles<float>, grid, dim3(kWave), 0, s, in.q, in.gl, in.gkey,
                           in.gval, in.qf, in.jop_s, in.jmeta, in.gp_s, in.gw_s, in.nwin, in.nonq,
                           in.cb1, in.cb2, in.cb3, in.T, blk0, nblocks, list, run, out);
}

void launch_join_redo(const JoinIn &in, const uint32_t *list, uint32_t n, hipStream_t s) {
    if (n == 0) return;
    // (two wavefronts a SIMD fit)
    const uint32_t parts = std::min(std::max(2048u / n, 1u), 32u);
    const dim3 grid(std::min(n * parts, 2048u));
    if (in.precision == 0)
        hipLaunchKernelGGL(k_join_redo<double>, grid, dim3(kWave), 0, s, in.q, in.gl, in.gkey,
                           in.gval, in.qf, in.jop_s, in.jmeta, in.gp_s, in.gw_s, in.nwin, in.nonq,
                           in.cb1, in.cb2, in.cb3, in.T, list, n, parts, JoinOut{});
    else
        hipLaunchKernelGGL(k_join_redo<float>, grid, dim3(kWave), 0, s, in.q, in.gl, in.gkey,
                           in.gval, in.qf, in.jop_s, in.jmeta, in.gp_s, in.gw_s, in.nwin, in.nonq,
                           in.cb1, in.cb2, in.cb3, in.T, list, n, parts, JoinOut{});
}

void launch_join_verify(int precision, const Req &q, const GridLen *gl, const JoinOut &out,
                        double T, const Quant &x, hipStream_t s) {
    // enough wavefronts to keep every SIMD busy with eight, each striding; a
    // whole number of blocks per segment
    const int64_t want = (out.segcap + kBlock - 1) / kBlock;
    const unsigned nb = kCtrSlots * (unsigned)(want < 32 ? want : 32);
    if (x.x16 && precision == 0)
        hipLaunchKernelGGL(k_join_verify_q<double>, dim3(nb), dim3(kBlock), 0, s, q, gl, out, T,
                           x.x16, x.pitch, x.xw);
    else if (x.x16)
        hipLaunchKernelGGL(k_join_verify_q<float>, dim3(nb), dim3(kBlock), 0, s, q, gl, out, T,
                           x.x16, x.pitch, x.xw);
    else if (precision == 0)
        hipLaunchKernelGGL(k_join_verify<double>, dim3(nb), dim3(kBlock), 0, s, q, gl, out, T);
    else
        hipLaunchKernelGGL(k_join_verify<float>, dim3(nb), dim3(kBlock), 0, s, q, gl, out, T);
}

// room past a window's last sample for whole loads of the prefilter
int64_t quant_pitch(int64_t n) { return (n + 64 + 7) & ~(int64_t)7; }

void launch_quant_series(const double *t, int64_t n, const Quant &x, hipStream_t s) {
    launch_fill_u64((uint64_t *)x.mm, 1, ~0ull, s);
    launch_fill_u64((uint64_t *)x.mm + 1, 1, 0ull, s);
    const unsigned nb = nblk(n);
    hipLaunchKernelGGL(k_quant_range, dim3(nb < 256 ? nb : 256), dim3(kBlock), 0, s, t, n, x.mm);
    hipLaunchKernelGGL(k_quantize, dim3(nblk(x.pitch)), dim3(kBlock), 0, s, t, n,
                       (const unsigned long long *)x.mm, x.x16, x.pitch);
}

void launch_quant_windows(const Req &q, int64_t k0, int64_t k1, const Quant &x, hipStream_t s) {
    if (k1 <= k0) return;
    hipLaunchKernelGGL(k_quant_windows, dim3(nblk(k1 - k0)), dim3(kBlock), 0, s, q, k0, k1,
                       (const unsigned long long *)x.mm, x.xw);
}

}  // namespace pmp
