// pmp_dev.h -- internal declarations shared by the HIP translation units of
// libpmp (not a public header).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

namespace pmp {

// ------------------------------------------------------------ constants
constexpr int    kBlock      = 256;       // threads per block (4 waves of 64)
constexpr int    kWave       = 64;
constexpr int    kMaxK       = 16;        // largest spectral width K
constexpr int    kRec        = 32;        // feature record: 30 features + e_i + |F|
constexpr int    kSlotErr    = 30;        // record slot of the error bound e_i
constexpr int    kSlotNorm   = 31;        // record slot of ||F||
constexpr int    kMaxBits    = 24;        // SimHash bits B (Sec. 4: B = 24)
constexpr int    kProbeSlots = 8;         // Hamming-1 probes kept per key word
constexpr int    kProbeQ     = 8;         // queries per probe wavefront (eight lanes each)
constexpr int    kMaxM       = 2048;      // longest window supported
constexpr int    kTileW      = 1024;      // windows per sketch tile
constexpr int    kSegW       = 64;        // windows per sliding-DFT segment
constexpr int    kSegs       = kTileW / kSegW;   // 16 segments, one per 16 lanes
constexpr double kEps0       = 1e-6;      // zero snap (Sec. 3.6)
constexpr uint64_t kInfBits  = 0x7FF0000000000000ull;   // +inf as FP64 bits

// Per-length metadata, device resident.  Every per-window array is indexed
// by the compacted position k of the non-constant ("indexed") windows in
// (length, start) order; the windows of length l are k in [kbase, kbase + n_index).
struct LenInfo {
    int32_t m;            // window length
    int32_t kprime;       // K' = min(K-1, ceil(m/2)-1)
    int32_t depth;        // directory depth d (Prop. 4 final state)
    int32_t probes;       // Hamming-1 probes h = min(cap, d, 1 + max(0, d - d0))
    int64_t W;            // windows n - m + 1
    int64_t cell_base;    // first cell of this length in (length, start) order
    int64_t kbase;        // first indexed position of this length
    int64_t bucket_base;  // first bucket of this length
    int64_t n_index;      // non-constant windows (entries of the directory)
    int64_t tile_base;    // first sketch tile of this length
    int64_t blk_base;     // first block of this length in k_keys (anchors own blocks)
    // anchor lengths (Sec. 3.3): the one pass probes only these.  pblk_base
    // is non-decreasing over the lengths: an anchor owns probe blocks
    // [pblk_base, pblk_base + ceil(n_index / kProbeQ)), a non-anchor none.
    // Likewise hblk_base for the hint blocks of the non-anchor lengths.
    int32_t anchor;       // 1: an anchor length
    int32_t a_lo, a_hi;   // a non-anchor's nearest anchors below and above
                          // (indices; -1: none)
    int32_t aidx;         // an anchor's number among the anchors (its projections)
    int64_t pblk_base;    // first probe block of this length
    int64_t hblk_base;    // first hint block of this length
    // Keys and buckets exist at the anchor lengths only (nothing else reads
    // them): a non-anchor has depth 0 and no k_keys blocks, and an anchor's
    // sort entries sit at [abase, abase + n_index) of the anchor windows
    int64_t abase;        // first slot of this length among the anchor windows
};

// Everything a kernel needs to know about one request.
struct Req {
    const double *t;       // series
    int64_t n;
    int32_t L;             // number of lengths
    int32_t K;             // spectral width
    int32_t B;             // signature bits
    int32_t excl;          // exclusion zone
    int32_t budget_R;      // inspections per query (R = gamma * alpha)
    int32_t key_shift;     // bucket key: len_idx << key_shift | prefix << (key_shift - d)
    int32_t jkey_shift;    // join key: len_idx << jkey_shift | quantized p1
    int32_t precision;
    const LenInfo *len;    // [L]
    // per indexed window k, in (length, start) order
    uint32_t *cell;        // [N] cell id (cell_base of its length + start)
    double  *mu;           // [N] window mean
    double  *isig;         // [N] 1 / sigma (population standard deviation)
    uint64_t *P;           // [N] profile, FP64 bits (atomicMin)
    void    *F;            // [N][kRec] features (float or double)
    uint64_t *keyw;        // [N] key word: signature | probe order << 24
    uint4   *jop;          // [N][kJoinOp] join operands: 30 fp16 features G, then twice
                           //     join_scale(m)
    float4  *jmeta;        // [N] |G|^2, e' >= |G - F|, bound on |G|, 0
    float4  *gp;           // [N] principal coordinates of the FP32 feature copy, and
                           //     0.5 |G|^2 (rounded down) with the sign bit = (P != 0)
    const double *udir;    // [L][kJoinDirs][32] principal directions (null: none)
    // bucket order (slots)
    uint32_t *skey;        // [N] sort keys
    uint32_t *sval;        // [N] sort values (k)
    uint32_t *perm;        // [N] slot -> k
    uint32_t *pcell;       // [N] slot -> cell
    const float *gproj;    // [L][B][30] SimHash projections
    uint32_t *kmap;        // [cells] cell -> indexed position k (kNone: constant);
                           // written by the sketch when not null
    uint32_t *hint;        // [N] start of a partner that lowered the cell
                           // (kNone: none), written when a cell is lowered
    float   *emax;         // [L] largest e_i of each length
    float   *jemax;        // [kJeSets][je_pitch] largest e' of each length's join operands
    unsigned long long *counters;   // stats counters: kCtrSlots sets, kCtrStride apart
    int     *bad;          // raised on inputs the library cannot represent
};

enum Counter {
    C_PASS_CAND = 0, C_PASS_VER, C_JOIN_CAND, C_JOIN_VER, C_HOT, C_JOIN_PAIRS,
    C_SIEVE_VER, C_HINT_VER, C_COMPL_VER, C_COMPL_IMPROVED, C_NCOUNTERS
};

constexpr uint32_t kNone = 0xFFFFFFFFu;      // no entry (kmap, hint)

// Counters that every wavefront adds to are kept in kCtrSlots sets, one per
// residue of the block index and each in a cache line of its own, and summed
// by whoever reads them: atomics on one address follow each other at about
// 8 ns, which a million wavefronts would wait for (measured: the probe of 1e6
// windows at 8 per wavefront took 2.7 ms with one set of counters).  Blocks go
// to the eight XCDs in turn, so a set belongs to one of them.
constexpr int kCtrSlots = 64;
constexpr int kCtrStride = 16;               // in 64-bit words: 128 bytes
// Likewise the largest feature error of a length's join operands, which every
// wavefront of k_join_ops may raise: kJeSets sets of a float per length, on
// lines of their own.  With one set its atomics queued: 2.1 million windows of
// 51 lengths took 265 to 298 us, 200,000 took 69; with 16 sets 157 and 30, with
// 64 132 and 23, but they lie in the head that is read back.
constexpr int kJeSets = 32;
__host__ __device__ inline int64_t je_pitch(int L) { return ((int64_t)L + 31) & ~(int64_t)31; }

// ------------------------------------------------------------- helpers

__device__ __forceinline__ int lane_id() { return __lane_id(); }

__device__ __forceinline__ uint64_t lanemask_lt() {
    return (1ull << lane_id()) - 1ull;
}

// Snapped distance (Sec. 3.6: values below eps0 are reported as 0).
__device__ __forceinline__ double snap(double d) { return d < kEps0 ? 0.0 : d; }

__device__ __forceinline__ uint64_t dbits(double d) {
    return (uint64_t)__double_as_longlong(d);
}
__device__ __forceinline__ double bitsd(uint64_t b) {
    return __longlong_as_double((long long)b);
}

// fp16 with round to nearest even, as its 16 bits, and back.
__device__ __forceinline__ uint32_t half_bits(float x) {
    const _Float16 h = (_Float16)x;
    uint16_t u;
    __builtin_memcpy(&u, &h, 2);
    return u;
}
__device__ __forceinline__ float half_float(uint32_t b) {
    const uint16_t u = (uint16_t)b;
    _Float16 h;
    __builtin_memcpy(&h, &u, 2);
    return (float)h;
}

// The value of lane (l ^ X), X in {1, 2, 4}, through the data-parallel
// primitives (no LDS round trip as in a general shuffle).
template <int X>
__device__ __forceinline__ int xor_lane(int v) {
    static_assert(X == 1 || X == 2 || X == 4, "within a group of eight lanes");
    if (X == 1) return __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true);   // quad 1 0 3 2
    if (X == 2) return __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true);   // quad 2 3 0 1
    // l ^ 3 within quads, then l ^ 7 within halves of a row
    v = __builtin_amdgcn_update_dpp(0, v, 0x1B, 0xF, 0xF, true);
    return __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, true);
}
template <int X>
__device__ __forceinline__ uint32_t xor_lane(uint32_t v) {
    return (uint32_t)xor_lane<X>((int)v);
}
template <int X>
__device__ __forceinline__ float xor_lane(float v) {
    return __int_as_float(xor_lane<X>(__float_as_int(v)));
}
template <int X>
__device__ __forceinline__ double xor_lane(double v) {
    return __hiloint2double(xor_lane<X>(__double2hiint(v)), xor_lane<X>(__double2loint(v)));
}

// Adds to this block's set of a counter.
__device__ __forceinline__ void count_add(unsigned long long *counters, int c,
                                          unsigned long long v) {
    atomicAdd(&counters[(blockIdx.x % kCtrSlots) * kCtrStride + c], v);
}

// Length index of a cell (binary search over cell_base, L is small).
__device__ __forceinline__ int find_len(const LenInfo *len, int L, int64_t cell) {
    int lo = 0, hi = L - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (len[mid].cell_base <= cell) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Length index of an indexed position k (slots share the per-length ranges).
__device__ __forceinline__ int find_len_k(const LenInfo *len, int L, int64_t k) {
    int lo = 0, hi = L - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (len[mid].kbase <= k) lo = mid; else hi = mid - 1;
    }
    return lo;
}

constexpr int kJoinTile = 32;             // windows per threshold-join tile
constexpr int kJoinBlock = 4;             // query tiles per block (one wavefront)
constexpr int kJoinOp = 4;                // uint4 words of one window's join operands
constexpr int kJoinDirs = 3;              // principal directions per length in the join
constexpr int kJoinNb = 1;                // join grid cells are 1/kJoinNb of the radius wide; a
                                          // pair within it lies at most kJoinNb cells apart

// Per length, one round of the threshold join (k_join.hip).
struct GridLen {
    int64_t blk_base;     // first join block (kJoinBlock tiles) of this length
    double qlo;           // grid origin of both coordinates
    double hinv;          // 1 / cell width of the first coordinate (0: one cell)
    double hinv2;         // 1 / cell width of the second and third coordinates
    double Tr;            // T sqrt(m/2), the radius on the true features (+inf: every pair)
    double eps_c;         // MFMA dot-product error per unit |G_q| (times the largest |G_c|)
    double nmax2;         // square of the largest |G|
    float sqrt2m;         // sqrt(2/m) (1 + 1e-7)
    float rp;             // bound on any coordinate difference of a pair within R_f
};

// The power of two c >= 1 that brings every filter term of the join, at most
// 2.5 nmax^2 in absolute value (nmax: the largest |G| of length m), into the
// range of an fp16 number: the two operand slots past the features hold c on
// the candidate's side and the term over c, as hi + lo, on the query's.
__host__ __device__ inline float join_scale(int m) {
    const float nmax2 = 0.5f * (float)m * (float)m * 1.03f + 2.0f * (float)m + 2.0f;
    float c = 1.0f;
    while (32768.0f * c < 2.5f * nmax2) c *= 2.0f;
    return c;
}

// The largest |G| of windows of m samples, and the join's dot-product error per
// unit |G_q| (times that |G_c|): at most 34 additions of its products that round
// by up to 2^-23, four times over.
__host__ __device__ inline double join_nmax(int m) {
    return (double)m / 1.4142135623730951 * 1.01 + 1.0;
}
__host__ __device__ inline double join_eps(double nmax) { return 1.6e-5 * nmax; }

// The query's filter term v: a pair is kept iff <G_q, G_c> + v - 0.5 |G_c|^2 >= 0
// as the tiles sum it, so v is at least 0.5 (R^2 - |G_q|^2) plus every rounding
// of the left side.  Tr: radius on the true features; eps_c, nmax2: of the length
// (GridLen); n2, ep, gn: |G|^2, e' and the bound on |G| of the query; je: the
// length's largest e'.
__host__ __device__ inline double join_filter_term(double Tr, double eps_c, double nmax2, float n2,
                                                   float ep, float gn, float je, float scale) {
    const double R = (Tr + (double)ep + (double)je) * (1.0 + 1e-9);
    const double nG2 = (double)n2 * (1.0 - 0x1.0p-23);
    double v = 0.5 * (R * R * (1.0 + 1e-9) - nG2) + eps_c * (double)gn + 1e-30;
    v += 0x1.0p-22 * (fabs(v) + nmax2);
    // the sums start at -0.5 |G_c|^2: at most 34 additions that round by up to
    // 2^-23 of it
    v += 4.5e-6 * nmax2;
    // the slots' share of the accumulation (at most 34 additions) and of the
    // split into hi + lo
    v += 5e-6 * fabs(v) + 0x1.0p-12 * (double)scale;
    return v;
}

// State of the device-side radix select (k_certify.hip).
constexpr int kSelBins = 2048;            // bins of one select pass (11 bits)
struct SelState {
    uint64_t high;        // bits of the selected prefix so far
    uint64_t pivot;       // cells below it are taken (kInfBits: every value)
    int64_t remaining;    // values still wanted at or below the prefix
    int64_t below;        // values known to lie below the pivot (or, with ties, before tie_lo)
    int64_t need_eq;      // values equal to the pivot to take, in position order
    int64_t tie_lo, tie_hi;   // positions among which the last of them lies
    int64_t pos_limit;    // ties before this position are taken (0: not known yet)
    uint32_t nless;       // cells found by the emit pass
    int32_t done;         // the pivot is known
    uint64_t kept;        // the join's counts when the greedy ran: kept pairs,
    uint32_t nredo;       // overflowed blocks
    uint32_t ticket;      // blocks of the running pass that have arrived (0 between passes)
    int32_t naccept;      // cells accepted by the device's greedy
    int32_t pad_;
    uint64_t improved;    // *Select::improved
};
// A selected cell: its value's bits, position and cell.
struct SelCell {
    uint64_t v;
    uint32_t k, cell;
};
// Where the lengths' cells begin, for the greedy: first cell and window length
// of each, read out of an array of any record type.
struct LenView {
    const char *base;     // record of length 0
    int64_t stride;       // bytes from one record to the next
    int32_t off_cell, off_m;   // offsets of the first cell (int64) and the length (int32)
    int32_t L;
    __device__ __forceinline__ int64_t cell0(int l) const {
        return *(const int64_t *)(base + l * stride + off_cell);
    }
    __device__ __forceinline__ int m(int l) const {
        return *(const int32_t *)(base + l * stride + off_m);
    }
    __device__ __forceinline__ int find(int64_t cell) const {
        int lo = 0, hi = L - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (cell0(mid) <= cell) lo = mid; else hi = mid - 1;
        }
        return lo;
    }
};
// One selection's buffers.  The greedy runs on the device while the selected
// cells fit one block's registers and k rounds of it are short against a copy
// and a sort on the host (about 1 us each); otherwise the host reads all of
// them.
constexpr int kGreedyMax = 16384;         // selected cells the device's greedy holds
constexpr int kGreedyRounds = 128;
constexpr int64_t kSelSlack = 2048;       // cells beyond `need` that the select may take
struct Select {
    SelState *st;
    SelCell *acc;         // [k] accepted cells (device greedy)
    uint64_t *sel_val;    // [cap] selected cells: value bits, position, cell,
    uint32_t *sel, *sel_cell;
    int2 *sel_len;        // index and window length of its length
    unsigned int *hist;   // [kSelBins], zero between selections (as st->ticket)
    const unsigned long long *improved;   // a counter that travels with the state, or null
    int64_t need, cap;
    int k;
    bool on_device() const { return cap <= kGreedyMax && k <= kGreedyRounds; }
};

struct RowReq {
    int32_t l;          // length index
    int32_t pad;
    int64_t k;          // indexed position of the cell
    uint64_t target;    // pass 2: FP64 bits of the value whose smallest j is wanted
};

// The canonical exact distance, computed by a group of kGroup consecutive
// lanes (kPerRound groups per wavefront, each with its own pair): lane g of
// the group sums the terms r = g, g + kGroup, ... in ascending order, then a
// butterfly over the group adds the partial sums.  Every kernel that writes,
// compares or reports a distance calls this function, so they all agree bit
// for bit; every step is symmetric in (a, b), so d(a, b) == d(b, a).  Loads
// of a group are contiguous.  All 64 lanes of the wavefront must call it.
constexpr int kGroup = 8;                 // lanes per exact distance
constexpr int kPerRound = kWave / kGroup; // distances per wavefront round
constexpr int kZBatch = 8;                // terms per lane loaded together
constexpr int kLaneMode = 32;             // proposals from which each lane takes its own,
constexpr int kLaneModeMaxM = 100;        // for windows up to this length: longer ones
                                          // read better in groups (contiguous loads);
                                          // measured crossover between 100 and 124

// The first window's samples are read through an accessor: the series
// itself, or a copy of the same samples staged in LDS; the second window's
// come from the series.
struct SeriesA {
    const double *t;
    __device__ __forceinline__ double operator()(int64_t x) const { return t[x]; }
};

template <int kB = kZBatch, class A>
__device__ __forceinline__ double group_zdist_a(A qa, const double *__restrict__ t, int64_t a,
                                                double mua, double ia, int64_t b, double mub,
                                                double ib, int m, double lim2 = INFINITY) {
#pragma clang fp contract(off)
    double acc = 0.0;
    // kB terms per lane are loaded before they are summed (in order), so that
    // a window of up to kB * kGroup samples costs one memory latency (kB = 1:
    // the fewest registers; the sum and its order are the same for any kB)
    for (int r0 = lane_id() & (kGroup - 1); r0 < m; r0 += kB * kGroup) {
        double xa[kB], xb[kB];
#pragma unroll
        for (int u = 0; u < kB; ++u) {
            const int r = r0 + u * kGroup;
            xa[u] = r < m ? qa(a + r) : 0.0;
            xb[u] = r < m ? t[b + r] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < kB; ++u) {
            if (r0 + u * kGroup < m) {
                const double za = (xa[u] - mua) * ia;
                const double zb = (xb[u] - mub) * ib;
                const double e = za - zb;
                acc = fma(e, e, acc);
            }
        }
        // early exit: the partial sums only grow (every term is >= 0 and
        // rounding is monotone), so once their total reaches lim2 the
        // finished sum would too; the group decides together (all its lanes
        // compute the same total)
        if (lim2 != INFINITY && (r0 | (kGroup - 1)) + 1 + (kB - 1) * kGroup < m) {
            double sp = acc;
            sp += xor_lane<1>(sp);
            sp += xor_lane<2>(sp);
            sp += xor_lane<4>(sp);
            if (sp >= lim2) return INFINITY;
        }
    }
    acc += xor_lane<1>(acc);
    acc += xor_lane<2>(acc);
    acc += xor_lane<4>(acc);
    return sqrt(acc);
}
__device__ __forceinline__ double group_zdist(const double *__restrict__ t, int64_t a, double mua,
                                              double ia, int64_t b, double mub, double ib, int m,
                                              double lim2 = INFINITY) {
    return group_zdist_a(SeriesA{t}, t, a, mua, ia, b, mub, ib, m, lim2);
}

// The same canonical distance evaluated by one lane alone, bit for bit: the
// kGroup partial sums of group_zdist become kGroup accumulators of the lane
// (accumulator g takes the terms r = g, g + kGroup, ... in ascending order),
// combined in the order of group_zdist's butterfly.  Used when most lanes of a
// wavefront have a pair of their own, where it avoids the group's shuffles.
static_assert(kGroup == 8, "lane_zdist combines eight partial sums");
__device__ __forceinline__ double butterfly8(const double *p) {
    return ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
}
template <class A>
__device__ __forceinline__ double lane_zdist_a(A qa, const double *__restrict__ t, int64_t a,
                                               double mua, double ia, int64_t b, double mub,
                                               double ib, int m, double lim2 = INFINITY) {
#pragma clang fp contract(off)
    double acc[kGroup];
#pragma unroll
    for (int g = 0; g < kGroup; ++g) acc[g] = 0.0;
    for (int r0 = 0; r0 < m; r0 += kGroup) {
        double xa[kGroup], xb[kGroup];
#pragma unroll
        for (int g = 0; g < kGroup; ++g) {
            xa[g] = r0 + g < m ? qa(a + r0 + g) : 0.0;
            xb[g] = r0 + g < m ? t[b + r0 + g] : 0.0;
        }
#pragma unroll
        for (int g = 0; g < kGroup; ++g) {
            if (r0 + g < m) {
                const double za = (xa[g] - mua) * ia;
                const double zb = (xb[g] - mub) * ib;
                const double e = za - zb;
                acc[g] = fma(e, e, acc[g]);
            }
        }
        // early exit as in group_zdist (any partial total is a lower bound
        // of the finished sum), tested every kZBatch terms per accumulator
        if (lim2 != INFINITY && ((r0 / kGroup) % kZBatch) == kZBatch - 1 && r0 + kGroup < m &&
            butterfly8(acc) >= lim2)
            return INFINITY;
    }
    return sqrt(butterfly8(acc));
}
__device__ __forceinline__ double lane_zdist(const double *__restrict__ t, int64_t a, double mua,
                                             double ia, int64_t b, double mub, double ib, int m,
                                             double lim2 = INFINITY) {
    return lane_zdist_a(SeriesA{t}, t, a, mua, ia, b, mub, ib, m, lim2);
}

// Squared bound for group_zdist's early exit: a sum that reaches it has a
// computed root >= thr (the factor covers the roundings of thr^2 and sqrt).
__device__ __forceinline__ double exit_bound(double thr) {
    return thr == INFINITY ? INFINITY : thr * thr * (1.0 + 8.0 * 1.1102230246251565e-16);
}

// Length index of the indexed positions handled by a wavefront: a scalar
// binary search for the wavefront's first position (uniform, so it runs on
// the scalar unit), then a short per-lane step forward.
__device__ __forceinline__ int find_len_k_wave(const LenInfo *len, int L, int64_t k_first,
                                               int64_t k) {
    int lo = 0, hi = L - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (len[mid].kbase <= k_first) lo = mid; else hi = mid - 1;
    }
    while (lo + 1 < L && len[lo + 1].kbase <= k) ++lo;
    return lo;
}

// Canonical moments of one window x[0..m) (Sec. 3.2: population, two
// passes): returns sigma and sets mu.  Four partial sums in a fixed order
// keep the loads independent; every caller gets the same bits for the same
// samples, which the distances below depend on.
__device__ __forceinline__ double window_moments(const double *x, int m, double &mu) {
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    int r = 0;
    // (the sums are chains; unrolled so that their reads are in flight together)
#pragma unroll 4
    for (; r + 4 <= m; r += 4) {
        a0 += x[r];
        a1 += x[r + 1];
        a2 += x[r + 2];
        a3 += x[r + 3];
    }
    for (; r < m; ++r) a0 += x[r];
    mu = ((a0 + a1) + (a2 + a3)) / (double)m;
    a0 = a1 = a2 = a3 = 0.0;
#pragma unroll 4
    for (r = 0; r + 4 <= m; r += 4) {
        const double c0 = x[r] - mu, c1 = x[r + 1] - mu;
        const double c2 = x[r + 2] - mu, c3 = x[r + 3] - mu;
        a0 = fma(c0, c0, a0);
        a1 = fma(c1, c1, a1);
        a2 = fma(c2, c2, a2);
        a3 = fma(c3, c3, a3);
    }
    for (; r < m; ++r) {
        const double c0 = x[r] - mu;
        a0 = fma(c0, c0, a0);
    }
    return sqrt(((a0 + a1) + (a2 + a3)) / (double)m);
}

// The bound from the squared distance of two feature records and the sum of
// their errors.
template <typename FT>
__device__ __forceinline__ float lb_of(FT acc, FT es, float sqrt2m) {
    const FT nd = sqrt(acc);
    if (sizeof(FT) == 4) {
        float v = (float)nd * (1.0f - 1e-5f) - (float)es * (1.0f + 1e-5f);
        return v > 0.0f ? v * sqrt2m * (1.0f - 1e-6f) : 0.0f;
    } else {
        double v = (double)nd * (1.0 - 1e-12) - (double)es * (1.0 + 1e-12);
        return v > 0.0 ? __double2float_rd(v * (double)sqrt2m * (1.0 - 1e-6)) : 0.0f;
    }
}

// Certified lower bound on d_m(q, c) from two stored feature records: the
// Parseval bound (Lemma 2) of the true features is at least
//   sqrt(2/m) (||F~q - F~c|| - e_q - e_c),
// and every rounding of this evaluation is absorbed by the relative slacks
// (applied to the norm before the subtraction, so the result never exceeds
// the true bound even when the two terms nearly cancel).  All 30 slots are
// used: slots beyond 2K' are zero on both sides and add nothing.
template <typename FT>
__device__ __forceinline__ float lb_mem(const FT *__restrict__ fq, const FT *__restrict__ fc,
                                        float sqrt2m) {
    FT acc = 0;
    if (sizeof(FT) == 8) {
        const double2 *a = (const double2 *)fq;
        const double2 *b = (const double2 *)fc;
#pragma unroll
        for (int x = 0; x < kMaxK - 1; ++x) {
            const double2 u = a[x], v = b[x];
            const double e0 = u.x - v.x, e1 = u.y - v.y;
            acc = fma(e0, e0, acc);
            acc = fma(e1, e1, acc);
        }
    } else {
        const float4 *a = (const float4 *)fq;
        const float4 *b = (const float4 *)fc;
#pragma unroll
        for (int x = 0; x < 7; ++x) {
            const float4 u = a[x], v = b[x];
            const float e0 = u.x - v.x, e1 = u.y - v.y, e2 = u.z - v.z, e3 = u.w - v.w;
            acc = fmaf(e0, e0, acc);
            acc = fmaf(e1, e1, acc);
            acc = fmaf(e2, e2, acc);
            acc = fmaf(e3, e3, acc);
        }
        const float2 u = ((const float2 *)fq)[14], v = ((const float2 *)fc)[14];
        const float e0 = u.x - v.x, e1 = u.y - v.y;
        acc = fmaf(e0, e0, acc);
        acc = fmaf(e1, e1, acc);
    }
    return lb_of(acc, fq[kSlotErr] + fc[kSlotErr], sqrt2m);
}

constexpr int kPart = kRec / kGroup;          // record slots per lane of a group

// A lane's part of one record (slots kPart g .. + kPart - 1).
template <typename FT>
struct RecPart {
    FT v[kPart];
};
__device__ __forceinline__ RecPart<double> load_part(const double *rec, int g) {
    const double2 a = ((const double2 *)rec)[2 * g], b = ((const double2 *)rec)[2 * g + 1];
    return {{a.x, a.y, b.x, b.y}};
}
__device__ __forceinline__ RecPart<float> load_part(const float *rec, int g) {
    const float4 a = ((const float4 *)rec)[g];
    return {{a.x, a.y, a.z, a.w}};
}

// The certified bounds of lb_mem for the eight candidates of a group, whose
// indices sit one per lane (kc; `want`: this lane's is wanted; m8: the wanted
// ones of the group as a bit mask).  Lane g returns candidate g's bound (0 if
// not wanted).  fq: this lane's part of the query's record, eq its error.
template <typename FT>
__device__ __forceinline__ float group_lb(const FT *__restrict__ F, const RecPart<FT> &fq, FT eq,
                                          uint32_t kc, bool want, uint32_t m8, int g,
                                          float sqrt2m) {
    FT ec = 0;
    if (want) ec = F[(int64_t)kc * kRec + kSlotErr];
    FT p[kGroup];
#pragma unroll
    for (int c = 0; c < kGroup; ++c) {
        p[c] = 0;
        const uint32_t kcc = (uint32_t)__shfl((int)kc, c, kGroup);
        if ((m8 >> c) & 1u) {
            const RecPart<FT> r = load_part(F + (int64_t)kcc * kRec, g);
            const FT e0 = r.v[0] - fq.v[0], e1 = r.v[1] - fq.v[1];
            FT e2 = r.v[2] - fq.v[2], e3 = r.v[3] - fq.v[3];
            if (g == kGroup - 1) e2 = e3 = 0;           // the error and the norm
            p[c] = e0 * e0 + e1 * e1 + e2 * e2 + e3 * e3;
        }
    }
    // transposed reduction: after it lane g holds the sum of candidate g
    FT h[4], q[2];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const FT send = (g & 4) ? p[c] : p[c + 4], keep = (g & 4) ? p[c + 4] : p[c];
        h[c] = keep + xor_lane<4>(send);
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const FT send = (g & 2) ? h[c] : h[c + 2], keep = (g & 2) ? h[c + 2] : h[c];
        q[c] = keep + xor_lane<2>(send);
    }
    const FT send = (g & 1) ? q[0] : q[1], keep = (g & 1) ? q[1] : q[0];
    const FT acc = keep + xor_lane<1>(send);
    return lb_of(acc, eq + ec, sqrt2m);
}

// Verification of the proposals of a wavefront.  Every lane whose bit is set
// in `mask` has a proposal (a, b: window starts; mua, ia, mub, ib: moments;
// m; lim2: the squared distance at or above which the result is of no use,
// see exit_bound).  With at least kLaneMode proposals of windows up to
// kLaneModeMaxM samples (the length of the first proposal decides for the
// wavefront) every proposing lane evaluates its own (lane_zdist); otherwise
// they are taken kPerRound at a time,
// one per group of kGroup lanes (group_zdist).  Both give the same bits.
// `on_result(d)` runs on the proposing lane with its snapped distance (+inf
// when the sum stopped early).
template <bool kLaneForm = true, int kB = kZBatch, class A, typename F>
__device__ __forceinline__ void verify_proposals(uint64_t mask, A qa, const double *__restrict__ t,
                                                 int64_t a, double mua, double ia, int64_t b,
                                                 double mub, double ib, int m, F &&on_result,
                                                 double lim2 = INFINITY) {
    const int lane = lane_id();
    if (kLaneForm && __popcll(mask) >= kLaneMode &&
        __shfl(m, __ffsll((unsigned long long)mask) - 1, kWave) <= kLaneModeMaxM) {
        // most lanes propose short windows: each evaluates its own pair
        if ((mask >> lane) & 1ull)
            on_result(snap(lane_zdist_a(qa, t, a, mua, ia, b, mub, ib, m, lim2)));
        return;
    }
    const int grp = lane / kGroup;
    while (mask) {
        // the next kPerRound proposing lanes, in lane order
        int src[kPerRound];
        int cnt = 0;
#pragma unroll
        for (int g = 0; g < kPerRound; ++g) {
            src[g] = -1;
            if (mask) {
                src[g] = __ffsll((unsigned long long)mask) - 1;
                mask &= mask - 1;
                ++cnt;
            }
        }
        int mys = src[0];
#pragma unroll
        for (int g = 1; g < kPerRound; ++g)
            if (grp == g && src[g] >= 0) mys = src[g];
        const bool live = grp == 0 || (grp < cnt);
        const int my = mys;
        const int64_t ga = __shfl(a, my, kWave);
        const int64_t gb = __shfl(b, my, kWave);
        const double gmua = __shfl(mua, my, kWave), gia = __shfl(ia, my, kWave);
        const double gmub = __shfl(mub, my, kWave), gib = __shfl(ib, my, kWave);
        const double glim = __shfl(lim2, my, kWave);
        int gm = __shfl(m, my, kWave);
        if (!live) gm = 0;
        const double d = snap(group_zdist_a<kB>(qa, t, ga, gmua, gia, gb, gmub, gib, gm, glim));
        // hand each result back to its proposing lane
#pragma unroll
        for (int g = 0; g < kPerRound; ++g) {
            const double dg = __shfl(d, g * kGroup, kWave);
            if (g < cnt && lane == src[g]) on_result(dg);
        }
    }
}

// ------------------------------------------------------------- stream

// One anchor length of a stream session, as the kernels of one batch see it
// (Sec. 3.1, 3.5, Algorithm 1).  Cells of the anchor are its window starts
// q at cbase + q.  The directory is the anchor's indexed windows in
// arrival order, cut into sorted runs: run r holds the indexed positions
// [runs[r], runs[r + 1]), sorted by (SimHash key, start).
constexpr int kStreamMaxRuns = 48;
constexpr uint32_t kStreamMergeLds = 4096;    // entries of a merge that one block holds
struct SAnchor {
    int32_t m, kprime;
    int64_t cbase;        // first cell
    int64_t bbase;        // offset of the basis table (m rows of 2 K' doubles)
    int32_t nidx;         // indexed windows before this batch
    int32_t nnew;         // indexed windows this batch completes
    int32_t j0;           // first entry of the batch list that is this anchor's
    int32_t depth;        // directory depth d (Prop. 4)
    int32_t probes;       // Hamming-1 probes h
    int32_t nruns;
    int32_t merge;        // the merge that k_stream_finish does for it (-1: none)
    int32_t pad_;
    uint32_t runs[kStreamMaxRuns + 1];
};

// A candidate endpoint's improvement, merged after the batch's searches.
struct SUpdate {
    uint32_t cell;
    int32_t j;            // the query start that reached it
    uint64_t d;           // FP64 bits of the distance
};

// One merge of the newest runs of one anchor into a single run.
struct SMerge {
    int64_t cbase;
    int64_t first;        // first thread of this merge in the launch
    int32_t nruns;        // runs merged
    int32_t pad_;
    uint32_t runs[kStreamMaxRuns + 1];
};

// Kernel arguments of a stream batch.
struct StreamDev {
    const double *t;      // resident series
    double *F;            // [cells][kRec] records
    double *mu, *isig;    // [cells]
    uint64_t *P;          // [cells] upper profile (FP64 bits; +inf: none)
    int32_t *I;           // [cells] its neighbour (-1: none)
    int32_t *Icand;       // [cells] merge scratch
    uint32_t *perm, *skey;   // [cells] directory runs (start, key) by position
    uint32_t *ptmp, *ktmp;   // [cells] merge scratch
    const double *basis;
    const float *gproj;   // [anchor][kMaxBits][30] SimHash projections
    const SAnchor *anc;
    const int32_t *la, *lq;  // batch list: anchor, start
    int32_t nlist;
    int32_t B;            // signature bits
    int32_t R;            // budget per query (gamma alpha)
    int32_t excl;
    uint32_t *bkey;       // [list] SimHash key
    float *bmarg;         // [list][kMaxBits] projection margins
    SUpdate *upd;
    uint32_t *nupd;
    uint32_t updcap;
    unsigned long long *counters;   // kCtrSlots sets, kCtrStride apart (count_add)
};
enum { CS_CAND = 0, CS_VER, CS_UPD, CS_DROP, kStreamCounters };

// The 16-bit copy of the series for the prefilter of exact distances (quant.h;
// x16 null: none): two arrays of `pitch` entries, the range of the samples
// they were made from, and per indexed window what the sums need.
struct Quant {
    int16_t *x16;
    int64_t pitch;
    unsigned long long *mm;
    float4 *xw;
};

// --------------------------------------------------- host-side launchers
// (k_scan.hip)
size_t scan_temp_bytes(int64_t n);
// out[i] = sum_{j<i} in[j]; total (optional, device) = sum of all.
void scan_exclusive_u32(const uint32_t *in, uint32_t *out, int64_t n, uint32_t *total,
                        void *temp, hipStream_t s);
size_t sort_temp_bytes(int64_t n);
// Stable LSD radix sort of (key, val) pairs on key bits [lo, hi).  Result in
// (k0, v0), or, after an odd number of passes with copy_back false, in
// (k1, v1): the return value is 1 then, 0 otherwise.  (k1, v1) are scratch
// of the same size.  ticket: a word that is 0 before and after.
int radix_sort_pairs(uint32_t *k0, uint32_t *v0, uint32_t *k1, uint32_t *v1, int64_t n,
                     int lo, int hi, void *temp, uint32_t *ticket, hipStream_t s,
                     bool copy_back = true);

// (k_sketch.hip)
void launch_changepoints(const double *t, int64_t n, uint32_t *flag, int *bad, hipStream_t s);
// (also clears tile_cnt[ntiles]; starts = windows of the shortest length)
void launch_tile_counts(const LenInfo *len, int L, const uint32_t *E, int64_t starts, int max_m,
                        int64_t ntiles, uint32_t *tile_cnt, hipStream_t s);
// Which tiles the sketch gives records: every length (kSketchAll), the anchor
// lengths (kSketchAnchors), or the lengths between anchors (kSketchBetween)
enum { kSketchAll = 0, kSketchAnchors = 1, kSketchBetween = 2 };
// The tiles of a sketch launch: all tiles [0, ntiles) of the lengths in turn, or
// the anchors' (every stride-th length and the last; starts: windows of the
// shortest length).
struct SketchGrid {
    int64_t ntiles, starts;
    int stride, anchors;
};
// Positions, moments and initial values of every window.
void launch_moments(const Req &q, const uint32_t *E, const uint32_t *tile_off, const SketchGrid &g,
                    int max_m, hipStream_t s);
void launch_sketch(const Req &q, const uint32_t *E, const uint32_t *tile_off, const SketchGrid &g,
                   int max_m, int mode, hipStream_t s);
void launch_keys(int precision, const Req &q, int64_t nblocks, hipStream_t s);
void launch_join_ops(int precision, const Req &q, int64_t k0, int64_t k1, hipStream_t s);
int64_t basis_elems(const LenInfo *len_host, int L, std::vector<int64_t> &base);
void launch_basis(const LenInfo *len, int L, const int64_t *base, uint16_t *bh, uint16_t *bm,
                  uint16_t *bl, int max_m, hipStream_t s);
void launch_sketch_mfma(const Req &q, const uint32_t *E, const uint32_t *tile_off,
                        const SketchGrid &g, int max_m, const int64_t *bbase, const uint16_t *bh,
                        const uint16_t *bm, const uint16_t *bl, int mode, hipStream_t s);
void launch_bucket_bounds(const Req &q, int64_t N, int64_t nbuckets, uint32_t *bstart,
                          hipStream_t s);
// A probe that the device may call off: nothing runs once *zeros >= limit (null:
// always).
struct ProbeIf {
    const unsigned long long *zeros;
    unsigned long long limit;
};
// (k_probe.hip)
// one wavefront per kProbeQ indexed windows of each anchor length (LenInfo.pblk_base):
// the probe blocks [blk0, blk0 + nblocks)
// cut: pairs above it are of no interest (+inf: none), x: the prefilter for
// them (x16 null with cut = +inf)
void launch_probe(int precision, const Req &q, const uint32_t *bstart, int64_t blk0,
                  int64_t nblocks, int max_m, double cut, const Quant &x, const ProbeIf &go,
                  hipStream_t s);
// the work-items of the largest launch of a probe of that many blocks
int64_t probe_work_items(int64_t nblocks);
void launch_hot_buckets(const uint32_t *bstart, int64_t nb, int R, unsigned long long *cnt,
                        hipStream_t s);
// (k_complete.hip): the emit stage
// the hints: one wavefront per 64 indexed windows of each length between
// anchors (LenInfo.hblk_base)
// (cut and x as in launch_probe)
void launch_hints(int precision, const Req &q, int64_t nblocks, double cut, const Quant &x,
                  hipStream_t s);
void launch_sieve_count(const Req &q, const uint32_t *bstart, int64_t nbuckets, int R,
                        uint32_t *cnt, hipStream_t s);
void launch_sieve_keys(int precision, const Req &q, const uint32_t *bstart, const uint32_t *off,
                       int64_t nbuckets, uint32_t total, const float *dir, uint32_t *key,
                       uint32_t *val, uint32_t *seg, hipStream_t s);
void launch_sieve_regroup(const uint32_t *val, const uint32_t *seg, uint32_t total, uint32_t *key2,
                          hipStream_t s);
void launch_sieve_verify(int precision, const Req &q, const uint32_t *bstart, const uint32_t *off,
                         const uint32_t *order, const uint32_t *seg, uint32_t total, int w,
                         hipStream_t s);
void launch_complete(int precision, const Req &q, const uint32_t *seeds, int nseeds, int dm,
                     int dp, hipStream_t s);
// (k_certify.hip)
// The first `need` values of P[0 .. n) in (value, position) order (perhaps a
// few more, st->nless of them, unordered in sel / sel_val), then the greedy over
// them, or with on_device() false the cells of all of them.  Everything runs on
// the stream; the state holds the counts when the stream reaches the end, with
// the join's counts (null: none).
void launch_select(const Select &x, const uint64_t *P, int64_t n, const uint32_t *cell,
                   const LenView &lv, const unsigned long long *counts, hipStream_t s);
// Spectral width from samples (Sec. 3.2; k_sketch.hip): up to kWidthSets
// lengths, up to kWidthWin windows of each.
constexpr int kWidthSets = 3, kWidthWin = 256, kWidthMin = 4;
struct WidthSets {
    int32_t sets;
    int32_t m[kWidthSets];
    int64_t W[kWidthSets];
};
// What the choice of K needs of one length's samples at one candidate K.
struct WidthSums {
    double energy;         // retained energy, summed over the windows
    double coll;           // collision probability, summed over the pairs
    int64_t pairs, windows;
};
__host__ __device__ inline int64_t width_start(int64_t W, int j) {
    return W <= kWidthWin ? j : (int64_t)((double)j * (double)(W - 1) / 255.0);
}
__host__ __device__ inline int width_kprime(int K, int m) {
    const int half = (m + 1) / 2 - 1, kp = K - 1 < half ? K - 1 : half;
    return kp < 0 ? 0 : kp;
}
constexpr int64_t kWidthSpec = (int64_t)kWidthSets * kWidthWin * kMaxK;   // double2 of scratch
// out[set][K - kWidthMin], K = kWidthMin .. kMaxK
void launch_width(const double *t, const WidthSets &w, int B, double2 *spec, WidthSums *out,
                  hipStream_t s);
// Small host data to the device through kernel arguments, read when the call
// returns; also clears `zero_words` words at `zero` (null: none).  False: too
// long for that, nothing was done.  (k_scan.hip)
bool launch_upload(void *dst, const void *src, size_t bytes, uint32_t *zero, int64_t zero_words,
                   hipStream_t s);
// offs[l] = tile_off at length l's first tile, offs[L] at the end
void launch_len_offsets(const LenInfo *len, int L, const uint32_t *tile_off, int64_t ntiles,
                        uint32_t *offs, hipStream_t s);
// (k_join.hip)
// Bytes of the sorted operands of N windows of L lengths; the directions'
// sample sums lie there before.
size_t join_sorted_bytes(int64_t N, int L);
// principal directions: covariance of a sample, then power iteration (GPU)
// principal directions of the lengths [0, nlen) (the lengths whose records
// exist)
void launch_join_dirs(int precision, const Req &q, int nlen, double *cov, double *udir,
                      hipStream_t s);
// grid keys over cb1 (and cb2, cb3 when nonzero) bits of the principal
// coordinates, of the first N indexed windows; queries are the cells not at 0
// with (length, start) <= (l_lim, i_lim); nonq[l] is set where some window of
// length l is not one
void launch_grid_keys(const Req &q, const GridLen *gl, int64_t N, int cb1, int cb2, int cb3,
                      int l_lim, int64_t i_lim, uint32_t *gkey, uint32_t *gval, uint8_t *qf,
                      float4 *gp, uint32_t *nonq, hipStream_t s);
// the join operands and coordinates of the first n sorted positions, in
// sorted order
void launch_join_gather(const uint32_t *gval, const uint4 *jop, const float4 *gp, int64_t n,
                        uint4 *jop_s, float4 *gp_s, float *gw_s, hipStream_t s);
// What one round's tiles read.
struct JoinIn {
    int precision;
    Req q;
    const GridLen *gl;
    const uint32_t *gkey, *gval;
    const uint8_t *qf;
    const uint4 *jop_s;
    const float4 *jmeta, *gp_s;
    const float *gw_s;
    int64_t nwin;         // windows in the order
    const uint32_t *nonq;
    int cb1, cb2, cb3;
    double T;
};
// Where the tiles' kept pairs go: kCtrSlots segments of segcap pairs each,
// their fill counts kCtrStride apart in pcount (a block writes to the segment
// of its workgroup, workgroup % kCtrSlots, so that reservations do not queue on
// one address: the blocks of a launch of up to kCtrSlots have a segment each);
// blocks that find theirs full go to `redo` (*nredo of them, one entry per block
// of a launch).
struct JoinOut {
    uint2 *pairs;
    unsigned long long *pcount;
    int64_t segcap;
    uint32_t *redo;
    uint32_t *nredo;
};
// Which of a launch's blocks a workgroup takes.  Consecutive blocks share most of
// their candidates and workgroups go to the eight XCDs in turn, so each XCD takes
// runs of consecutive blocks: 128 (16,384 queries), or an eighth of a launch of
// fewer than 1024, so that every XCD has some.  The tiles themselves hardly care
// (ECG-like 1M with runs of 1, 16 and 128: 91.6, 91.3, 91.1 ms a request), but the
// pairs of a segment are then neighbours and k_join_verify takes them on the XCD
// that found them: with runs of 8 instead of 128 it took 372 us instead of 270 for
// a random walk of 20,714 at 292..317 (4,150 blocks).  Longer runs leave XCDs
// waiting for the one with the heavy blocks: 100.6 ms with 1024 at ECG-like 1M;
// 128 themselves cost 200,000 samples of one length (1,563 blocks) 7.4 ms against
// 6.9 with 16.  (128 whatever the launch put up to 128 blocks on one XCD and 64 into
// eight segments of the pair buffer, so that lists of overflowed blocks overflowed
// again: 13.9 ms there, 30.2 instead of 9.2 at 30,000, 41 lengths and four bins.)
constexpr int kXcds = 8;
constexpr int64_t kJoinRun = 128;
inline int join_run(int64_t nblocks) {
    const int64_t r = (nblocks + kXcds - 1) / kXcds;
    return (int)(r < 1 ? 1 : r < kJoinRun ? r : kJoinRun);
}
// (whole rounds of runs: workgroups past the last block end at once)
inline int64_t join_workgroups(int64_t nblocks) {
    const int64_t round = (int64_t)kXcds * join_run(nblocks);
    return (nblocks + round - 1) / round * round;
}
__host__ __device__ inline int64_t join_block_of(int64_t workgroup, int run) {
    const int64_t seq = workgroup / kXcds;
    return (seq / run * kXcds + workgroup % kXcds) * run + seq % run;
}
// one wavefront of kJoinBlock query tiles per GridLen block: the blocks
// [blk0, blk0 + nblocks) of the round, or the first nblocks of a list
void launch_join_tiles(const JoinIn &in, int64_t blk0, int64_t nblocks, const uint32_t *list,
                       const JoinOut &out, hipStream_t s);
// the n blocks of a list, their kept pairs verified in place
void launch_join_redo(const JoinIn &in, const uint32_t *list, uint32_t n, hipStream_t s);
int64_t quant_pitch(int64_t n);
void launch_quant_series(const double *t, int64_t n, const Quant &x, hipStream_t s);
void launch_quant_windows(const Req &q, int64_t k0, int64_t k1, const Quant &x, hipStream_t s);
// the exact stage of the pairs in the buffer's segments, behind the prefilter
// when x holds one
void launch_join_verify(int precision, const Req &q, const GridLen *gl, const JoinOut &out,
                        double T, const Quant &x, hipStream_t s);
void launch_rows(const Req &q, const RowReq *rr, int nrows, int64_t maxN,
                 unsigned long long *out_min, unsigned long long *out_arg, hipStream_t s);
void launch_stream_basis(const SAnchor *anc, int na, int64_t elems, double *basis,
                         hipStream_t s);
void launch_stream_windows(const StreamDev &S, int max_m, hipStream_t s);
void launch_stream_probe(const StreamDev &S, int max_m, hipStream_t s);
void launch_stream_finish(const StreamDev &S, int na, const SMerge *mg, hipStream_t s);
void launch_stream_merge(const StreamDev &S, const SMerge *mg, int nmerge, int64_t nthreads,
                         hipStream_t s);
void launch_iota_u32(uint32_t *p, int64_t n, hipStream_t s);
void launch_fill_u64(uint64_t *p, int64_t n, uint64_t v, hipStream_t s);
// *out += the number of zeros among P[0 .. n)
void launch_count_zero(const uint64_t *P, int64_t n, unsigned long long *out, hipStream_t s);
void launch_fill_u32(uint32_t *p, int64_t n, uint32_t v, hipStream_t s);

}  // namespace pmp
