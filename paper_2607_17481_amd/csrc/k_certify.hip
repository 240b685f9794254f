// k_certify.hip -- top-k selection, exact threshold join and exact rows.
//
// Selection (paper Sec. 2 top-k rule; Sec. 3.6 final report): the greedy
// reads cells in (distance, m, i) order and accepts a cell unless an accepted
// cell of the same length lies within m/2.  Each accepted cell excludes at
// most m others, so the first k(m_max + 1) cells of that order decide the
// first k acceptances; they are found by a radix select on the FP64 bit
// pattern of the profile followed by an ordered compaction.
//
// Certificate (not in the paper): after the one pass the profile is a sound
// upper bound (Prop. 1).  Let T be the k-th value the greedy accepts on it.
// The threshold join (k_join.hip) gives every cell whose exact value is <= T
// its exact value; if the greedy's k-th acceptance is then still <= T the
// top-k is exact, otherwise T grows and the join repeats.
//
// Rows: the nearest neighbour j of each reported cell is the smallest j at
// the minimum, found by a brute-force scan of the whole row (two passes: the
// minimum, then the smallest j attaining it).
#include "pmp_dev.h"

namespace pmp {

// ---------------------------------------------------------------- select

// The radix select runs on the device from start to end: up to six passes of a
// histogram over 11 (the last 2) bits of a key of the value, whose last block
// picks the bin holding the `remaining`-th smallest value and narrows the
// prefix `high`.  The key counts the bit pattern from 2^-20 on, below every value
// but 0, so that the first pass's 2048 bins divide 1e-6 to 128 (distances are at
// most 2 sqrt(m), 90.5) sixty-four to the octave: the pattern's own top bits fill
// about twenty of them, which took a second pass and put a wavefront's counts on
// the same few addresses.  It is over as soon as the cells at or below that bin fit the
// output (usually after two or three passes; the greedy sorts out the rest),
// and the passes after that return at once.  The state lives in a SelState,
// whose ticket and histogram every pass leaves cleared for the next.
//
// What bounds it: launches and the reads of P.  With a pick kernel per pass,
// always six passes, a three-kernel scan for ties and the greedy on the host
// (a copy and a sort of k (m_max + 1) cells), a selection took about 0.3 ms at
// 200,000 cells and 0.6 ms at windows of 400; it now takes 0.1 ms there, half
// of it the greedy's chain of rounds.

// Arrival of a block at the end of a kernel: true in the last one (uniform).
// Everything the blocks wrote before is visible to it.
__device__ __forceinline__ bool last_block(SelState *st) {
    __shared__ int last;
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) last = atomicAdd(&st->ticket, 1u) == gridDim.x - 1;
    __syncthreads();
    if (last) {
        __threadfence();
        if (threadIdx.x == 0) st->ticket = 0;
    }
    return last != 0;
}

// The histogram as one block of kBlock threads sees it: eight bins a thread
// and the sums before them.
struct SelPick {
    static constexpr int kPer = kSelBins / kBlock;
    unsigned int hv[kPer];
    unsigned long long before, upto, total;
    // true in the one thread whose bins hold the rem-th value: the bin, the
    // count before it and in it
    __device__ __forceinline__ bool holds(unsigned long long rem, int &bin,
                                          unsigned long long &cum, unsigned int &in_bin) const {
        if (!(before < rem && upto >= rem)) return false;
        cum = before;
        bin = threadIdx.x * kPer;
        in_bin = 0;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            in_bin = hv[u];
            if (cum + hv[u] >= rem) { bin = threadIdx.x * kPer + u; break; }
            cum += hv[u];
        }
        return true;
    }
};
__device__ __forceinline__ SelPick pick_bin(const unsigned int *hist, int nbins) {
    __shared__ unsigned long long part[kBlock];
    SelPick p;
    unsigned long long mine = 0;
#pragma unroll
    for (int u = 0; u < SelPick::kPer; ++u) {
        const int b = threadIdx.x * SelPick::kPer + u;
        p.hv[u] = b < nbins
                      ? __hip_atomic_load(&hist[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
        mine += p.hv[u];
    }
    part[threadIdx.x] = mine;
    __syncthreads();
    // inclusive scan of the per-thread sums (Hillis-Steele)
    for (int off = 1; off < kBlock; off <<= 1) {
        const unsigned long long x = threadIdx.x >= off ? part[threadIdx.x - off] : 0ull;
        __syncthreads();
        part[threadIdx.x] += x;
        __syncthreads();
    }
    p.upto = part[threadIdx.x];
    p.before = p.upto - mine;
    p.total = part[kBlock - 1];
    return p;
}

constexpr int kSelShift = 46;                              // of the first pass
constexpr uint64_t kSelLo = 0x3EB0000000000000ull;         // 2^-20
__device__ __forceinline__ uint64_t sel_key(uint64_t v) {
    return v < kSelLo ? 0ull : v - kSelLo + (1ull << kSelShift);
}
__device__ __forceinline__ uint64_t sel_value(uint64_t key) {
    return key < (1ull << kSelShift) ? 0ull : key - (1ull << kSelShift) + kSelLo;
}

// Histogram of bits [shift, shift + nbits) of the keys of P over cells whose
// bits above shift + nbits equal the state's prefix, then (last block) the bin
// of the remaining-th value.  Pass 0 also settles two cases: fewer finite values than
// wanted (take them all), and a first bin of 0, whose values are exact zeros
// (the snap leaves nothing between 0 and 1e-6).
__global__ __launch_bounds__(kBlock) void k_select_hist(const uint64_t *__restrict__ P,
                                                        int64_t n, int shift, int nbits, int pass,
                                                        int last, int64_t need, int64_t cap,
                                                        SelState *st, unsigned int *hist) {
    if (pass > 0 && st->done) return;
    const uint64_t high = pass > 0 ? st->high : 0ull;
    __shared__ unsigned int h[kSelBins];
    for (int i = threadIdx.x; i < (1 << nbits); i += kBlock) h[i] = 0;
    __syncthreads();
    const int top = shift + nbits;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock) {
        const uint64_t v = P[i];
        if (v >= kInfBits) continue;                       // no value
        const uint64_t u = sel_key(v);
        if (pass > 0 && (u >> top) != high) continue;
        atomicAdd(&h[pass > 0 ? (u >> shift) & ((1ull << nbits) - 1)
                              : min(u >> shift, (uint64_t)(kSelBins - 1))], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < (1 << nbits); i += kBlock)
        if (h[i]) atomicAdd(&hist[i], h[i]);
    if (!last_block(st)) return;

    const SelPick pk = pick_bin(hist, 1 << nbits);
    const int64_t remaining = pass > 0 ? st->remaining : need;
    const unsigned long long rem = (unsigned long long)remaining;
    __syncthreads();                                       // the state is rewritten below
    if (pass == 0 && pk.total < rem) {
        if (threadIdx.x == 0) {              // fewer finite cells than needed: take all
            st->pivot = kInfBits;
            st->need_eq = 0;
            st->nless = 0;
            st->done = 1;
        }
    } else {
        int bin;
        unsigned int in_bin;
        unsigned long long cum;
        if (pk.holds(rem, bin, cum, in_bin)) {             // exactly one thread
            const unsigned long long r2 = rem - cum;       // still wanted within the bin
            const uint64_t hi = (high << nbits) | (uint64_t)bin;
            // cells below the bin: those the earlier passes passed by, and cum
            const int64_t below = need - remaining + (int64_t)cum;
            st->remaining = (int64_t)r2;
            st->high = hi;
            st->below = below;
            st->tie_lo = 0;
            st->tie_hi = n;
            st->pos_limit = 0;
            st->need_eq = 0;
            st->nless = 0;
            st->done = 0;
            if (pass == 0 && bin == 0) {
                st->pivot = 0;
                st->need_eq = (int64_t)r2;
                st->done = 1;
            } else if (last) {
                st->pivot = sel_value(hi);
                st->need_eq = (int64_t)r2;
                st->done = 1;
            } else if (below + (int64_t)in_bin <= cap) {
                st->pivot = sel_value((hi + 1) << shift);  // the whole bin
                st->done = 1;
            }
        }
    }
    for (int i = threadIdx.x; i < kSelBins; i += kBlock) hist[i] = 0;
}

// Ties at the pivot: the first need_eq of them in position order are wanted,
// i.e. those before some position.  Level 0 counts them over 2048 bins of all
// positions, level 1 over bins of the one bin that holds the last wanted tie,
// unless that bin fits the output as it is.
__global__ __launch_bounds__(kBlock) void k_select_ties(const uint64_t *__restrict__ P, int64_t n,
                                                        int64_t cap, SelState *st,
                                                        unsigned int *hist) {
    if (st->need_eq == 0 || st->pos_limit > 0) return;
    const uint64_t pivot = st->pivot;
    const int64_t lo = st->tie_lo, hi = st->tie_hi;
    const int64_t width = (hi - lo + kSelBins - 1) / kSelBins;
    __shared__ unsigned int h[kSelBins];
    for (int i = threadIdx.x; i < kSelBins; i += kBlock) h[i] = 0;
    __syncthreads();
    for (int64_t i = lo + (int64_t)blockIdx.x * kBlock + threadIdx.x; i < hi;
         i += (int64_t)gridDim.x * kBlock)
        if (P[i] == pivot) atomicAdd(&h[(i - lo) / width], 1u);
    __syncthreads();
    for (int i = threadIdx.x; i < kSelBins; i += kBlock)
        if (h[i]) atomicAdd(&hist[i], h[i]);
    if (!last_block(st)) return;
    const SelPick pk = pick_bin(hist, kSelBins);
    const int64_t need_eq = st->need_eq, below = st->below;
    __syncthreads();
    int bin;
    unsigned int in_bin;
    unsigned long long cum;
    if (pk.holds((unsigned long long)need_eq, bin, cum, in_bin)) {
        const int64_t b0 = lo + bin * width, b1 = min(b0 + width, n);
        if (below + (int64_t)cum + (int64_t)in_bin <= cap) {
            st->pos_limit = b1;
        } else {
            st->tie_lo = b0;
            st->tie_hi = b1;
            st->below = below + (int64_t)cum;
            st->need_eq = need_eq - (int64_t)cum;
        }
    }
    for (int i = threadIdx.x; i < kSelBins; i += kBlock) hist[i] = 0;
}

// The selected cells: those below the pivot and the ties before the position
// limit (any order, one reservation per block).
constexpr int kSelTile = kBlock * 16;

__global__ __launch_bounds__(kBlock) void k_select_emit(const uint64_t *__restrict__ P, int64_t n,
                                                        const uint32_t *__restrict__ cell,
                                                        LenView lv, Select out) {
    __shared__ uint32_t found[kSelTile];
    __shared__ uint32_t nfound, at;
    SelState *st = out.st;
    const uint64_t pivot = st->pivot;
    const int64_t limit = st->need_eq > 0 ? st->pos_limit : 0;
    const int64_t base = (int64_t)blockIdx.x * kSelTile;
    if (pivot == 0 && base >= limit) return;               // nothing lies below 0
    if (threadIdx.x == 0) nfound = 0;
    __syncthreads();
    uint64_t v[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int64_t i = base + (int64_t)r * kBlock + threadIdx.x;
        v[r] = i < n ? P[i] : kInfBits;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int64_t i = base + (int64_t)r * kBlock + threadIdx.x;
        if (v[r] < kInfBits && (v[r] < pivot || (v[r] == pivot && i < limit)))
            found[atomicAdd(&nfound, 1u)] = (uint32_t)(r * kBlock + threadIdx.x);
    }
    __syncthreads();
    const uint32_t nf = nfound;
    if (nf == 0) return;
    if (threadIdx.x == 0) at = atomicAdd(&st->nless, nf);
    __syncthreads();
    for (uint32_t x = threadIdx.x; x < nf; x += kBlock) {
        const uint32_t p = at + x;
        if ((int64_t)p < out.cap) {
            const int64_t i = base + found[x];
            const uint32_t c = cell[i];
            const int l = lv.find((int64_t)c);
            out.sel[p] = (uint32_t)i;
            out.sel_val[p] = P[i];
            out.sel_cell[p] = c;
            out.sel_len[p] = make_int2(l, lv.m(l));
        }
    }
}

// The greedy of Sec. 2 over the selected cells (one block): up to k times the
// smallest (value, position) still in is accepted and every cell of its length
// within m/2 of it goes.  Positions follow the (length, start) order.  k = 0:
// the host runs the greedy (more than one block's registers hold).  The join's
// counts (when given) travel with the state, which the host reads.
constexpr int kGreedyThreads = 1024;

// Smallest value over the wavefront, in every lane (all 64 lanes active), by
// shifts within rows of 16 and row broadcasts.
template <int kCtrl, int kRows>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, kCtrl, kRows, 0xF, false);
}
template <int kCtrl, int kRows>
__device__ __forceinline__ void min_step(uint32_t &v) {
    v = min(v, dpp_u32<kCtrl, kRows>(v));
}
template <int kCtrl, int kRows>
__device__ __forceinline__ void min_step(unsigned long long &v) {
    const unsigned long long o =
        (unsigned long long)dpp_u32<kCtrl, kRows>((uint32_t)(v >> 32)) << 32 |
        dpp_u32<kCtrl, kRows>((uint32_t)v);
    v = o < v ? o : v;
}
// kRows: only over each row of 16 lanes (the result in its last lane).
template <bool kRows, typename T>
__device__ __forceinline__ void wave_min_steps(T &v) {
    min_step<0x111, 0xF>(v);
    min_step<0x112, 0xF>(v);
    min_step<0x114, 0xF>(v);
    min_step<0x118, 0xF>(v);
    if (kRows) return;
    min_step<0x142, 0xA>(v);
    min_step<0x143, 0xC>(v);
}
template <bool kRows>
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
    wave_min_steps<kRows>(v);
    return (uint32_t)__builtin_amdgcn_readlane((int)v, kRows ? 15 : 63);
}
template <bool kRows>
__device__ __forceinline__ unsigned long long wave_min_u64(unsigned long long v) {
    wave_min_steps<kRows>(v);
    constexpr int kLast = kRows ? 15 : 63;
    return (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), kLast) << 32 |
           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, kLast);
}

constexpr int kGreedyPer = kGreedyMax / kGreedyThreads;

__global__ __launch_bounds__(kGreedyThreads) void k_select_greedy(
    Select in, int k, SelCell *__restrict__ acc, const unsigned long long *__restrict__ counts) {
    // the smallest entry of each wavefront, in two sets used in turn
    struct Best {
        unsigned long long v;
        uint32_t p, c;
        int lm;
    };
    constexpr int kWaves = kGreedyThreads / kWave;
    static_assert(kWaves == 16, "a row of lanes takes the wavefronts' entries");
    __shared__ Best wbest[2][kWaves], own[kWaves];
    __shared__ unsigned long long kept;
    const int tid = threadIdx.x, lane = lane_id(), w = tid / kWave;
    SelState *st = in.st;
    if (tid == 0) kept = 0;
    __syncthreads();
    if (counts && tid < kCtrSlots) atomicAdd(&kept, counts[tid * kCtrStride]);
    __syncthreads();
    const int64_t nl = (int64_t)st->nless < in.cap ? (int64_t)st->nless : in.cap;
    if (tid == 0) {
        st->kept = kept;
        st->nredo = counts ? (uint32_t)counts[kCtrSlots * kCtrStride] : 0u;
        st->naccept = 0;
        st->improved = in.improved ? *in.improved : 0ull;
    }
    if (k == 0) return;
    // every entry with its cell and length, in registers
    unsigned long long v[kGreedyPer];
    uint32_t p[kGreedyPer], c[kGreedyPer];
    int lm[kGreedyPer];                                    // length index << 12 | window length
    static_assert(kMaxM < 4096, "a window length fits 12 bits");
    const int nu = (int)((nl + kGreedyThreads - 1) / kGreedyThreads);     // entries per thread
#pragma unroll
    for (int u = 0; u < kGreedyPer; ++u) {
        const int64_t x = (int64_t)u * kGreedyThreads + tid;
        v[u] = ~0ull;                                      // none
        p[u] = kNone;
        c[u] = 0;
        lm[u] = -1;
        if (x < nl) {
            v[u] = in.sel_val[x];
            p[u] = in.sel[x];
            c[u] = in.sel_cell[x];
            const int2 y = in.sel_len[x];
            lm[u] = y.x << 12 | y.y;
        }
    }
    // the wavefront's smallest entry, kept until an entry of it goes
    unsigned long long ov = ~0ull;
    uint32_t op = kNone, oc = 0u;
    int ol = -1;
    bool stale = true;
    int r = 0;
    for (; r < k; ++r) {
        if (stale) {                                       // (uniform in the wavefront)
            unsigned long long bv = ~0ull;
            uint32_t bp = kNone;
#pragma unroll
            for (int u = 0; u < kGreedyPer; ++u)
                if (u < nu && (v[u] < bv || (v[u] == bv && p[u] < bp))) {
                    bv = v[u];
                    bp = p[u];
                }
            const unsigned long long mv = wave_min_u64<false>(bv);
            const uint32_t mp = wave_min_u32<false>(bv == mv ? bp : kNone);
            if (lane == 0) own[w] = Best{~0ull, kNone, 0u, -1};
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int u = 0; u < kGreedyPer; ++u)
                if (u < nu && mp != kNone && p[u] == mp) own[w] = Best{mv, mp, c[u], lm[u]};
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            ov = own[w].v;
            op = own[w].p;
            oc = own[w].c;
            ol = own[w].lm;
        }
        if (lane == 0) wbest[r & 1][w] = Best{ov, op, oc, ol};
        __syncthreads();
        const Best &x = wbest[r & 1][lane & (kWaves - 1)];
        const unsigned long long xv = x.v;
        const uint32_t xp = x.p, xc = x.c;
        const int xl = x.lm;
        const unsigned long long bv = wave_min_u64<true>(xv);
        const uint32_t bp = wave_min_u32<true>(xv == bv ? xp : kNone);
        if (bp == kNone) break;                            // (uniform) nothing is left
        const int src = __ffsll((unsigned long long)__ballot(xp == bp)) - 1;
        const uint32_t bc = (uint32_t)__builtin_amdgcn_readlane((int)xc, src);
        const int bl = __builtin_amdgcn_readlane(xl, src), bm = bl & 0xFFF;
        if (tid == 0) acc[r] = SelCell{bv, bp, bc};
        bool gone = false;
#pragma unroll
        for (int u = 0; u < kGreedyPer; ++u) {
            const int64_t d = (int64_t)c[u] - (int64_t)bc;
            if (u < nu && lm[u] == bl && 2 * (d < 0 ? -d : d) <= bm) {
                v[u] = ~0ull;
                p[u] = kNone;
                lm[u] = -1;
                gone = true;
            }
        }
        stale = __ballot(gone) != 0ull;
    }
    if (tid == 0) st->naccept = r;
}

// ------------------------------------------------------------------ rows

// One pass over each requested row c: out_min[c] = min over valid j of the
// snapped distance where that lies at or below req[c].target, else +inf or a
// value above it (the certificate's check), and out_arg[c] = smallest valid j
// whose snapped distance equals req[c].target (the reported neighbour when the
// check holds).  Constant windows are not indexed and never scanned.  A sum
// past the target stops.  At most 128 blocks a row, and one pair of atomics a
// block: with one per wavefront, 20 rows queued 300,000 atomics
// on 20 addresses and took 926 us for 981,000 windows a row, 512 now.
// Each lane takes every (threads)-th window of the length and evaluates the
// canonical distance on its own (lane_zdist): neighbouring lanes read
// neighbouring windows, and the row's own window is shared by all.
__global__ __launch_bounds__(kBlock) void k_rows(Req q, const RowReq *__restrict__ rr,
                                                 unsigned long long *__restrict__ out_min,
                                                 unsigned long long *__restrict__ out_arg) {
    const RowReq R = rr[blockIdx.y];
    const LenInfo L = q.len[R.l];
    const int m = L.m;
    const int64_t i = (int64_t)q.cell[R.k] - L.cell_base;
    const double mui = q.mu[R.k], isi = q.isig[R.k];
    const int64_t nt = (int64_t)gridDim.x * kBlock;
    unsigned long long best = (unsigned long long)kInfBits, arg = ~0ull;
    // (well above the target: only values above it stop early)
    const double lim2 = exit_bound(fmax(bitsd(R.target), kEps0) * (1.0 + 1e-9));
    for (int64_t x = (int64_t)blockIdx.x * kBlock + threadIdx.x; x < L.n_index; x += nt) {
        const int64_t kc = L.kbase + x;
        const int64_t j = (int64_t)q.cell[kc] - L.cell_base;
        const int64_t gap = j > i ? j - i : i - j;
        if (gap < q.excl) continue;
        const double dd = snap(lane_zdist(q.t, i, mui, isi, j, q.mu[kc], q.isig[kc], m, lim2));
        const unsigned long long b = (unsigned long long)dbits(dd);
        best = b < best ? b : best;
        if (b == R.target && (unsigned long long)j < arg) arg = (unsigned long long)j;
    }
    for (int off = 1; off < kWave; off <<= 1) {
        const unsigned long long o = __shfl_xor(best, off, kWave);
        const unsigned long long a = __shfl_xor(arg, off, kWave);
        best = o < best ? o : best;
        arg = a < arg ? a : arg;
    }
    __shared__ unsigned long long wb[kBlock / kWave], wa[kBlock / kWave];
    if (lane_id() == 0) {
        wb[threadIdx.x / kWave] = best;
        wa[threadIdx.x / kWave] = arg;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int v = 1; v < kBlock / kWave; ++v) {
            best = wb[v] < best ? wb[v] : best;
            arg = wa[v] < arg ? wa[v] : arg;
        }
        atomicMin(&out_min[blockIdx.y], best);
        if (arg != ~0ull) atomicMin(&out_arg[blockIdx.y], arg);
    }
}

__global__ __launch_bounds__(kBlock) void k_fill_u64(uint64_t *__restrict__ p, int64_t n,
                                                     uint64_t v) {
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock)
        p[i] = v;
}

// The number of the n values of P that are 0 (the FP64 bits of +0),
// added to *out.
__global__ __launch_bounds__(kBlock) void k_count_zero(const uint64_t *__restrict__ P, int64_t n,
                                                       unsigned long long *__restrict__ out) {
    unsigned long long c = 0;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock)
        c += P[i] == 0ull;
    __shared__ unsigned long long wc[kBlock / kWave];
    for (int off = kWave / 2; off > 0; off >>= 1) c += __shfl_xor(c, off, kWave);
    if (lane_id() == 0) wc[threadIdx.x / kWave] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        c = 0;
        for (int k = 0; k < kBlock / kWave; ++k) c += wc[k];
        if (c) atomicAdd(out, c);
    }
}

__global__ __launch_bounds__(kBlock) void k_fill_u32(uint32_t *__restrict__ p, int64_t n,
                                                     uint32_t v) {
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock)
        p[i] = v;
}

// ------------------------------------------------------------ launchers

static inline unsigned nblk(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }
static inline unsigned gridcap(int64_t n, int64_t cap) {
    int64_t b = (n + kBlock - 1) / kBlock;
    if (b < 1) b = 1;
    return (unsigned)(b < cap ? b : cap);
}

void launch_select(const Select &x, const uint64_t *P, int64_t n, const uint32_t *cell,
                   const LenView &lv, const unsigned long long *counts, hipStream_t s) {
    static const int shifts[6] = {kSelShift, 35, 24, 13, 2, 0};
    static const int widths[6] = {11, 11, 11, 11, 11, 2};
    if (n <= 0) return;
    // (each block ends with a fence and a ticket: eight turns a thread at
    // least, and no more blocks than fill the chip)
    const unsigned nb = gridcap((n + 7) / 8, 1024);
    for (int ps = 0; ps < 6; ++ps)
        hipLaunchKernelGGL(k_select_hist, dim3(nb), dim3(kBlock), 0, s, P, n, shifts[ps], widths[ps],
                           ps, ps == 5 ? 1 : 0, x.need, x.cap, x.st, x.hist);
    for (int level = 0; level < 2; ++level)
        hipLaunchKernelGGL(k_select_ties, dim3(level && nb > 32 ? 32u : nb), dim3(kBlock), 0, s,
                           P, n, x.cap, x.st, x.hist);
    hipLaunchKernelGGL(k_select_emit, dim3((unsigned)((n + kSelTile - 1) / kSelTile)), dim3(kBlock),
                       0, s, P, n, cell, lv, x);
    hipLaunchKernelGGL(k_select_greedy, dim3(1), dim3(kGreedyThreads), 0, s, x,
                       x.on_device() ? x.k : 0, x.acc, counts);
}

void launch_rows(const Req &q, const RowReq *rr, int nrows, int64_t maxN,
                 unsigned long long *out_min, unsigned long long *out_arg, hipStream_t s) {
    if (nrows <= 0) return;
    hipLaunchKernelGGL(k_rows, dim3(gridcap(maxN, 128), (unsigned)nrows), dim3(kBlock), 0, s,
                       q, rr, out_min, out_arg);
}

void launch_count_zero(const uint64_t *P, int64_t n, unsigned long long *out, hipStream_t s) {
    if (n > 0)
        hipLaunchKernelGGL(k_count_zero, dim3(gridcap(n, 512)), dim3(kBlock), 0, s, P, n, out);
}

void launch_fill_u64(uint64_t *p, int64_t n, uint64_t v, hipStream_t s) {
    if (n > 0)
        hipLaunchKernelGGL(k_fill_u64, dim3(gridcap(n, 8192)), dim3(kBlock), 0, s, p, n, v);
}

void launch_fill_u32(uint32_t *p, int64_t n, uint32_t v, hipStream_t s) {
    if (n > 0)
        hipLaunchKernelGGL(k_fill_u32, dim3(gridcap(n, 8192)), dim3(kBlock), 0, s, p, n, v);
}

}  // namespace pmp
