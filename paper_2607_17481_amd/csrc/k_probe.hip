// k_probe.hip -- streaming candidate generation, Parseval prune and exact
// verification (paper Sec. 3.4, Algorithm 1 phase B).
//
// Every indexed window q is a query.  Its candidates are the windows stored
// in its own bucket (the d-bit signature prefix) and then in the Hamming-1
// buckets of its `probes` lowest-margin prefix bits, in increasing margin
// order.  As in the stream, a query only sees earlier windows, and only valid
// ones (i <= q - excl); each bucket is sorted by start, so those form a prefix
// of the bucket.  Inspections are capped at R = gamma * alpha per query; when
// a bucket holds more valid entries than the remaining budget, half of it goes
// to the most recent entries and half to entries at even intervals over the
// rest of the bucket.
//
// A candidate c is evaluated exactly only if its certified Parseval bound is
// below max(P[q], P[c]) -- the two cells the pair can lower (Sec. 3.4, the
// definition of S_stream).  Each exact distance lowers both cells through a
// 64-bit atomic min on the FP64 bit pattern (non-negative doubles order like
// their bit patterns), which is order independent.  Which candidates pass the
// prune depends on how far the cells have been lowered when they are
// inspected, so the upper profile may differ slightly between runs; the exact
// top-k built on it by the certificate does not (the role of the fixed merge
// order of Prop. 5).
//
// GPU mapping: a team of 8 to 64 lanes per query, the more the fewer queries a
// launch has (launch_probe gives the thresholds).  Every group of eight lanes
// of a team inspects eight candidates at a time, one per lane; their records
// are read by the eight lanes together (one contiguous row per load) and the
// eight bounds summed by a transposed reduction.  The survivors are verified
// smallest bound first, each result tightening the prune of the rest; queries
// without survivors search on meanwhile.
//
// One departure from the paper: a query stops once its own cell reaches 0
// (the smallest possible value); the remaining candidates could only lower
// their own cells, which their own queries, or the certificate, cover.
#include "pmp_dev.h"
#include "quant.h"

namespace pmp {

// The query windows of a wavefront, staged in LDS when they lie within a
// short span of the series (dynamic size: kQwinExtra + the longest window, in
// doubles).  The staged samples are the series' own, so a distance read
// through them has the same bits.
extern __shared__ double probe_qwin[];
constexpr int kQwinExtra = 128;
struct QwinA {
    int64_t base;
    __device__ __forceinline__ double operator()(int64_t x) const { return probe_qwin[x - base]; }
};

// Queries are taken in (length, start) order (indexed position k), so that
// neighbouring windows, which tend to cost alike, share a wavefront; only the
// anchor lengths are probed (Sec. 3.3), each from its first probe block, so a
// wavefront never spans two lengths.  A block is one wavefront: wavefront
// times vary over two orders of magnitude, and a single-wave block lets a
// compute unit start new work as soon as any one wavefront ends.  Whenever a
// verification lowers a cell, the partner's start is recorded as the cell's
// hint (any partner that lowered it will do: the hints only propose pairs at
// the lengths between anchors).
//
// What bounds it: the chain of dependent loads of a query (bucket, slot, cell
// value, record, moments, samples) where few queries are in flight, the record
// and sample reads where many are.  With one lane per query a wavefront waited
// for the slowest of 64 chains of up to R candidates; eight lanes shorten a
// chain eightfold and give eight times the wavefronts.  Measured: random walk
// 4,000 x 51 (19,700 queries) 3.0 -> 0.63 ms, Wafer-like 40,000 x 41 of 480..520
// 5.4 -> 1.2 ms, Wafer-like 5M (981,000 queries) 1.69 -> 0.77 ms, ECG-like 1M
// (5.0e6 queries, FP64) 65 -> 53 ms.
//
// kCut: only pairs at or below `cut` are of interest (the caller holds a k-th
// value that cells above it cannot undercut).  The bound and the 16-bit
// prefilter then test every pair against the smaller of the cut and the two
// cells, so that nearly all pairs of noisy windows end without a distance:
// at ECG-like 1M the four anchors after the first take 9.5 ms instead of 44.
//
// kTeam: lanes per query.  Eight are enough while the queries fill the chip;
// with fewer, a query takes up to the whole wavefront: its lanes look at that
// many candidates at once and every eight of them verify their own survivor.
// (A survivor verified beside another that would have ruled it out is work for
// nothing, about 5 % of the verifications, on lanes that were idle.)
template <typename FT, bool kCut, int kTeam>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(4)))
void k_probe(Req q, const uint32_t *__restrict__ bstart, int qcap, int64_t blk0, double cut,
             Quant x, ProbeIf go) {
    if (go.zeros && *go.zeros >= go.limit) return;           // (uniform)
    // the anchor length of this block (blocks [blk0, blk0 + gridDim.x) of
    // the probe): the last length whose first probe block is at or below it
    // (uniform)
    constexpr int kSplit = kTeam / kGroup;       // wavefronts per probe block of kProbeQ queries
    const int64_t gb = blk0 + (int64_t)blockIdx.x / kSplit;
    int l = 0;
    {
        int hi = q.L - 1;
        while (l < hi) {
            const int mid = (l + hi + 1) >> 1;
            if (q.len[mid].pblk_base <= gb) l = mid; else hi = mid - 1;
        }
    }
    const LenInfo &L = q.len[l];
    const int m = L.m, d = L.depth, probes = L.probes;
    const int64_t cell_base = L.cell_base;
    const uint32_t *const bb = bstart + L.bucket_base;
    const float sqrt2m = (float)sqrt(2.0 / (double)m) * (1.0f + 1e-7f);
    const FT *const F = (const FT *)q.F;
    const int g = threadIdx.x & (kGroup - 1), grp = threadIdx.x / kGroup;
    const int tl = threadIdx.x & (kTeam - 1);    // lane in the team
    const int64_t kend = L.kbase + L.n_index;
    const int64_t k0 = L.kbase + (gb - L.pblk_base) * kProbeQ +
                       (int64_t)(blockIdx.x % kSplit) * (kWave / kTeam);
    if (k0 >= kend) return;
    const int64_t k = k0 + threadIdx.x / kTeam;
    uint32_t n_cand = 0, n_ver = 0;

    // ---- the team's query (every lane of a team holds the same state)
    bool done = k >= kend;
    uint32_t prefix = 0, lim = 0;
    int64_t iq = 0;
    uint64_t kw = 0;
    double Pq = 0.0, muq = 0.0, isq = 0.0;
    RecPart<FT> fq = {};
    FT eq = 0;
    float4 wq = make_float4(0.0f, 0.0f, 0.0f, 0.0f), wc = wq;   // prefilter: query, candidate
    const bool mine = !done;
    if (mine) {
        iq = (int64_t)q.cell[k] - cell_base;
        kw = q.keyw[k];
        prefix = d ? (uint32_t)(kw & 0xFFFFFFu) >> (q.B - d) : 0u;
        Pq = bitsd(q.P[k]);
        muq = q.mu[k];
        isq = q.isig[k];
        fq = load_part(F + k * kRec, g);
        eq = F[k * kRec + kSlotErr];
        if (kCut) wq = x.xw[k];
        done = Pq == 0.0 || iq - q.excl < 0;
        lim = (uint32_t)(cell_base + iq - q.excl);
    }
    // ---- stage the query windows (uniform decision): the span from the first
    // start to the last window's end fits
    bool staged;
    const int64_t qlo = __shfl(iq, 0, kWave);
    {
        const int last = 63 - __clzll((long long)__ballot(mine));
        const int64_t span = __shfl(iq, last, kWave) + m - qlo;
        staged = span <= (int64_t)qcap;
        if (staged) {
            for (int64_t x = lane_id(); x < span; x += kWave) probe_qwin[x] = q.t[qlo + x];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    }
    // candidate iterator of the query
    int pr = -1, budget = q.budget_R;
    int64_t bs = 0, vend = 0, span = 0;
    int take = 0, rec = 0, str = 1, j = 0;
    // this lane's candidate, while it waits for its verification
    bool alive = false;
    uint32_t kc = 0;
    int64_t ic = 0;
    double Pc = 0.0, muc = 0.0, isc = 0.0;
    float lb = 0.0f;

    const int gshift = grp * kGroup;
    auto group_bits = [&](bool b) -> uint32_t { return (uint32_t)(__ballot(b) >> gshift) & 0xFFu; };
    auto team_bits = [&](bool b) -> uint64_t {
        const uint64_t x = __ballot(b);
        return kTeam == kWave ? x
                              : (x >> (threadIdx.x & ~(kTeam - 1))) & ((1ull << (kTeam & 63)) - 1ull);
    };
    for (;;) {
        // ---- every query still at work searches until it has a survivor
        for (;;) {
            const bool search = !done && team_bits(alive) == 0ull;
            if (__ballot(search) == 0) break;
            if (!search) continue;
            if (j >= take) {
                // open the next bucket
                ++pr;
                if (pr > probes || budget <= 0) { done = true; continue; }
                uint32_t b = prefix;
                if (pr > 0) {
                    const int bit = (int)((kw >> (24 + 5 * (pr - 1))) & 31u);
                    b = prefix ^ (1u << (d - 1 - bit));
                }
                bs = bb[b];
                // the valid entries (cell <= lim) form a prefix of the bucket
                // (in the own bucket the query and everything after it lie
                // past the prefix); the team narrows it down kTeam ways
                int64_t lo = bs, hi = (int64_t)bb[b + 1];
                while (lo < hi) {
                    const int64_t step = (hi - lo + kTeam - 1) / kTeam;
                    const int64_t at = lo + tl * step;
                    const int below = __popcll(team_bits(at < hi && q.pcell[at] <= lim));
                    if (below == 0) break;
                    hi = min(hi, lo + below * step);
                    lo += (below - 1) * step + 1;
                }
                vend = lo;
                const int64_t cnt = vend - bs;
                j = 0;
                if (cnt <= 0) { take = 0; continue; }
                if (cnt <= budget) {
                    take = (int)cnt; rec = take; span = 0;
                } else {
                    take = budget; rec = budget - budget / 2; span = cnt - rec;
                }
                str = take - rec > 0 ? take - rec : 1;
                budget -= take;
                continue;
            }
            // the next candidates, one per lane; a single one while the
            // query's own cell has no value (its first distance often ends
            // the query: a repeat at 0), and no bound can prune below +inf
            const bool first = !kCut && Pq == INFINITY;
            const int jj = j + tl;
            const bool in = jj < take && (!first || tl == 0);
            j += first ? 1 : kTeam;
            double thr = 0.0;
            if (in) {
                const int64_t cs = jj < rec ? vend - 1 - jj : bs + ((int64_t)(jj - rec) * span) / str;
                kc = q.perm[cs];
                ic = (int64_t)q.pcell[cs] - cell_base;
                Pc = bitsd(q.P[kc]);
                thr = fmax(Pq, Pc);
                if (kCut) thr = fmin(thr, cut);
                ++n_cand;
            }
            alive = thr > 0.0;
            lb = 0.0f;
            if (!first) {
                const uint32_t m8 = group_bits(alive);
                if (m8) {
                    lb = group_lb<FT>(F, fq, eq, kc, alive, m8, g, sqrt2m);
                    alive = alive && (double)lb < thr;
                }
            }
            if (alive && kCut) {
                wc = x.xw[kc];
            } else if (alive) {
                muc = q.mu[kc];
                isc = q.isig[kc];
            }
        }
        if (__ballot(alive) == 0) break;
        // ---- every group of eight lanes verifies its survivor of the smallest bound
        const bool go = group_bits(alive) != 0u;
        uint32_t key = alive ? (__float_as_uint(lb) & ~7u) | (uint32_t)g : 0xFFFFFFFFu;
        key = min(key, xor_lane<1>(key));
        key = min(key, xor_lane<2>(key));
        key = min(key, xor_lane<4>(key));
        const int sel = (int)(key & 7u);
        const uint32_t vk = (uint32_t)__shfl((int)kc, sel, kGroup);
        const int64_t vi = __shfl(ic, sel, kGroup);
        const double vP = __shfl(Pc, sel, kGroup);
        double vmu = 0.0, vis = 0.0, thr = fmax(Pq, vP);
        bool exact = go;
        if (kCut) {
            thr = fmin(thr, cut);
            const float4 wv = make_float4(__shfl(wc.x, sel, kGroup), __shfl(wc.y, sel, kGroup),
                                          __shfl(wc.z, sel, kGroup), __shfl(wc.w, sel, kGroup));
            float qlim;
            if (go && quant_limit(wq, wv, m, thr, qlim))
                exact = quant_below<8>(x.x16, x.pitch, (uint32_t)iq, (uint32_t)vi, wq.y, wv.y,
                                       wq.z - wv.z, m, qlim, g);
            if (exact) {
                vmu = q.mu[vk];
                vis = q.isig[vk];
            }
        } else {
            vmu = __shfl(muc, sel, kGroup);
            vis = __shfl(isc, sel, kGroup);
        }
        const double lim2 = exit_bound(thr);
        const int vm = exact ? m : 0;
        double dd = INFINITY;
        if (!kCut || __ballot(exact))
            dd = snap(staged
                ? group_zdist_a(QwinA{qlo}, q.t, iq, muq, isq, vi, vmu, vis, vm, lim2)
                : group_zdist_a(SeriesA{q.t}, q.t, iq, muq, isq, vi, vmu, vis, vm, lim2));
        if (!exact) dd = INFINITY;
        double best = dd;                                  // the team's smallest
#pragma unroll
        for (int off = kGroup; off < kTeam; off <<= 1) best = fmin(best, __shfl_xor(best, off, kWave));
        {
            const unsigned long long db = (unsigned long long)dbits(dd);
            if (g == 0 && exact) {
                ++n_ver;
                if (dd < Pq && dd == best) {
                    atomicMin((unsigned long long *)&q.P[k], db);
                    q.hint[k] = (uint32_t)vi;
                }
                if (dd < vP) {
                    atomicMin((unsigned long long *)&q.P[vk], db);
                    q.hint[vk] = (uint32_t)iq;
                }
            }
            Pq = fmin(Pq, best);
            if (Pq == 0.0) done = true;
            if (g == sel || done || (double)lb >= fmax(Pq, Pc)) alive = false;
        }
    }
    // stats: one atomic per wave
    unsigned long long a = n_cand, v = n_ver;
    for (int off = kWave / 2; off > 0; off >>= 1) {
        a += __shfl_xor(a, off, kWave);
        v += __shfl_xor(v, off, kWave);
    }
    if (lane_id() == 0) {
        if (a) count_add(q.counters, C_PASS_CAND, a);
        if (v) count_add(q.counters, C_PASS_VER, v);
    }
}

// Buckets holding more than R entries (hot classes, Sec. 3.6) -- statistics.
__global__ __launch_bounds__(kBlock) void k_hot_buckets(const uint32_t *__restrict__ bstart,
                                                        int64_t nb, int R,
                                                        unsigned long long *__restrict__ cnt) {
    int64_t b = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    unsigned long long h = 0;
    if (b < nb) h = (bstart[b + 1] - bstart[b]) > (uint32_t)R;
    for (int off = kWave / 2; off > 0; off >>= 1) h += __shfl_xor(h, off, kWave);
    if (lane_id() == 0 && h) atomicAdd(cnt, h);
}

static inline unsigned nblk(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

// Lanes per query by the launch's blocks of eight queries.  Measured in whole
// requests, fewer lanes against more at the same size: random walk 4,000 (500
// blocks, then 1,500 of the other anchors) 249 us at 8 lanes, 87 at 64, and 1.71
// ms against 1.60 with 32 lanes for the others, 1.70 with 64; ECG-like 50,000
// at 24..67 (6,250 blocks) 3.83 -> 3.60 ms with 16 lanes; Wafer-like 5M (123,000
// blocks) 6.06 ms with 8 lanes, 6.45 with 16: queries that fill the chip only
// add the verifications that another would have spared.
constexpr int64_t kTeam64 = 1024, kTeam32 = 4096, kTeam16 = 65536;

// A launch has fewer than 2^32 work-items (blocks times threads), and a block of
// eight queries has 64 at least: 2^29 queries and more take several launches.
// Pieces of 2^20 blocks keep every launch far below that and still fill the
// chip a hundred times over.
constexpr int64_t kProbePiece = (int64_t)1 << 20;
static_assert(kTeam16 <= kProbePiece, "the larger teams take one launch");
static_assert(kProbePiece * kWave < (int64_t)1 << 32, "work-items of a launch");

template <typename FT, int kTeam>
static void launch_probe_team(const Req &q, const uint32_t *bstart, int64_t blk0, int64_t nblocks,
                              int qcap, const Quant &x, const ProbeIf &go, hipStream_t s) {
    hipLaunchKernelGGL((k_probe<FT, false, kTeam>), dim3((unsigned)(nblocks * (kTeam / kGroup))),
                       dim3(kWave), (size_t)qcap * sizeof(double), s, q, bstart, qcap, blk0,
                       INFINITY, x, go);
}
template <typename FT>
static void launch_probe_ft(const Req &q, const uint32_t *bstart, int64_t blk0, int64_t nblocks,
                            int qcap, double cut, const Quant &x, const ProbeIf &go, hipStream_t s) {
    if (!x.x16 && nblocks <= kTeam64)
        launch_probe_team<FT, 64>(q, bstart, blk0, nblocks, qcap, x, go, s);
    else if (!x.x16 && nblocks <= kTeam32)
        launch_probe_team<FT, 32>(q, bstart, blk0, nblocks, qcap, x, go, s);
    else if (!x.x16 && nblocks <= kTeam16)
        launch_probe_team<FT, 16>(q, bstart, blk0, nblocks, qcap, x, go, s);
    else
        for (int64_t at = 0; at < nblocks; at += kProbePiece) {
            const int64_t n = nblocks - at < kProbePiece ? nblocks - at : kProbePiece;
            if (x.x16)            // (over 2^20 windows: the queries fill the chip)
                hipLaunchKernelGGL((k_probe<FT, true, kGroup>), dim3((unsigned)n), dim3(kWave),
                                   (size_t)qcap * sizeof(double), s, q, bstart, qcap, blk0 + at,
                                   cut, x, go);
            else
                launch_probe_team<FT, 8>(q, bstart, blk0 + at, n, qcap, x, go, s);
        }
}

void launch_probe(int precision, const Req &q, const uint32_t *bstart, int64_t blk0,
                  int64_t nblocks, int max_m, double cut, const Quant &x, const ProbeIf &go,
                  hipStream_t s) {
    if (nblocks <= 0) return;
    const int qcap = kQwinExtra + max_m;
    if (precision == 0) launch_probe_ft<double>(q, bstart, blk0, nblocks, qcap, cut, x, go, s);
    else launch_probe_ft<float>(q, bstart, blk0, nblocks, qcap, cut, x, go, s);
}

int64_t probe_work_items(int64_t nblocks) {
    const int64_t n = nblocks < kProbePiece ? nblocks : kProbePiece;
    const int team = nblocks <= kTeam64 ? 64 : nblocks <= kTeam32 ? 32 : nblocks <= kTeam16 ? 16 : 8;
    return n * (team / kGroup) * kWave;
}

void launch_hot_buckets(const uint32_t *bstart, int64_t nb, int R, unsigned long long *cnt,
                        hipStream_t s) {
    if (nb > 0)
        hipLaunchKernelGGL(k_hot_buckets, dim3(nblk(nb)), dim3(kBlock), 0, s, bstart, nb, R, cnt);
}

}  // namespace pmp
