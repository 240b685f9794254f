// k_stream.hip -- the stream update (Sec. 3.1, 3.5, Algorithm 1) on the GPU.
//
// Samples arrive in batches of beta <= excl consecutive samples.  At every
// anchor length a batch completes up to beta windows (the windows ending at
// its samples, Sec. 3.1); no two of them form a valid pair, so they never
// search each other (Sec. 3.5).  One batch is:
//   windows  one wavefront per completed non-constant window: moments,
//            normalized spectral features F (Sec. 3.2) by a direct FP64 DFT
//            against a per-anchor basis table, their error bound, SimHash
//            key and projection margins (Sec. 3.4);
//   probe    one block per completed window: its exact-prefix bucket and
//            the h Hamming-1 buckets of its smallest-margin prefix bits, at
//            most R candidates (the rest of the budget spent half on a
//            bucket's most recent entries, half at even intervals over it),
//            the Parseval prune against max(best_q, P[c]) (Lemma 2), exact
//            FP64 distances of the survivors; the query's own best is
//            written, the candidates' improvements are buffered;
//   finish   one block merges the buffered improvements into the profile;
//            equal distances resolve to the smallest query start, so the
//            result does not depend on the order the searches ran in
//            (Prop. 5); one block per anchor makes the batch's windows a new
//            sorted run of its directory and merges the newest runs as a
//            binary counter (large merges in launches of their own).
// The directory of an anchor is its indexed windows in arrival order, cut
// into runs sorted by (key, start).  A bucket at depth d is the d-bit key
// prefix, so it is one contiguous range of every run, found by binary
// search: when the population passes alpha 2^d the depth grows (Prop. 4)
// and nothing is rehomed.
#include "pmp_dev.h"

namespace pmp {

namespace {

// First position in keys[lo, hi) with key >= v.
__device__ __forceinline__ uint32_t lower_bound_u32(const uint32_t *__restrict__ keys,
                                                    uint32_t lo, uint32_t hi, uint32_t v) {
    while (lo < hi) {
        const uint32_t mid = lo + ((hi - lo) >> 1);
        if (keys[mid] < v) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// First position in keys[lo, hi) with key > v.
__device__ __forceinline__ uint32_t upper_bound_u32(const uint32_t *__restrict__ keys,
                                                    uint32_t lo, uint32_t hi, uint32_t v) {
    while (lo < hi) {
        const uint32_t mid = lo + ((hi - lo) >> 1);
        if (keys[mid] <= v) lo = mid + 1; else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

constexpr int kFDs = 2 * (kMaxK - 1);          // 30 feature reals

}  // namespace

// Basis tables: anchor a, sample r, feature c (bin k = c / 2 + 1; even ones
// cos, odd ones -sin): the value at the exact phase ((k r) mod m) / m.
__global__ __launch_bounds__(kBlock) void k_stream_basis(const SAnchor *__restrict__ anc, int na,
                                                         double *__restrict__ basis) {
    const int a = blockIdx.y;
    if (a >= na) return;
    const int m = anc[a].m, kp = anc[a].kprime;
    const int64_t o = anc[a].bbase;
    for (int x = blockIdx.x * kBlock + threadIdx.x; x < 2 * kp * m; x += gridDim.x * kBlock) {
        const int r = x / (2 * kp), c = x % (2 * kp);
        const int k = c / 2 + 1;
        const int64_t j = ((int64_t)k * r) % m;
        double sn, cs;
        sincospi(2.0 * (double)j / (double)m, &sn, &cs);
        basis[o + x] = (c & 1) ? -sn : cs;
    }
}

// One completed non-constant window per block (one wavefront).  Two serial
// chains over the window bound it (the moments' and the features' sums, whose
// order is part of the result); the features' table is laid out by sample, so
// that a step reads one line instead of one per feature (ECG-like batches of
// 500 windows: 23 us).
__global__ __launch_bounds__(kWave) void k_stream_windows(StreamDev S) {
    extern __shared__ double ys[];                 // the window's samples, then y = x - mu
    __shared__ double s_mu, s_is;
    const int j = blockIdx.x;
    const int lane = threadIdx.x;
    const int a = S.la[j];
    const int64_t q = S.lq[j];
    const SAnchor &A = S.anc[a];
    const int m = A.m, kp = A.kprime;
    const int64_t cell = A.cbase + q;
    for (int r = lane; r < m; r += kWave) ys[r] = S.t[q + r];
    __syncthreads();
    if (lane == 0) {
        double mu;
        const double sg = window_moments(ys, m, mu);
        s_mu = mu;
        s_is = 1.0 / sg;
    }
    __syncthreads();
    const double mu = s_mu, is = s_is;
    double sabs = 0.0;
    for (int r = lane; r < m; r += kWave) {
        const double y = ys[r] - mu;
        ys[r] = y;
        sabs += fabs(y);
    }
    sabs = wave_sum(sabs);
    __syncthreads();
    // feature c = lane: X_c = sum_r y_r B[c][r], in order, then F = X / sigma
    double f = 0.0;
    if (lane < 2 * kp) {
        const double *b = S.basis + A.bbase + lane;
        const int ld = 2 * kp;
        double x = 0.0;
#pragma unroll 24
        for (int r = 0; r < m; ++r) x = fma(ys[r], b[(int64_t)r * ld], x);
        f = x * is;
    }
    const double nrm = sqrt(wave_sum(lane < kFDs ? f * f : 0.0)) * (1.0 + 1e-15);
    // Error bound e >= ||F~ - F||.  With u = 2^-53: each y_r is the rounded
    // difference x_r - mu~ (u relative), and by Lemma 1 the bins k >= 1 of
    // x - mu~ are the window's own for any constant mu~; each basis value is
    // within 12u of the exact cos / sin (the phase 2 j / m rounded by up to
    // 2u, times pi, and sincospi's own error); the in-order sum of m
    // products adds gamma_m sum |y|.
    // Per component that is (13u + gamma_m) sum_r |y_r| (1 + 2u), over 2K'
    // components sqrt(2K') times as much; scaling by 1/sigma~ (within
    // (m + 8) u of 1/sigma, plus the product's u) adds (m + 10) u ||F||.
    const double u = 1.1102230246251565e-16;
    const double gm = (double)m * u / (1.0 - (double)m * u);
    const double ex = sqrt(2.0 * kp) * (13.0 * u + gm) * (1.0 + 2e-15) * sabs * (1.0 + (double)m * u);
    const double e = (ex * is * (1.0 + (m + 10.0) * u) + (m + 10.0) * u * nrm * 1.001) * (1.0 + 1e-6) +
                     1e-300;
    if (lane < kRec)
        S.F[cell * kRec + lane] = lane < kFDs ? f : lane == kSlotErr ? e : nrm;
    if (lane == 0) {
        S.mu[cell] = mu;
        S.isig[cell] = is;
        S.P[cell] = kInfBits;
        S.I[cell] = -1;
    }
    // SimHash (Sec. 3.4): bit l = [<g_l, F> >= 0], paper bit 1 at the key's
    // top; the margins |<g_l, F>| order the Hamming-1 probes
    double v = 0.0;
    const float *g = S.gproj + ((int64_t)a * kMaxBits + (lane < kMaxBits ? lane : 0)) * kFDs;
    for (int c = 0; c < kFDs; ++c) {
        const double fc = __shfl(f, c, kWave);
        if (lane < S.B) v = fma((double)g[c], fc, v);
    }
    const uint64_t bits = __ballot(lane < S.B && v >= 0.0);
    if (lane < kMaxBits) S.bmarg[(int64_t)j * kMaxBits + lane] = lane < S.B ? (float)fabs(v) : INFINITY;
    if (lane == 0) {
        uint32_t key = 0;
        for (int l = 0; l < S.B; ++l) key |= (uint32_t)((bits >> l) & 1ull) << (S.B - 1 - l);
        S.bkey[j] = key;
    }
}

// One completed window per block of kProbeWaves wavefronts: candidates, prune,
// verify.  The search is defined as a chain of turns: a turn is up to 64 entries
// of one bucket, pruned against max(best, P[c]) as it stood before the turn.
// Only that bound ties the turns together, and it only falls.  So the block
// lists the candidates of several turns, bounds all of them at once, verifies
// the first turn's, then everything that its best leaves of the later ones, and
// replays the turns over these values: which pairs count as verified, which
// improve a cell and the query's best are those of the chain.
//
// A chain of dependent loads bounds it (a batch completes a few hundred windows,
// too few to hide one behind another): bounds of the buckets in the runs, entry,
// record and cell, samples twice.  ECG-like batches of 500 windows: 97 us with
// one wavefront a window that looked up a bucket when it came to it, 53 with a
// block, all buckets looked up at once and nine turns one after the other, 40
// now.
constexpr int kProbeWaves = 4;
constexpr int kTurn = kWave;                          // entries per turn
constexpr int kList = kProbeWaves * kWave;            // candidates listed at a time
constexpr int kGroups = kList / kGroup;
constexpr int kPreload = 64;                          // entries per bucket read ahead

__global__ __launch_bounds__(kProbeWaves *kWave) void k_stream_probe(StreamDev S) {
    extern __shared__ double qwin[];               // the query's samples
    __shared__ uint32_t roff[kProbeSlots + 1][kStreamMaxRuns];   // bucket: offset of each run's part
    __shared__ uint32_t rlo[kProbeSlots + 1][kStreamMaxRuns];    // and its first position in the run
    __shared__ uint32_t tot[kProbeSlots + 1], pre[kProbeSlots + 1];
    __shared__ int nbk;
    __shared__ int32_t ent[kProbeSlots + 1][kPreload];
    // the listed candidates: start, bound, cell value, distance, whether it
    // improves the cell; first candidate of each turn
    __shared__ int32_t lc[kList];
    __shared__ float llb[kList];
    __shared__ double lP[kList], ld[kList];
    __shared__ uint8_t lup[kList];
    __shared__ uint16_t lturn[kList], tstart[kList + 1];
    __shared__ double wbest[kProbeWaves];
    __shared__ double qbest;
    __shared__ int32_t qbestc;
    const int j = blockIdx.x;
    const int tid = threadIdx.x, lane = lane_id(), w = tid / kWave;
    const int g = lane & (kGroup - 1), grp = lane / kGroup;
    const int a = S.la[j];
    const int64_t q = S.lq[j];
    const SAnchor &A = S.anc[a];
    const int m = A.m, d = A.depth, nr = A.nruns;
    const int64_t cbase = A.cbase, cq = cbase + q;
    const double *F = S.F + cbase * kRec;
    const RecPart<double> fq = load_part(S.F + cq * kRec, g);
    const double eq = S.F[cq * kRec + kSlotErr];
    const double muq = S.mu[cq], isq = S.isig[cq];
    const float sqrt2m = (float)sqrt(2.0 / (double)m) * (1.0f + 1e-7f);
    const uint32_t key = S.bkey[j];
    const int sh = S.B - d;
    for (int r = tid; r < m; r += kProbeWaves * kWave) qwin[r] = S.t[q + r];

    // the buckets: the key's own prefix, then the Hamming-1 probes, the h
    // prefix bits of smallest margin in that order
    if (w == 0) {
        const uint32_t pfx = d > 0 ? key >> sh : 0u;
        if (lane == 0) pre[0] = pfx;
        float mg = lane < d ? S.bmarg[(int64_t)j * kMaxBits + lane] : INFINITY;
        int n = 1;
        for (int x = 0; x < kProbeSlots && x < A.probes; ++x) {
            // smallest (margin, bit) over the lanes still in
            float bm = mg;
            int bl = lane < d ? lane : kWave;
#pragma unroll
            for (int off = kWave / 2; off > 0; off >>= 1) {
                const float om = __shfl_xor(bm, off, kWave);
                const int ol = __shfl_xor(bl, off, kWave);
                if (om < bm || (om == bm && ol < bl)) {
                    bm = om;
                    bl = ol;
                }
            }
            if (bl >= d) break;
            if (lane == 0) pre[n] = pfx ^ (1u << (d - 1 - bl));
            if (lane == bl) mg = INFINITY;
            ++n;
        }
        if (lane == 0) nbk = n;
    }
    __syncthreads();
    const int nb = nbk;
    const uint32_t *keys = S.skey + cbase;
    for (int x = tid; x < nb * nr; x += kProbeWaves * kWave) {
        const int pi = x / nr, r = x - pi * nr;
        const uint32_t p = pre[pi], e = A.runs[r + 1];
        const uint32_t klo = d > 0 ? p << sh : 0u;
        const uint32_t khi = d > 0 ? (p + 1u) << sh : 1u << S.B;
        // both ends of the range in one chain
        uint32_t l0 = A.runs[r], h0 = e, l1 = l0, h1 = e;
        while (l0 < h0 || l1 < h1) {
            const uint32_t m0 = l0 + ((h0 - l0) >> 1), m1 = l1 + ((h1 - l1) >> 1);
            const uint32_t k0 = l0 < h0 ? keys[m0] : 0u, k1 = l1 < h1 ? keys[m1] : 0u;
            if (l0 < h0) {
                if (k0 < klo) l0 = m0 + 1; else h0 = m0;
            }
            if (l1 < h1) {
                if (k1 < khi) l1 = m1 + 1; else h1 = m1;
            }
        }
        rlo[pi][r] = l0;
        roff[pi][r] = l1 - l0;
    }
    __syncthreads();
    for (int pi = w; pi < nb; pi += kProbeWaves) {
        const uint32_t sz = lane < nr ? roff[pi][lane] : 0u;
        uint32_t incl = sz;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const uint32_t y = __shfl_up(incl, off, kWave);
            if (lane >= off) incl += y;
        }
        if (lane < nr) roff[pi][lane] = incl - sz;
        if (lane == kWave - 1) tot[pi] = incl;
    }
    __syncthreads();

    // bucket position (runs oldest first) -> window start
    auto entry = [&](int pi, uint32_t pos) -> int32_t {
        int rl = 0, rh = nr - 1;
        while (rl < rh) {
            const int mid = (rl + rh + 1) >> 1;
            if (roff[pi][mid] <= pos) rl = mid; else rh = mid - 1;
        }
        return (int32_t)S.perm[cbase + rlo[pi][rl] + (pos - roff[pi][rl])];
    };
    // the entries of the small buckets, all at once
    for (int x = tid; x < nb * kPreload; x += kProbeWaves * kWave) {
        const int pi = x / kPreload, pos = x % kPreload;
        if (tot[pi] <= (uint32_t)kPreload && (uint32_t)pos < tot[pi]) ent[pi][pos] = entry(pi, pos);
    }
    __syncthreads();

    double best = INFINITY;                         // the same in the whole block
    int32_t bestc = -1;
    unsigned long long n_cand = 0;
    uint32_t n_ver = 0;                             // (wavefront 0)
    int brem = S.R, n = 0, turns = 0;               // listed candidates, their turns
    struct QueryA {
        const double *w;
        int64_t base;
        __device__ __forceinline__ double operator()(int64_t x) const { return w[x - base]; }
    };
    const QueryA qa{qwin, q};
    auto group_bits = [&](bool b) -> uint32_t {
        return (uint32_t)(__ballot(b) >> (grp * kGroup)) & 0xFFu;
    };

    // the bucket at work: all of its entries, or (more than budget) half of the
    // rest of the budget on the most recent and half at even intervals over the
    // older ones
    int pi = 0, part = 0;                           // part: all, recent, spread
    uint32_t base = 0, used = 0, nrec = 0;
    for (;;) {
        // the next turn: an entry per lane, the same in every wavefront
        int32_t c = -1;
        bool have = false;
        while (!have && pi < nb && brem > 0) {
            const uint32_t total = tot[pi], pos = base + lane;
            if (part == 0 && base == 0 && total > (uint32_t)brem) {
                part = 1;
                nrec = (uint32_t)(brem / 2);
            }
            const uint32_t end = part == 0 ? total : part == 1 ? nrec : (uint32_t)brem - nrec;
            if (base >= end) {
                base = 0;
                if (part == 1) {
                    part = 2;
                    continue;
                }
                brem = part == 0 ? brem - (int)used : 0;
                used = 0;
                ++pi;
                continue;
            }
            have = true;
            base += kTurn;
            if (pos >= end) continue;
            uint32_t at = pos;
            if (part == 1) at = total - 1u - pos;
            if (part == 2) at = (uint32_t)((uint64_t)pos * (total - nrec) / (uint64_t)end);
            c = total <= (uint32_t)kPreload ? ent[pi][at] : entry(pi, at);
        }
        const bool valid = c >= 0 && q - (int64_t)c >= S.excl;
        const uint64_t vmask = __ballot(valid);
        const int nv = __popcll(vmask);
        if (n > 0 && (!have || n + nv > kList)) {
            // ---- the listed turns (uniform in the block)
            if (w == 0 && lane == 0) tstart[turns] = (uint16_t)n;
            __syncthreads();
            // candidates over the groups in turn, so that every group has as few
            const int i = g * kGroups + w * kPerRound + grp;
            const bool mine = i < n;
            const int32_t cm = mine ? lc[i] : 0;
            const bool first = mine && lturn[i] == 0;
            double Pc = INFINITY, muc = 0.0, isc = 0.0;
            if (mine) {
                Pc = bitsd(S.P[cbase + cm]);
                muc = S.mu[cbase + cm];
                isc = S.isig[cbase + cm];
            }
            const uint32_t m8 = group_bits(mine);
            float lb = 0.0f;
            if (m8) lb = group_lb<double>(F, fq, eq, (uint32_t)cm, mine, m8, g, sqrt2m);
            // the distances of the group's lanes with `prop`, one after the other
            double dist = INFINITY;
            auto verify = [&](bool prop, double thr) {
                const uint32_t p8 = group_bits(prop);
                for (int x = 0; x < kGroup; ++x) {
                    if (__ballot((p8 >> x) & 1u) == 0) continue;
                    const bool go = (p8 >> x) & 1u;
                    const int32_t vc = __shfl(cm, x, kGroup);
                    const double vthr = __shfl(thr, x, kGroup);
                    const double vmu = __shfl(muc, x, kGroup), vis = __shfl(isc, x, kGroup);
                    const double dd = snap(group_zdist_a(qa, S.t, q, muq, isq, go ? (int64_t)vc : q, vmu,
                                                         vis, go ? m : 0, exit_bound(vthr)));
                    if (go && g == x) dist = dd;
                }
            };
            double thr = fmax(best, Pc);
            verify(first && (double)lb < thr, thr);
            if (turns > 1) {
                double v = dist;
#pragma unroll
                for (int off = kWave / 2; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off, kWave));
                if (lane == 0) wbest[w] = v;
                __syncthreads();
                double b1 = best;
#pragma unroll
                for (int x = 0; x < kProbeWaves; ++x) b1 = fmin(b1, wbest[x]);
                thr = fmax(b1, Pc);
                verify(mine && !first && (double)lb < thr, thr);
            }
            if (mine) {
                llb[i] = lb;
                lP[i] = Pc;
                ld[i] = dist;
            }
            __syncthreads();
            // the turns in order, on one wavefront
            if (w == 0) {
                for (int u = 0; u < turns; ++u) {
                    const int x = tstart[u] + lane;
                    const bool in = x < (int)tstart[u + 1];
                    double d1 = INFINITY;
                    int32_t c1 = -1;
                    bool prop = false, up = false;
                    if (in) {
                        const double p = lP[x];
                        prop = (double)llb[x] < fmax(best, p);
                        if (prop) {
                            d1 = ld[x];
                            if (d1 < INFINITY) c1 = lc[x];
                            up = d1 < p;
                        }
                        lup[x] = up;
                    }
                    n_ver += (uint32_t)__popcll(__ballot(prop));
                    // the query's best over the turn: smallest (distance, start)
                    if (__ballot(c1 >= 0 && (d1 < best || (d1 == best && c1 < bestc))) == 0) continue;
#pragma unroll
                    for (int off = kWave / 2; off > 0; off >>= 1) {
                        const double od = __shfl_xor(d1, off, kWave);
                        const int32_t oc = __shfl_xor(c1, off, kWave);
                        if (od < d1 || (od == d1 && (uint32_t)oc < (uint32_t)c1)) {
                            d1 = od;
                            c1 = oc;
                        }
                    }
                    best = d1;
                    bestc = c1;
                }
                if (lane == 0) {
                    qbest = best;
                    qbestc = bestc;
                }
            }
            __syncthreads();
            best = qbest;
            bestc = qbestc;
            // the improvements, one reservation per wavefront
            const bool up = mine && lup[i];
            const uint64_t um = __ballot(up);
            if (um) {
                uint32_t at = 0;
                if (lane == 0) at = atomicAdd(S.nupd, (uint32_t)__popcll(um));
                at = (uint32_t)__shfl((int)at, 0, kWave) + (uint32_t)__popcll(um & lanemask_lt());
                if (up) {
                    if (at < S.updcap) S.upd[at] = SUpdate{(uint32_t)(cbase + cm), (int32_t)q, dbits(dist)};
                    else count_add(S.counters, CS_DROP, 1ull);
                }
            }
            n = turns = 0;
        }
        if (!have) break;
        if (nv == 0) continue;
        n_cand += (unsigned long long)nv;
        used += (uint32_t)nv;
        if (w == 0) {
            if (valid) {
                const int x = n + __popcll(vmask & lanemask_lt());
                lc[x] = c;
                lturn[x] = (uint16_t)turns;
            }
            if (lane == 0) tstart[turns] = (uint16_t)n;
        }
        n += nv;
        ++turns;
    }
    if (tid == 0) {
        S.P[cq] = dbits(best);
        S.I[cq] = bestc;
        if (n_cand) count_add(S.counters, CS_CAND, n_cand);
        if (n_ver) count_add(S.counters, CS_VER, (unsigned long long)n_ver);
    }
}

// The end of a batch, a block per anchor and one more, all independent: the
// anchors' directories and the buffered improvements.  As launches of their own
// the new runs, merges, copies back and improvements took 9 + 8 + 5 + 5.5 us of
// an ECG-like batch, and 5 us of host time each; together 9.
constexpr int kFinish = 1024;

// The buffered improvements into the profile.  Every buffered distance is
// below its cell's value when the searches started, so each touched cell drops
// to the smallest one; its neighbour is the smallest query start among those
// reaching that value.
__device__ __forceinline__ void stream_apply(const StreamDev &S) {
    const uint32_t n = min(*S.nupd, S.updcap);
    for (uint32_t x = threadIdx.x; x < n; x += kFinish)
        __hip_atomic_store(&S.Icand[S.upd[x].cell], INT_MAX, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    for (uint32_t x = threadIdx.x; x < n; x += kFinish)
        atomicMin((unsigned long long *)&S.P[S.upd[x].cell], (unsigned long long)S.upd[x].d);
    __syncthreads();
    // values other threads changed by atomics are read at device scope (not
    // from this compute unit's cache)
    for (uint32_t x = threadIdx.x; x < n; x += kFinish) {
        const SUpdate u = S.upd[x];
        if (__hip_atomic_load(&S.P[u.cell], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == u.d)
            atomicMin(&S.Icand[u.cell], u.j);
    }
    __syncthreads();
    for (uint32_t x = threadIdx.x; x < n; x += kFinish) {
        const uint32_t c = S.upd[x].cell;
        S.I[c] = __hip_atomic_load(&S.Icand[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (n) atomicAdd(&S.counters[CS_UPD], (unsigned long long)n);
        *S.nupd = 0;
    }
}

// Block a < na: the batch's windows of anchor a as a new run, sorted by (key,
// start) (the list holds an anchor's windows in start order), then the merge of
// its newest runs (binary counter) if one block holds it: each element's place
// is its rank in its own run plus, in every other run, the entries before it (an
// older run's equal keys come first).  Larger merges: k_stream_merge.
__global__ __launch_bounds__(kFinish) void k_stream_finish(StreamDev S, int na,
                                                           const SMerge *__restrict__ mg) {
    __shared__ uint32_t mk[kStreamMergeLds], mp[kStreamMergeLds];
    if ((int)blockIdx.x == na) {
        stream_apply(S);
        return;
    }
    const SAnchor &A = S.anc[blockIdx.x];
    const int nn = A.nnew, g = threadIdx.x & (kGroup - 1);
    // eight lanes per window count the keys before its own
    for (int i0 = 0; i0 < nn; i0 += kFinish / kGroup) {
        const int i = i0 + threadIdx.x / kGroup;
        const uint32_t ki = i < nn ? S.bkey[A.j0 + i] : 0u;
        int rank = 0;
        for (int x0 = 0; x0 < nn; x0 += (int)kStreamMergeLds) {
            const int xn = min(nn - x0, (int)kStreamMergeLds);
            if (i0 == 0 || nn > (int)kStreamMergeLds) {
                __syncthreads();
                for (int x = threadIdx.x; x < xn; x += kFinish) mk[x] = S.bkey[A.j0 + x0 + x];
                __syncthreads();
            }
            for (int x = g; x < xn; x += kGroup) {
                const uint32_t kx = mk[x];
                rank += kx < ki || (kx == ki && x0 + x < i);
            }
        }
        rank += xor_lane<1>(rank);
        rank += xor_lane<2>(rank);
        rank += xor_lane<4>(rank);
        if (i < nn && g == 0) {
            const int64_t pos = A.cbase + A.nidx + rank;
            S.skey[pos] = ki;
            S.perm[pos] = (uint32_t)S.lq[A.j0 + i];
        }
    }
    if (A.merge < 0) return;
    __syncthreads();                               // (the new run is read back)
    const SMerge &M = mg[A.merge];
    const uint32_t r0 = M.runs[0], n = M.runs[M.nruns] - r0;
    for (uint32_t x = threadIdx.x; x < n; x += kFinish) {
        mk[x] = S.skey[M.cbase + r0 + x];
        mp[x] = S.perm[M.cbase + r0 + x];
    }
    __syncthreads();
    for (uint32_t x = threadIdx.x; x < n; x += kFinish) {
        const uint32_t k = mk[x];
        int r = 0;
        while (r + 1 < M.nruns && M.runs[r + 1] - r0 <= x) ++r;
        uint32_t out = x - (M.runs[r] - r0);
        for (int o = 0; o < M.nruns; ++o) {
            if (o == r) continue;
            const uint32_t b0 = M.runs[o] - r0, b1 = M.runs[o + 1] - r0;
            out += (o < r ? upper_bound_u32(mk, b0, b1, k) : lower_bound_u32(mk, b0, b1, k)) - b0;
        }
        S.skey[M.cbase + r0 + out] = k;
        S.perm[M.cbase + r0 + out] = mp[x];
    }
}

// The merges of more entries than one block holds, placed likewise.  Written to
// the scratch arrays, then copied back.
__global__ __launch_bounds__(kBlock) void k_stream_merge(StreamDev S, const SMerge *__restrict__ mg,
                                                         int nmerge, int64_t nthreads) {
    const int64_t x = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (x >= nthreads) return;
    int lo = 0, hi = nmerge - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (mg[mid].first <= x) lo = mid; else hi = mid - 1;
    }
    const SMerge &M = mg[lo];
    const uint32_t e = M.runs[0] + (uint32_t)(x - M.first);
    if (e >= M.runs[M.nruns]) return;
    const uint32_t *keys = S.skey + M.cbase;
    int r = 0;
    while (r + 1 < M.nruns && M.runs[r + 1] <= e) ++r;
    const uint32_t k = keys[e];
    uint32_t out = M.runs[0] + (e - M.runs[r]);
    for (int o = 0; o < M.nruns; ++o) {
        if (o == r) continue;
        const uint32_t b0 = M.runs[o], b1 = M.runs[o + 1];
        out += (o < r ? upper_bound_u32(keys, b0, b1, k) : lower_bound_u32(keys, b0, b1, k)) - b0;
    }
    S.ktmp[M.cbase + out] = k;
    S.ptmp[M.cbase + out] = S.perm[M.cbase + e];
}

__global__ __launch_bounds__(kBlock) void k_stream_merge_back(StreamDev S,
                                                              const SMerge *__restrict__ mg,
                                                              int nmerge, int64_t nthreads) {
    const int64_t x = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (x >= nthreads) return;
    int lo = 0, hi = nmerge - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (mg[mid].first <= x) lo = mid; else hi = mid - 1;
    }
    const SMerge &M = mg[lo];
    const uint32_t e = M.runs[0] + (uint32_t)(x - M.first);
    if (e >= M.runs[M.nruns]) return;
    S.skey[M.cbase + e] = S.ktmp[M.cbase + e];
    S.perm[M.cbase + e] = S.ptmp[M.cbase + e];
}

__global__ __launch_bounds__(kBlock) void k_iota_u32(uint32_t *__restrict__ p, int64_t n) {
    const int64_t x = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (x < n) p[x] = (uint32_t)x;
}

// ------------------------------------------------------------ launchers

static inline unsigned sblk(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

void launch_stream_basis(const SAnchor *anc, int na, int64_t max_elems, double *basis,
                         hipStream_t s) {
    if (na <= 0) return;
    const unsigned gx = (unsigned)std::min<int64_t>(64, (max_elems + kBlock - 1) / kBlock);
    hipLaunchKernelGGL(k_stream_basis, dim3(gx, (unsigned)na), dim3(kBlock), 0, s, anc, na, basis);
}

void launch_stream_windows(const StreamDev &S, int max_m, hipStream_t s) {
    if (S.nlist <= 0) return;
    hipLaunchKernelGGL(k_stream_windows, dim3((unsigned)S.nlist), dim3(kWave),
                       (size_t)max_m * sizeof(double), s, S);
}

// Windows per launch of the search.  A launch has fewer than 2^32 work-items,
// which a batch of 2^24 windows has at 256 threads each; 2^16 windows fill the
// chip thirty times over.
constexpr int kStreamPiece = 1 << 16;
static_assert((int64_t)kStreamPiece * kProbeWaves * kWave < (int64_t)1 << 32, "work-items of a launch");

void launch_stream_probe(const StreamDev &S, int max_m, hipStream_t s) {
    for (int64_t at = 0; at < S.nlist; at += kStreamPiece) {
        StreamDev B = S;
        B.la += at;
        B.lq += at;
        B.bkey += at;
        B.bmarg += at * kMaxBits;
        hipLaunchKernelGGL(k_stream_probe, dim3((unsigned)std::min<int64_t>(S.nlist - at, kStreamPiece)),
                           dim3(kProbeWaves * kWave), (size_t)max_m * sizeof(double), s, B);
    }
}

void launch_stream_finish(const StreamDev &S, int na, const SMerge *mg, hipStream_t s) {
    if (S.nlist <= 0) return;
    hipLaunchKernelGGL(k_stream_finish, dim3((unsigned)na + 1), dim3(kFinish), 0, s, S, na, mg);
}

void launch_stream_merge(const StreamDev &S, const SMerge *mg, int nmerge, int64_t nthreads,
                         hipStream_t s) {
    if (nmerge <= 0 || nthreads <= 0) return;
    hipLaunchKernelGGL(k_stream_merge, dim3(sblk(nthreads)), dim3(kBlock), 0, s, S, mg, nmerge,
                       nthreads);
    hipLaunchKernelGGL(k_stream_merge_back, dim3(sblk(nthreads)), dim3(kBlock), 0, s, S, mg,
                       nmerge, nthreads);
}

void launch_iota_u32(uint32_t *p, int64_t n, hipStream_t s) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_iota_u32, dim3(sblk(n)), dim3(kBlock), 0, s, p, n);
}

}  // namespace pmp
