// quant.h -- the 16-bit prefilter in front of the FP64 distance (device code,
// shared by the probe, the hints and the join's exact stage).
//
// Nearly every pair that the Parseval bound lets through at noisy data lies past
// the value it would have to undercut all the same (its noise is in the bins
// that no record holds), and its exact distance reads two windows of FP64
// samples only to say so.  The series is
// therefore also held as 16-bit integers x = rint((t - c) / s), c its centre
// and s its half range over 32767 (2 MB for 1e6 samples, which an XCD's L2
// holds, a quarter of the bytes), and a pair is first summed on those, in
// FP32.  With z = (t - mu) / sigma = x s / sigma + (c - mu) / sigma up to
//   delta = (2^-16 (1 + 1e-4) + 2^-21) max|t - c| / sigma
// per sample (the rounding of x; the second term covers the FP32 factors and
// the FP32 evaluation of the difference: six units of 2^-24 max|t - c| / sigma on
// one side and seven on the other, of eight each), the sum S over the window obeys
//   sqrt(S) <= d + sqrt(m) (delta_i + delta_j),  S's own roundings < 1e-4,
// so a pair whose S reaches (thr + sqrt(m) (delta_i + delta_j))^2 (1 + 2e-4)
// has d > thr and can lower no cell from above thr.  Every other pair goes on
// to the FP64 distance, which alone decides; a pair whose margin exceeds
// thr / 8 (windows of a spread far below the series' range) skips the
// prefilter.  Measured at the join's exact stage (ECG-like 1M, 4.2e8 pairs of
// 100..400 samples): 96 -> 15 ms, 335 distances instead of 4.0e8.
#pragma once

#include "pmp_dev.h"

namespace pmp {

typedef uint32_t u32x4a __attribute__((ext_vector_type(4), aligned(4)));   // 16 bytes at 4

// acc += sum of the squared differences of eight samples (two per word);
// kTail: only those with index r + e < m.
template <bool kTail>
__device__ __forceinline__ void quant_add(u32x4a x, u32x4a y, float ai, float aj, float b, int r,
                                          int m, float &s0, float &s1) {
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const float x0 = (float)(int16_t)(x[w] & 0xFFFFu), x1 = (float)((int32_t)x[w] >> 16);
        const float y0 = (float)(int16_t)(y[w] & 0xFFFFu), y1 = (float)((int32_t)y[w] >> 16);
        float e0 = fmaf(x0, ai, fmaf(-y0, aj, b)), e1 = fmaf(x1, ai, fmaf(-y1, aj, b));
        if (kTail) {
            e0 = r + 2 * w < m ? e0 : 0.0f;
            e1 = r + 2 * w + 1 < m ? e1 : 0.0f;
        }
        s0 = fmaf(e0, e0, s0);
        s1 = fmaf(e1, e1, s1);
    }
}

// Whether a pair is worth the prefilter at thr (finite, > 0), and the squared
// sum from which it is out.  wi, wj: the windows' entries of Quant::xw.
__device__ __forceinline__ bool quant_limit(const float4 &wi, const float4 &wj, int m, double thr,
                                            float &lim) {
    const double margin = sqrt((double)m) * ((double)wi.w + (double)wj.w);
    const double r = thr + margin;
    lim = (float)(r * r * (1.0 + 2e-4) * (1.0 + 1e-6));
    return margin <= 0.125 * thr && thr < INFINITY;
}

// False when the 16-bit sum of the windows starting at si and sj reaches lim.
// A group of kLanes lanes (4 or 8; g: the lane's place) takes one pair, whose
// arguments all its lanes hold; whole groups call.  Reads up to 63 entries past
// the longer window, within the arrays' padding.
template <int kLanes>
__device__ __forceinline__ bool quant_below(const int16_t *__restrict__ x16, int64_t pitch,
                                            uint32_t si, uint32_t sj, float ai, float aj, float b,
                                            int m, float lim, int g) {
    static_assert(kLanes == 4 || kLanes == 8, "lanes of a pair");
    constexpr int kStep = 8 * kLanes;
    const int16_t *const px = x16 + (si & 1u) * pitch + (si & ~1u) + 8 * g;
    const int16_t *const py = x16 + (sj & 1u) * pitch + (sj & ~1u) + 8 * g;
    float s0 = 0.0f, s1 = 0.0f;
    for (int r0 = 0; r0 < m; r0 += 64) {
        // (64 samples a turn: two loads a window with four lanes, one with
        // eight)
        const u32x4a x0 = *(const u32x4a *)(px + r0), y0 = *(const u32x4a *)(py + r0);
        u32x4a x1, y1;
        if (kLanes == 4) {
            x1 = *(const u32x4a *)(px + r0 + kStep);
            y1 = *(const u32x4a *)(py + r0 + kStep);
        }
        if (r0 + 64 <= m) {
            quant_add<false>(x0, y0, ai, aj, b, 0, 0, s0, s1);
            if (kLanes == 4) quant_add<false>(x1, y1, ai, aj, b, 0, 0, s0, s1);
        } else {
            quant_add<true>(x0, y0, ai, aj, b, r0 + 8 * g, m, s0, s1);
            if (kLanes == 4) quant_add<true>(x1, y1, ai, aj, b, r0 + kStep + 8 * g, m, s0, s1);
        }
        float s = s0 + s1;
        s += xor_lane<1>(s);
        s += xor_lane<2>(s);
        if (kLanes == 8) s += xor_lane<4>(s);
        if (s >= lim) return false;
    }
    return true;
}

}  // namespace pmp
