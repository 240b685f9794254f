// k_scan.hip -- exclusive scan and stable LSD radix sort for gfx950.
//
// The radix sort ranks keys inside a wave with ballots (one ballot per digit
// bit gives each lane the set of lanes holding the same digit), so a block
// needs no LDS histogram per thread; each wave takes a contiguous slice of
// its block's tile, waves are chained through a small LDS table of digit
// counts (one block barrier), and blocks through a scan of per-(digit,
// block) counts.  Stability
// (equal keys keep their input order) is what keeps each bucket of the
// directory sorted by window start.
#include "pmp_dev.h"

#include <algorithm>
#include <cstring>

namespace pmp {

namespace {

constexpr int kScanItems = 8;                       // per thread
constexpr int kScanTile = kBlock * kScanItems;      // 2048 per block

// Block-wide exclusive scan of one value per thread; returns the block total.
__device__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *lds /* >= 4 */, uint32_t &excl) {
    const int lane = lane_id();
    const int w = threadIdx.x / kWave;
    // inclusive wave scan by shuffles
    uint32_t x = v;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        uint32_t y = __shfl_up(x, off, kWave);
        if (lane >= off) x += y;
    }
    if (lane == kWave - 1) lds[w] = x;
    __syncthreads();
    uint32_t wbase = 0, total = 0;
#pragma unroll
    for (int i = 0; i < kBlock / kWave; ++i) {
        uint32_t s = lds[i];
        if (i < w) wbase += s;
        total += s;
    }
    __syncthreads();
    excl = wbase + x - v;
    return total;
}

// The whole scan by one block, for inputs of a few thousand: one launch for
// three.
constexpr int64_t kScanOne = 16384;
__global__ __launch_bounds__(1024) void k_scan_one(const uint32_t *in, uint32_t *out, int64_t n,
                                                   uint32_t *__restrict__ total) {
    __shared__ uint32_t lds[1024 / kWave];
    const int lane = lane_id(), w = threadIdx.x / kWave;
    constexpr int kPer = (int)(kScanOne / 1024);
    // a contiguous share per thread
    const int per = (int)((n + 1023) / 1024);
    const int64_t base = (int64_t)threadIdx.x * per;
    uint32_t v[kPer], s = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        v[k] = k < per && base + k < n ? in[base + k] : 0u;
        s += v[k];
    }
    uint32_t x = s;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t y = __shfl_up(x, off, kWave);
        if (lane >= off) x += y;
    }
    if (lane == kWave - 1) lds[w] = x;
    __syncthreads();
    uint32_t run = x - s, tot = 0;
#pragma unroll
    for (int i = 0; i < 1024 / kWave; ++i) {
        const uint32_t y = lds[i];
        if (i < w) run += y;
        tot += y;
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        if (k < per && base + k < n) out[base + k] = run;
        run += v[k];
    }
    if (threadIdx.x == 0 && total) *total = tot;
}

// Kernel arguments as the transport of small uploads: a copy from pageable
// memory costs the host about 35 us, a launch with 3.5 KB of arguments 5.
constexpr int kUploadWords = 896;
constexpr int kUploadMax = 8;                       // launches of one upload
struct UploadBlob {
    uint32_t w[kUploadWords];
};
__global__ __launch_bounds__(kBlock) void k_upload(UploadBlob b, int n, uint32_t *__restrict__ dst,
                                                   uint32_t *__restrict__ zero, int64_t nz) {
    for (int i = threadIdx.x; i < n; i += kBlock) dst[i] = b.w[i];
    for (int64_t i = threadIdx.x; i < nz; i += kBlock) zero[i] = 0u;
}

__global__ __launch_bounds__(kBlock) void k_len_offsets(const LenInfo *__restrict__ len, int L,
                                                        const uint32_t *__restrict__ tile_off,
                                                        int64_t ntiles,
                                                        uint32_t *__restrict__ offs) {
    for (int l = threadIdx.x; l <= L; l += kBlock)
        offs[l] = tile_off[l < L ? len[l].tile_base : ntiles];
}

__global__ __launch_bounds__(kBlock) void k_scan_reduce(const uint32_t *__restrict__ in,
                                                        int64_t n, uint32_t *__restrict__ sums) {
    __shared__ uint32_t lds[kBlock / kWave];
    int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        int64_t i = base + k;
        if (i < n) s += in[i];
    }
    uint32_t ex;
    uint32_t tot = block_exclusive_scan(s, lds, ex);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// One block scans the block sums in place (exclusive) and writes the total.
__global__ __launch_bounds__(1024) void k_scan_sums(uint32_t *__restrict__ sums, int64_t nb,
                                                    uint32_t *__restrict__ total) {
    __shared__ uint32_t lds[1024 / kWave];
    __shared__ uint32_t carry;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    const int lane = lane_id();
    const int w = threadIdx.x / kWave;
    for (int64_t base = 0; base < nb; base += 1024) {
        int64_t i = base + threadIdx.x;
        uint32_t v = i < nb ? sums[i] : 0u;
        uint32_t x = v;
        for (int off = 1; off < kWave; off <<= 1) {
            uint32_t y = __shfl_up(x, off, kWave);
            if (lane >= off) x += y;
        }
        if (lane == kWave - 1) lds[w] = x;
        __syncthreads();
        uint32_t wbase = 0, tot = 0;
        for (int k = 0; k < 1024 / kWave; ++k) {
            uint32_t s = lds[k];
            if (k < w) wbase += s;
            tot += s;
        }
        uint32_t c = carry;
        if (i < nb) sums[i] = c + wbase + x - v;
        __syncthreads();
        if (threadIdx.x == 0) carry = c + tot;
        __syncthreads();
    }
    if (threadIdx.x == 0 && total) *total = carry;
}

__global__ __launch_bounds__(kBlock) void k_scan_apply(const uint32_t *__restrict__ in,
                                                       uint32_t *__restrict__ out, int64_t n,
                                                       const uint32_t *__restrict__ sums) {
    __shared__ uint32_t lds[kBlock / kWave];
    int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    uint32_t v[kScanItems];
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        int64_t i = base + k;
        v[k] = i < n ? in[i] : 0u;
        s += v[k];
    }
    uint32_t ex;
    block_exclusive_scan(s, lds, ex);
    uint32_t run = sums[blockIdx.x] + ex;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        int64_t i = base + k;
        if (i < n) out[i] = run;
        run += v[k];
    }
}

// ------------------------------------------------------------ radix sort

constexpr int kSortRounds = 8;                       // items per thread
constexpr int kSortTile = kBlock * kSortRounds;      // 2048 per tile
constexpr int kRadix = 256;

// Consecutive tiles per block: four amortize a block's counts over 8192 keys
// once that fills the chip; below, one tile a block gives four times the
// blocks (200,000 keys: 98 instead of 25, a pass 50 -> 19 us with the scan in
// the histogram).
constexpr int kSortSub = 4;
constexpr int64_t kSortSmall = (int64_t)1 << 20;
inline int sort_sub(int64_t n) { return n < kSortSmall ? 1 : kSortSub; }

// Histograms of up to this many blocks are scanned by their own last block; more
// by the three-kernel scan.
constexpr int64_t kSortFused = 256;

// Digit counts per block, for the block's `sub` tiles.  Fused form (ticket not
// null): counts are laid out by block, and the last block to arrive turns them
// into offsets; otherwise they are laid out by digit, for a scan of its own.
__global__ __launch_bounds__(kBlock) void k_radix_hist(const uint32_t *__restrict__ keys,
                                                       int64_t n, int shift, int nbits, int sub_n,
                                                       uint32_t *counts,
                                                       uint32_t *__restrict__ offs,
                                                       int64_t nblocks, uint32_t *ticket) {
    __shared__ uint32_t h[kRadix];
    h[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t mask = (1u << nbits) - 1u;
    const int lane = lane_id();
    // the block's tiles; wavefront w counts the slice [w, w + 1) * kSortTile /
    // 4 of each.  Equal digits of a round are matched by ballots
    // (one per digit bit) and counted by one lane, so a tile whose keys share
    // a digit (as they do after the lower passes) costs one LDS atomic per
    // round, not 64
    for (int sub = 0; sub < sub_n; ++sub) {
        const int64_t base = ((int64_t)blockIdx.x * sub_n + sub) * kSortTile +
                             (int64_t)(threadIdx.x / kWave) * (kSortTile / (kBlock / kWave));
        if (base >= n) break;
        uint32_t key[kSortRounds];
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r) {
            const int64_t i = base + (int64_t)r * kWave + lane;
            key[r] = i < n ? keys[i] : 0u;
        }
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r) {
            const bool valid = base + (int64_t)r * kWave + lane < n;
            const uint32_t dig = (key[r] >> shift) & mask;
            uint64_t peers = __ballot(valid);
            for (int b = 0; b < nbits; ++b) {
                const uint64_t bal = __ballot((dig >> b) & 1u);
                peers &= ((dig >> b) & 1u) ? bal : ~bal;
            }
            if (valid && (peers & lanemask_lt()) == 0)
                atomicAdd(&h[dig], (uint32_t)__popcll(peers));
        }
    }
    __syncthreads();
    if (!ticket) {
        // digit-major so that the exclusive scan gives each (digit, block) its
        // first output position
        counts[(int64_t)threadIdx.x * nblocks + blockIdx.x] = h[threadIdx.x];
        return;
    }
    counts[(int64_t)blockIdx.x * kRadix + threadIdx.x] = h[threadIdx.x];
    __shared__ int last;
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) last = atomicAdd(ticket, 1u) == gridDim.x - 1;
    __syncthreads();
    if (!last) return;
    __threadfence();
    if (threadIdx.x == 0) *ticket = 0;
    // thread d: the digit's total, the digits' exclusive scan, then the digit's
    // first position in every block
    uint32_t sum = 0;
#pragma unroll 16
    for (int64_t b = 0; b < nblocks; ++b) sum += counts[b * kRadix + threadIdx.x];
    __shared__ uint32_t lds[kBlock / kWave];
    uint32_t run;
    block_exclusive_scan(sum, lds, run);
#pragma unroll 16
    for (int64_t b = 0; b < nblocks; ++b) {
        const uint32_t v = counts[b * kRadix + threadIdx.x];
        offs[b * kRadix + threadIdx.x] = run;
        run += v;
    }
}

// sub_n consecutive tiles of kSortTile keys per block, in order; in each tile
// wavefront w takes the contiguous slice [w, w + 1) * kSortTile / 4 in
// kSortRounds rounds of 64.  Pass 1 ranks each key among the equal digits of
// its round (one ballot per digit bit) and counts each wavefront's digits;
// after one block barrier every (wavefront, digit) knows its first output
// position (the digit's running position in the block, which starts at the
// block's offset of the digit, plus the counts of the earlier wavefronts);
// pass 2 writes the keys.  Stable: within a digit, tiles, wavefronts, rounds
// and lanes keep their input order.
__global__ __launch_bounds__(kBlock) void k_radix_scatter(
    const uint32_t *__restrict__ kin, const uint32_t *__restrict__ vin,
    uint32_t *__restrict__ kout, uint32_t *__restrict__ vout, int64_t n, int shift, int nbits,
    int sub_n, const uint32_t *__restrict__ offs, int64_t nblocks, bool by_block) {
    constexpr int kW = kBlock / kWave;
    __shared__ uint32_t wcnt[kW][kRadix];
    const int lane = lane_id();
    const int w = threadIdx.x / kWave;
    const uint32_t mask = (1u << nbits) - 1u;
    // thread d: the next output position of digit d
    uint32_t run = by_block ? offs[(int64_t)blockIdx.x * kRadix + threadIdx.x]
                            : offs[(int64_t)threadIdx.x * nblocks + blockIdx.x];
    for (int sub = 0; sub < sub_n; ++sub) {
        const int64_t tbase = ((int64_t)blockIdx.x * sub_n + sub) * kSortTile;
        if (tbase >= n) break;
        for (int q = 0; q < kW; ++q) wcnt[q][threadIdx.x] = 0;
        __syncthreads();
        const int64_t base = tbase + (int64_t)w * (kSortTile / kW);
        uint32_t key[kSortRounds], val[kSortRounds], rank[kSortRounds];
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r) {
            const int64_t i = base + (int64_t)r * kWave + lane;
            const bool valid = i < n;
            key[r] = valid ? kin[i] : 0u;
            val[r] = valid ? vin[i] : 0u;
        }
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r) {
            const int64_t i = base + (int64_t)r * kWave + lane;
            const bool valid = i < n;
            const uint32_t dig = (key[r] >> shift) & mask;
            uint64_t peers = __ballot(valid);
            for (int b = 0; b < nbits; ++b) {
                const uint64_t bal = __ballot((dig >> b) & 1u);
                peers &= ((dig >> b) & 1u) ? bal : ~bal;
            }
            const uint32_t below = (uint32_t)__popcll(peers & lanemask_lt());
            // the digit's count so far in this wavefront (earlier rounds) plus the
            // equal digits of earlier lanes; the leader then adds the round's count
            rank[r] = below + (valid ? wcnt[w][dig] : 0u);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (valid && below == 0) wcnt[w][dig] += (uint32_t)__popcll(peers);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        {
            // thread d: the first position of digit d for each wavefront
            const int d = threadIdx.x;
            for (int q = 0; q < kW; ++q) {
                const uint32_t c = wcnt[q][d];
                wcnt[q][d] = run;
                run += c;
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r) {
            const int64_t i = base + (int64_t)r * kWave + lane;
            if (i < n) {
                const uint32_t pos = wcnt[w][(key[r] >> shift) & mask] + rank[r];
                kout[pos] = key[r];
                vout[pos] = val[r];
            }
        }
        __syncthreads();                                 // wcnt is cleared next
    }
}

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

}  // namespace

size_t scan_temp_bytes(int64_t n) {
    return (size_t)(cdiv(n, kScanTile) + 64) * sizeof(uint32_t);
}

void scan_exclusive_u32(const uint32_t *in, uint32_t *out, int64_t n, uint32_t *total,
                        void *temp, hipStream_t s) {
    if (n <= 0) {
        if (total) launch_fill_u32(total, 1, 0u, s);
        return;
    }
    if (n <= kScanOne) {
        hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(1024), 0, s, in, out, n, total);
        return;
    }
    int64_t nb = cdiv(n, kScanTile);
    uint32_t *sums = (uint32_t *)temp;
    hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)nb), dim3(kBlock), 0, s, in, n, sums);
    hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(1024), 0, s, sums, nb, total);
    hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)nb), dim3(kBlock), 0, s, in, out, n,
                       (const uint32_t *)sums);
}

size_t sort_temp_bytes(int64_t n) {
    // (a smaller n in the same buffers may take more blocks, below kSortSmall)
    int64_t nb = std::max(cdiv(n, (int64_t)kSortTile * sort_sub(n)),
                          cdiv(std::min(n, kSortSmall), kSortTile));
    size_t counts = (size_t)(nb * kRadix) * sizeof(uint32_t);
    return 2 * counts + scan_temp_bytes(nb * kRadix) + 256;
}

int radix_sort_pairs(uint32_t *k0, uint32_t *v0, uint32_t *k1, uint32_t *v1, int64_t n,
                     int lo, int hi, void *temp, uint32_t *ticket, hipStream_t s, bool copy_back) {
    if (n <= 1 || hi <= lo) return 0;
    const int sub = sort_sub(n);
    int64_t nb = cdiv(n, (int64_t)kSortTile * sub);
    const bool fused = nb <= kSortFused;
    uint32_t *counts = (uint32_t *)temp;
    uint32_t *offs = counts + nb * kRadix;
    void *stemp = (void *)(offs + nb * kRadix);
    uint32_t *ka = k0, *va = v0, *kb = k1, *vb = v1;
    int passes = 0;
    for (int shift = lo; shift < hi; shift += 8, ++passes) {
        int nbits = hi - shift < 8 ? hi - shift : 8;
        hipLaunchKernelGGL(k_radix_hist, dim3((unsigned)nb), dim3(kBlock), 0, s, ka, n, shift,
                           nbits, sub, counts, offs, nb, fused ? ticket : nullptr);
        if (!fused) scan_exclusive_u32(counts, offs, nb * kRadix, nullptr, stemp, s);
        hipLaunchKernelGGL(k_radix_scatter, dim3((unsigned)nb), dim3(kBlock), 0, s, ka, va, kb,
                           vb, n, shift, nbits, sub, (const uint32_t *)offs, nb, fused);
        uint32_t *t;
        t = ka; ka = kb; kb = t;
        t = va; va = vb; vb = t;
    }
    if ((passes & 1) && copy_back) {
        (void)hipMemcpyAsync(k0, ka, (size_t)n * sizeof(uint32_t), hipMemcpyDeviceToDevice, s);
        (void)hipMemcpyAsync(v0, va, (size_t)n * sizeof(uint32_t), hipMemcpyDeviceToDevice, s);
        return 0;
    }
    return passes & 1;
}

bool launch_upload(void *dst, const void *src, size_t bytes, uint32_t *zero, int64_t zero_words,
                   hipStream_t s) {
    if (bytes > (size_t)kUploadMax * sizeof(UploadBlob) || bytes % 4) return false;
    UploadBlob b;
    for (size_t at = 0; at < bytes || zero_words > 0; at += sizeof(b)) {
        const size_t n = std::min(bytes - at, sizeof(b));
        memcpy(b.w, (const char *)src + at, n);
        hipLaunchKernelGGL(k_upload, dim3(1), dim3(kBlock), 0, s, b, (int)(n / 4),
                           (uint32_t *)((char *)dst + at), zero, zero_words);
        zero_words = 0;
        if (at + n >= bytes) break;
    }
    return true;
}

void launch_len_offsets(const LenInfo *len, int L, const uint32_t *tile_off, int64_t ntiles,
                        uint32_t *offs, hipStream_t s) {
    hipLaunchKernelGGL(k_len_offsets, dim3(1), dim3(kBlock), 0, s, len, L, tile_off, ntiles, offs);
}

}  // namespace pmp
