// Index build, candidate-site generation and the small device-wide scan.
//
// Step "decompress indices" of Algorithm 1 becomes: mark every occupied site in
// a bitmap over (sample, lin) and remember, per 64-bit word, the row index of
// its first occupied site.  Rows are sorted by (b, lin), so the row of any
// occupied site is  prefix[word] + popcount(bits below it)  -- the inverse of
// get_update_id without a hash table and without an r^d value buffer.
//
// Candidate output sites (the sites Algorithm 1's dense buffer could become
// non-zero at) are the occupied sites dilated by the filter's non-zero taps;
// they are marked in a second bitmap, counted per word, scanned, and written
// out as a sorted list of per-sample site indices.
#include <atomic>

#include "scnn_internal.h"

namespace scnn {

int device_cu_count() {
    static std::atomic<int> cache[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 256;
    int n = (dev >= 0 && dev < 64) ? cache[dev].load(std::memory_order_relaxed) : 0;
    if (n <= 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) return 256;
        if (dev >= 0 && dev < 64) cache[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}


// ------------------------------------------------------------------ zero fill
__global__ void k_zero(uint4* __restrict__ p, size_t n16) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n16; i += stride) p[i] = make_uint4(0, 0, 0, 0);
}

hipError_t launch_zero(void* p, size_t bytes, hipStream_t s) {
    size_t n16 = (bytes + 15) / 16;
    if (n16 == 0) return hipSuccess;
    int blocks = (int)((n16 + 255) / 256);
    if (blocks > 2048) blocks = 2048;
    hipLaunchKernelGGL(k_zero, dim3(blocks), dim3(256), 0, s, (uint4*)p, n16);
    return hipGetLastError();
}

// Plain streaming copy of a known size: the yardstick against which the memory-traffic counters of the
// other kernels are scaled.
__global__ void k_calibration_copy(uint4* __restrict__ dst, const uint4* __restrict__ src, size_t n16) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n16; i += stride) dst[i] = src[i];
}

hipError_t launch_calibration_copy(void* dst, const void* src, size_t bytes, hipStream_t s) {
    const size_t n16 = bytes / 16;
    if (n16 == 0) return hipSuccess;
    size_t blocks = (n16 + 255) / 256;
    if (blocks > 256 * 32) blocks = 256 * 32;
    hipLaunchKernelGGL(k_calibration_copy, dim3((unsigned)blocks), dim3(256), 0, s, (uint4*)dst, (const uint4*)src, n16);
    return hipGetLastError();
}

// ------------------------------------------------------------------ scan
__global__ __launch_bounds__(256) void k_scan_local(unsigned* __restrict__ vals, long long n_imm,
                                                    const long long* __restrict__ n_dev,
                                                    unsigned* __restrict__ block_sums) {
    __shared__ unsigned s_wave[4];
    const long long n = n_dev ? *n_dev : n_imm;
    const long long base = (long long)blockIdx.x * kScanChunk + (long long)threadIdx.x * 8;
    unsigned v[8];
    unsigned sum = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        v[i] = (base + i < n) ? vals[base + i] : 0u;
        sum += v[i];
    }
    unsigned total;
    unsigned excl = block_exclusive_scan_256(sum, s_wave, total);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if (base + i < n) vals[base + i] = excl;
        excl += v[i];
    }
    if (threadIdx.x == 0) block_sums[blockIdx.x] = total;
}

__global__ __launch_bounds__(256) void k_scan_top(unsigned* __restrict__ block_sums, long long n_blocks,
                                                  long long* __restrict__ total_out) {
    __shared__ unsigned s_wave[4];
    unsigned carry = 0;
    for (long long start = 0; start < n_blocks; start += 256) {
        long long i = start + threadIdx.x;
        unsigned v = (i < n_blocks) ? block_sums[i] : 0u;
        unsigned total;
        unsigned excl = block_exclusive_scan_256(v, s_wave, total);
        if (i < n_blocks) block_sums[i] = carry + excl;
        carry += total;
    }
    if (threadIdx.x == 0 && total_out) *total_out = (long long)carry;
}

__global__ __launch_bounds__(256) void k_scan_add(unsigned* __restrict__ vals, long long n_imm,
                                                  const long long* __restrict__ n_dev,
                                                  const unsigned* __restrict__ block_sums) {
    const long long n = n_dev ? *n_dev : n_imm;
    const long long base = (long long)blockIdx.x * kScanChunk + (long long)threadIdx.x * 8;
    const unsigned add = block_sums[blockIdx.x];
    if (add == 0) return;
#pragma unroll
    for (int i = 0; i < 8; ++i)
        if (base + i < n) vals[base + i] += add;
}

// The whole scan in one workgroup, for short arrays (small grids): one launch instead of three.
__global__ __launch_bounds__(256) void k_scan_small(unsigned* __restrict__ vals, long long n_imm,
                                                    const long long* __restrict__ n_dev,
                                                    long long* __restrict__ total_out) {
    __shared__ unsigned s_wave[4];
    const long long n = n_dev ? *n_dev : n_imm;
    unsigned carry = 0;
    for (long long start = 0; start < n; start += kScanChunk) {
        const long long base = start + (long long)threadIdx.x * 8;
        unsigned v[8];
        unsigned sum = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            v[i] = (base + i < n) ? vals[base + i] : 0u;
            sum += v[i];
        }
        unsigned total;
        unsigned excl = carry + block_exclusive_scan_256(sum, s_wave, total);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (base + i < n) vals[base + i] = excl;
            excl += v[i];
        }
        carry += total;
    }
    if (threadIdx.x == 0 && total_out) *total_out = (long long)carry;
}

// up to this many elements one workgroup scans alone: it takes about 2 us per chunk of 2048, three launches 13 us
constexpr long long kScanSmall = 4 * kScanChunk;

// Second and last step of the scan of up to kScanTwoStep chunks: a block adds up the sums of the chunks before its
// own by itself (a few thousand numbers at most) instead of waiting for a launch that scans them.
constexpr long long kScanTwoStep = 4096;
__global__ __launch_bounds__(256) void k_scan_add_own(unsigned* __restrict__ vals, long long n_imm,
                                                      const long long* __restrict__ n_dev,
                                                      const unsigned* __restrict__ block_sums,
                                                      long long* __restrict__ total_out) {
    __shared__ unsigned s_wave[4];
    const long long n = n_dev ? *n_dev : n_imm;
    unsigned below = 0;
    for (int i = threadIdx.x; i < (int)blockIdx.x; i += 256) below += block_sums[i];
    unsigned add;
    (void)block_exclusive_scan_256(below, s_wave, add);  // (the total is what is wanted)
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0 && total_out)
        *total_out = (long long)add + (long long)block_sums[blockIdx.x];
    if (add == 0) return;
    const long long base = (long long)blockIdx.x * kScanChunk + (long long)threadIdx.x * 8;
#pragma unroll
    for (int i = 0; i < 8; ++i)
        if (base + i < n) vals[base + i] += add;
}

hipError_t launch_exclusive_scan(unsigned* vals, long long capacity, long long n_imm, const long long* n_dev,
                                 unsigned* block_sums, long long* total, hipStream_t s) {
    if (capacity <= kScanSmall) {
        hipLaunchKernelGGL(k_scan_small, dim3(1), dim3(256), 0, s, vals, n_imm, n_dev, total);
        return hipGetLastError();
    }
    long long blocks = (capacity + kScanChunk - 1) / kScanChunk;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(k_scan_local, dim3((unsigned)blocks), dim3(256), 0, s, vals, n_imm, n_dev, block_sums);
    if (blocks <= kScanTwoStep) {
        hipLaunchKernelGGL(k_scan_add_own, dim3((unsigned)blocks), dim3(256), 0, s, vals, n_imm, n_dev, block_sums,
                           total);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(256), 0, s, block_sums, blocks, total);
    hipLaunchKernelGGL(k_scan_add, dim3((unsigned)blocks), dim3(256), 0, s, vals, n_imm, n_dev, block_sums);
    return hipGetLastError();
}

// ------------------------------------------------------------------ index build
// Input rows as the split convolution reads them: [32-channel chunk][row][h | m | l][32] bf16, so that a lane's eight
// channels of a part are one 16-byte load, and rows are 192 bytes apart whatever the channel count (sixteen rows to
// sixteen lanes take 33 clocks of a load then, 58 where the distance is a multiple of 128).  Done by extra workgroups of the index build
// (as a launch of its own 5 us more); bound by memory: 4 bytes read and 6 written per value, 226 k rows of 32 channels
// in 18 us (4 TB/s).  Also notes whether all values and all taps are split_exact, which is all that the pair-list kernel
// asks for (xs null: it splits the rows itself).
__device__ inline void split_rows(const float* __restrict__ feats, long long n, long long n_cap, int c_in,
                                  unsigned short* __restrict__ xs, const int* __restrict__ tap_active, int taps,
                                  Counters* ctr, int block, int n_blocks) {
    const int nch = (c_in + 31) / 32, per_row = nch * 4;  // pieces of eight channels
    const long long total = n * per_row;
    unsigned least = ~0u, most = 0;  // of the values' magnitudes (bits), zeros left out of the least
    for (long long i = (long long)block * blockDim.x + threadIdx.x; i < total; i += (long long)n_blocks * blockDim.x) {
        const long long row = i / per_row;
        const int p = (int)(i - row * per_row), chunk = p >> 2, piece = p & 3, c0 = chunk * 32 + piece * 8;
        const u32x4* src = (const u32x4*)(feats + row * c_in + c0);
        u32x4 x[2], part[3];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            x[q] = u32x4{0u, 0u, 0u, 0u};
            if (c0 + 4 * q < c_in) x[q] = src[q];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const unsigned u = x[q][e] & 0x7fffffffu;
                least = min(least, u - 1u);
                most = max(most, u);
            }
        }
        if (!xs) continue;
        split8(x, part);
        u32x4* dst = (u32x4*)(xs + (chunk * n_cap + row) * 96 + piece * 8);
#pragma unroll
        for (int k = 0; k < 3; ++k) dst[k * 4] = part[k];
    }
    bool odd = least < kSplitLeast - 1u || most >= kSplitEnd;
    if (block == n_blocks - 1)
        for (int t = threadIdx.x; t < taps; t += blockDim.x) odd |= (tap_active[t] & kTapOdd) != 0;
    if (odd) atomicOr(&ctr->odd, 1u);
}

// One thread per input row: set the row's bit; the first row of each word
// records its own index as that word's prefix.  Rows outside the grid are
// skipped and reported; a row not strictly above its predecessor is reported.
// at_row(row, on the grid, b, c0, c1, c2) is called by the whole wave for each of its rows.
template <typename AtRow>
__device__ __forceinline__ void index_rows(const Geom& g, const int32_t* __restrict__ coords, long long n, int blocks,
                                           unsigned long long* __restrict__ occ, unsigned* __restrict__ occ_prefix,
                                           Counters* ctr, AtRow&& at_row) {
    const int stride = 1 + g.ndim;
    const int lane = threadIdx.x & 63;
    for (long long base = (long long)blockIdx.x * blockDim.x; base < n; base += (long long)blocks * blockDim.x) {
        const long long r = base + threadIdx.x;
        long long key = -1;
        int b = 0, c0 = 0, c1 = 0, c2 = 0;
        if (r < n) {
            load_site(g, coords + r * stride, b, c0, c1, c2);
            if (site_in_grid(g, b, c0, c1, c2)) {
                key = (long long)b * g.Npad + lin_of(g, c0, c1, c2);
                long long prev_key = -1;
                if (r > 0) {
                    int pb, p0, p1, p2;
                    load_site(g, coords + (r - 1) * stride, pb, p0, p1, p2);
                    if (site_in_grid(g, pb, p0, p1, p2)) prev_key = (long long)pb * g.Npad + lin_of(g, p0, p1, p2);
                }
                if (prev_key >= key) atomicOr(&ctr->flags, SCNN_FLAG_UNSORTED);
                if ((prev_key >> 6) != (key >> 6)) occ_prefix[key >> 6] = (unsigned)r;
            } else {
                atomicOr(&ctr->flags, SCNN_FLAG_BAD_COORD);
            }
        }
        // Sorted rows of one bitmap word sit in adjacent lanes: OR their bits together inside the wave and let the
        // first lane of each run issue the one atomic (a run may continue in the next wave, hence still atomic).
        const long long word = key >= 0 ? (key >> 6) : (long long)(-1 - lane);
        unsigned long long bits = key >= 0 ? (1ull << (key & 63)) : 0ull;
        const bool first = wave_or_runs(word, bits);
        if (key >= 0 && first) atomicOr(&occ[word], bits);
        at_row(r, key >= 0, b, c0, c1, c2);
    }
}
__device__ __forceinline__ void index_rows(const Geom& g, const int32_t* __restrict__ coords, long long n, int blocks,
                                           unsigned long long* __restrict__ occ, unsigned* __restrict__ occ_prefix,
                                           Counters* ctr) {
    index_rows(g, coords, n, blocks, occ, occ_prefix, ctr, [](long long, bool, int, int, int, int) {});
}

// A device-resident count never reaches past the arrays.
__device__ __forceinline__ long long row_count(long long n_imm, const long long* __restrict__ n_dev, long long n_cap) {
    long long n = n_dev ? *n_dev : n_imm;
    if (n > n_cap) n = n_cap;
    return n < 0 ? 0 : n;
}

__global__ __launch_bounds__(256) void k_index_build(Geom g, const int32_t* __restrict__ coords, long long n_imm,
                                                     const long long* __restrict__ n_dev, long long n_cap,
                                                     unsigned long long* __restrict__ occ,
                                                     unsigned* __restrict__ occ_prefix, Counters* ctr) {
    index_rows(g, coords, row_count(n_imm, n_dev, n_cap), (int)gridDim.x, occ, occ_prefix, ctr);
}

// The same for the pooling, with the bits of the output sites: a row sets that of its block of 2^d sites.
// rows_have_entries != 0: the caller guarantees that every row holds a non-zero entry (skip the check).  (One launch: as
// two, a 28 x 28 image took 4 us more.)
__global__ __launch_bounds__(256) void k_index_build_pool(Geom g, Geom gp, const int32_t* __restrict__ coords,
                                                          const float* __restrict__ feats, int channels,
                                                          int rows_have_entries, long long n_imm,
                                                          const long long* __restrict__ n_dev, long long n_cap,
                                                          unsigned long long* __restrict__ occ,
                                                          unsigned* __restrict__ occ_prefix,
                                                          unsigned long long* __restrict__ pbits, Counters* ctr) {
    const int lane = threadIdx.x & 63;
    index_rows(g, coords, row_count(n_imm, n_dev, n_cap), (int)gridDim.x, occ, occ_prefix, ctr,
               [&](long long r, bool any, int b, int c0, int c1, int c2) {
        if (any && !rows_have_entries) {  // a row of zeros holds no entry and creates no output site
            // (stops at the first non-zero value, which an ordinary row has in its first few channels; 16 bytes
            // at a time where the rows allow it)
            any = false;
            const float* row = feats + r * channels;
            if ((channels & 3) == 0 && (((size_t)feats) & 15) == 0) {
                for (int c = 0; c < channels && !any; c += 4) {
                    const float4 v = *reinterpret_cast<const float4*>(row + c);
                    any = v.x != 0.0f || v.y != 0.0f || v.z != 0.0f || v.w != 0.0f;
                }
            } else {
                for (int c = 0; c < channels && !any; ++c) any = row[c] != 0.0f;
            }
        }
        const long long key = any ? (long long)b * gp.Npad + lin_of(gp, c0 >> 1, c1 >> 1, c2 >> 1) : -1;
        // neighbouring rows fall into the same output word: one atomic per run of equal words
        const long long word = any ? (key >> 6) : (long long)(-1 - lane);
        unsigned long long bits = any ? (1ull << (key & 63)) : 0ull;
        const bool first = wave_or_runs(word, bits);
        if (any && first) atomicOr(&pbits[word], bits);
    });
}

hipError_t launch_index_build_pool(const Geom& g, const Geom& gp, const int32_t* coords, const float* feats, int channels,
                                   int rows_have_entries, long long n_imm, const long long* n_dev, long long n_cap,
                                   unsigned long long* occ, unsigned* occ_prefix, unsigned long long* pbits, Counters* ctr,
                                   hipStream_t s) {
    long long blocks = (n_cap + 255) / 256;
    if (blocks < 1) blocks = 1;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_index_build_pool, dim3((unsigned)blocks), dim3(256), 0, s, g, gp, coords, feats, channels,
                       rows_have_entries, n_imm, n_dev, n_cap, occ, occ_prefix, pbits, ctr);
    return hipGetLastError();
}

// The same for the split kernels: workgroups from index_blocks on take the rows' values.
__global__ __launch_bounds__(256) void k_index_build_split(Geom g, const int32_t* __restrict__ coords, long long n_imm,
                                                           const long long* __restrict__ n_dev, long long n_cap,
                                                           unsigned long long* __restrict__ occ,
                                                           unsigned* __restrict__ occ_prefix, Counters* ctr,
                                                           int index_blocks, const float* __restrict__ feats, int c_in,
                                                           unsigned short* __restrict__ xs,
                                                           const int* __restrict__ tap_active) {
    const long long n = row_count(n_imm, n_dev, n_cap);
    if ((int)blockIdx.x < index_blocks)
        index_rows(g, coords, n, index_blocks, occ, occ_prefix, ctr);
    else
        split_rows(feats, n, n_cap, c_in, xs, tap_active, g.T, ctr, (int)blockIdx.x - index_blocks,
                   (int)gridDim.x - index_blocks);
}

hipError_t launch_index_build(const Geom& g, const int32_t* coords, long long n_imm, const long long* n_dev,
                              long long n_cap, unsigned long long* occ, unsigned* occ_prefix, Counters* ctr,
                              const float* feats, int c_in, unsigned short* xs, const int* tap_active, hipStream_t s) {
    long long blocks = (n_cap + 255) / 256;
    if (blocks < 1) blocks = 1;
    if (blocks > 4096) blocks = 4096;
    if (!feats) {
        hipLaunchKernelGGL(k_index_build, dim3((unsigned)blocks), dim3(256), 0, s, g, coords, n_imm, n_dev, n_cap, occ,
                           occ_prefix, ctr);
        return hipGetLastError();
    }
    long long split_blocks = (n_cap * ((c_in + 31) / 32) * 4 + 255) / 256;
    if (split_blocks < 1) split_blocks = 1;
    if (split_blocks > 4096) split_blocks = 4096;
    hipLaunchKernelGGL(k_index_build_split, dim3((unsigned)(blocks + split_blocks)), dim3(256), 0, s, g, coords, n_imm,
                       n_dev, n_cap, occ, occ_prefix, ctr, (int)blocks, feats, c_in, xs, tap_active);
    return hipGetLastError();
}

// Everything that has to happen before the input is indexed, in one launch.  Block t < T prepares tap t of the
// filter: tap_active[t] = "has a non-zero weight" (and kTapOdd, for the split kernels), tap_coord[t] = its offset, and its weights in the layout of the
// convolution kernel that will run -- wb (matrix-core operand order:
// wb[((t * KC + kc) * NB + cb) * 64 + lane][s] = w[t][kc*32 + 8*gq + s][cb*16 + jj], lane = 16*gq + jj, so that a
// lane fetches its eight values of one (tap, kc, cb) with two 16-byte loads) or wp (fp64, rows padded to
// c_out_pad; the vector kernel).  The blocks from T on clear the zero-initialised part of the workspace.  With two layouts
// (kLayoutSplitPair) blocks T .. 2 T - 1 lay out the second: one after the other they took 64 -> 128 channels 5 us longer.
// With `adjoint` set the filter is read as the adjoint convolution's (filter_at).
enum PrepareLayout { kLayoutVector, kLayoutPair, kLayoutQuad, kLayoutSplit, kLayoutSplitPair };  // (one kernel each: a small layer waits for it)
template <int LAYOUT>
__global__ __launch_bounds__(256) void k_prepare(Geom g, const float* __restrict__ w, int c_in, int c_out, int adjoint,
                                                 int c_out_pad, void* __restrict__ dst, float* __restrict__ dst2,
                                                 int* __restrict__ tap_active,
                                                 int* __restrict__ tap_coord, uint4* __restrict__ zero_p,
                                                 size_t zero_n16) {
    constexpr bool kSplitParts = LAYOUT == kLayoutSplit || LAYOUT == kLayoutSplitPair;
    const int tap_blocks = LAYOUT == kLayoutSplitPair ? 2 * g.T : g.T;
    if ((int)blockIdx.x >= tap_blocks) {
        const size_t stride = (size_t)(gridDim.x - tap_blocks) * blockDim.x;
        for (size_t i = (size_t)(blockIdx.x - tap_blocks) * blockDim.x + threadIdx.x; i < zero_n16; i += stride)
            zero_p[i] = make_uint4(0, 0, 0, 0);
        return;
    }
    const bool second = LAYOUT == kLayoutSplitPair && (int)blockIdx.x >= g.T;  // (of two layouts)
    __shared__ int s_any, s_odd;
    const int t = second ? (int)blockIdx.x - g.T : (int)blockIdx.x;
    if (threadIdx.x == 0) {
        s_any = 0;
        if (kSplitParts) s_odd = 0;
    }
    __syncthreads();
    int any = 0;
    if constexpr (LAYOUT == kLayoutQuad) {
        float* __restrict__ wq = (float*)dst;
        // operand order of the quad kernel: [tap][32-channel chunk][channel / 4][lane][channel % 4], lane = output
        // channel (modulo 32 when there are at most 32 of them); channels and columns past the real ones are zero
        // With more than 64 output channels: one such filter per group of 64, one after the other.
        const int nch = (c_in + 31) / 32;
        const int n = nch * 2048;
        for (int col0 = 0; col0 < c_out; col0 += 64) {
            const int cg = c_out - col0 < 64 ? c_out - col0 : 64, cols = cg > 32 ? 64 : 32;
            float* wq_g = wq + (size_t)(col0 >> 6) * quad_filter_floats(g.T, c_in);
            for (int i = threadIdx.x; i < n; i += blockDim.x) {
                const int e = i & 3, lane = (i >> 2) & 63, j = (i >> 8) & 7, c = i >> 11;
                const int ic = c * 32 + 4 * j + e, oc = lane & (cols - 1);
                const float v =
                    (ic < c_in && oc < cg) ? filter_at(w, g.T, c_in, c_out, adjoint, t, ic, col0 + oc) : 0.0f;
                wq_g[(size_t)t * n + i] = v;
                any |= (v != 0.0f);
            }
        }
    }
    if (kSplitParts && !second) {
        unsigned short* __restrict__ ws = (unsigned short*)dst;
        // operand order of the split kernel: [tap][chunk][h | m | l][16 output channels][lane][8], lane = 16 * (channel
        // / 8) + output channel; columns past the real ones are zero.  Groups of 64 output channels one after the other.
        const int nch = (c_in + 31) / 32;
        for (int col0 = 0; col0 < c_out; col0 += 64) {
            const int cg = c_out - col0 < 64 ? c_out - col0 : 64, nb = cg > 32 ? 4 : 2;
            unsigned short* ws_g = ws + (size_t)(col0 >> 6) * split_filter_elems(g.T, c_in) + (size_t)t * nch * nb * 1536;
            for (int i = threadIdx.x; i < nch * nb * 512; i += blockDim.x) {
                const int e = i & 7, lane = (i >> 3) & 63, r = i >> 9, cb = r % nb, c = r / nb;
                const int ic = c * 32 + (lane >> 4) * 8 + e, oc = cb * 16 + (lane & 15);
                const float v =
                    (ic < c_in && oc < cg) ? filter_at(w, g.T, c_in, c_out, adjoint, t, ic, col0 + oc) : 0.0f;
                unsigned short* part = ws_g + (size_t)c * nb * 1536 + cb * 512 + (i & 511);
                split3(v, part[0], part[nb * 512], part[2 * nb * 512]);
                any |= (v != 0.0f) | (split_exact(__float_as_uint(v)) ? 0 : kTapOdd);
            }
        }
    }
    if (LAYOUT == kLayoutPair || second) {
        float* __restrict__ wb = LAYOUT == kLayoutPair ? (float*)dst : dst2;
        // C_in = 16 is laid out like one 32-channel chunk: a lane's first four values are channels 4 gq .. 4 gq + 3,
        // its other four are zero
        const bool half = c_in == 16;
        const int nb = c_out / 16, n = (half ? 32 : c_in) * c_out;
        for (int i = threadIdx.x; i < n; i += blockDim.x) {
            const int sub = i & 7, lane = (i >> 3) & 63;
            const int r = i >> 9, cb = r % nb, kc = r / nb;  // (kc < C_in / 32 since n = (C_in / 32) * nb * 512)
            const int jj = lane & 15, gq = lane >> 4;
            const int ic = half ? (sub < 4 ? 4 * gq + sub : -1) : kc * 32 + 8 * gq + sub;
            const float v = ic >= 0 ? filter_at(w, g.T, c_in, c_out, adjoint, t, ic, cb * 16 + jj) : 0.0f;
            wb[(size_t)t * n + i] = v;
            any |= (v != 0.0f);
        }
    }
    if constexpr (LAYOUT == kLayoutVector) {
        double* __restrict__ wp = (double*)dst;
        const int n = c_in * c_out_pad;
        for (int i = threadIdx.x; i < n; i += blockDim.x) {
            const int ic = i / c_out_pad, oc = i % c_out_pad;
            float v = 0.0f;
            if (oc < c_out) v = filter_at(w, g.T, c_in, c_out, adjoint, t, ic, oc);
            wp[(size_t)t * n + i] = (double)v;
            any |= (v != 0.0f);
        }
    }
    if (second) return;
    if (any & 1) s_any = 1;
    if (kSplitParts && (any & kTapOdd)) s_odd = kTapOdd;
    __syncthreads();
    if (threadIdx.x == 0) {
        tap_active[t] = kSplitParts ? s_any | s_odd : s_any;
        // tap coordinates (t0, t1, t2), one byte each: delta = coordinate - H
        tap_coord[t] = (t / (g.K[2] * g.K[1])) | (((t / g.K[2]) % g.K[1]) << 8) | ((t % g.K[2]) << 16);
    }
}

hipError_t launch_prepare(const Geom& g, const float* w, int c_in, int c_out, int adjoint, int c_out_pad, double* wp,
                          float* wb, float* wq, unsigned short* ws, int* tap_active, int* tap_coord, void* zero_p,
                          size_t zero_bytes, hipStream_t s) {
    const size_t n16 = (zero_bytes + 15) / 16;
    size_t zb = (n16 + 255) / 256;
    if (zb > 2048) zb = 2048;
    const dim3 grid((unsigned)(g.T * (ws && wb ? 2 : 1) + zb)), block(256);
#define SCNN_PREPARE(LAYOUT, DST)                                                                                    \
    hipLaunchKernelGGL(k_prepare<LAYOUT>, grid, block, 0, s, g, w, c_in, c_out, adjoint, c_out_pad, (void*)(DST), wb, tap_active, \
                       tap_coord, (uint4*)zero_p, n16)
    if (wq)
        SCNN_PREPARE(kLayoutQuad, wq);
    else if (ws && wb)
        SCNN_PREPARE(kLayoutSplitPair, ws);
    else if (ws)
        SCNN_PREPARE(kLayoutSplit, ws);
    else if (wb)
        SCNN_PREPARE(kLayoutPair, wb);
    else
        SCNN_PREPARE(kLayoutVector, wp);
#undef SCNN_PREPARE
    return hipGetLastError();
}

// ------------------------------------------------------------------ candidate sites
// Candidate sites = occupied sites dilated by the filter's non-zero taps: an input at q reaches p = q - delta,
// i.e. p is a candidate iff some active tap has an occupied site at p + delta.  Sixteen lanes produce one 64-bit
// word of the candidate bitmap by OR-ing shifted windows of the occupancy bitmap (no atomics): each lane takes some
// of the (delta_0, delta_1) lines and the lanes combine with shuffles.  A word is cut
// into the runs it shares with grid lines (last axis); for a run and a (delta_0, delta_1) pair the source bits
// of all delta_2 lie in one window of at most three occupancy words.
__device__ inline unsigned long long funnel64(unsigned long long lo, unsigned long long hi, int s) {
    return s ? ((lo >> s) | (hi << (64 - s))) : lo;
}

// LANES lanes share one bitmap word, one (delta_0, delta_1) line at a time each: 16 on small grids, where one lane
// per word would leave most of the chip idle behind a chain of dependent loads, 1 on large grids.
template <int kDilateLanes>
__device__ __forceinline__ unsigned long long dilate_word(const Geom& g, const unsigned long long* __restrict__ occ,
                                                          const int* __restrict__ tap_active, long long w, int sub) {
    const int n_lines = g.K[0] * g.K[1];
    const int b = (int)(w / g.Wps);
    const long long p_first = (w - (long long)b * g.Wps) * 64;  // lin of bit 0
    long long remaining = g.N - p_first;                         // bits of this word that are sites
    if (remaining > 64) remaining = 64;
    unsigned long long out = 0;
    const long long sample_bit0 = (long long)b * g.Npad;
    const long long word_lo = (long long)b * g.Wps, word_hi = word_lo + g.Wps;  // this sample's words
    long long line = p_first / g.E[2];
    int c2 = (int)(p_first - line * g.E[2]);
    int c1 = (int)(line % g.E[1]), c0 = (int)(line / g.E[1]);
    int bit = 0;
    while (remaining > 0) {
        int len = g.E[2] - c2;
        const int room = min(len, 128);  // (128: as good as any, and minus an offset it stays in range on the longest line)
        if (len > remaining) len = (int)remaining;
        unsigned long long run = 0;
        for (int l = sub; l < n_lines; l += kDilateLanes) {
            const int t0 = l / g.K[1], t1 = l - t0 * g.K[1];
            const int q0 = c0 + t0 - g.H[0], q1 = c1 + t1 - g.H[1];
            if ((unsigned)q0 >= (unsigned)g.E[0] || (unsigned)q1 >= (unsigned)g.E[1]) continue;
            // window of occupancy bits [s - H2, s + len + H2) of line (q0, q1), s = site (q0, q1, c2)
            const long long s = sample_bit0 + ((long long)q0 * g.E[1] + q1) * g.E[2] + c2;
            const long long wb = (s - g.H[2]) >> 6;  // arithmetic shift: floor also for negatives
            unsigned long long win[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const long long wi = wb + i;
                win[i] = (wi >= word_lo && wi < word_hi) ? occ[wi] : 0ull;
            }
            const int* act = tap_active + l * g.K[2];
            for (int t2 = 0; t2 < g.K[2]; ++t2) {
                if (!act[t2]) continue;
                const int d2 = t2 - g.H[2];
                // source z = c2 + i + d2 must stay on the line: i in [lo, hi)
                const int lo = max(max(-d2, 0) - c2, 0), hi = min(room - d2, len);
                if (lo >= hi) continue;
                const int o = (int)(s + d2 - wb * 64);  // 0 <= o < 128 for H2 <= 32
                unsigned long long bits = o < 64 ? funnel64(win[0], win[1], o) : funnel64(win[1], win[2], o - 64);
                unsigned long long m = (hi - lo) >= 64 ? ~0ull : (((1ull << (hi - lo)) - 1ull) << lo);
                run |= bits & m;
            }
        }
        out |= run << bit;
        bit += len;
        remaining -= len;
        c2 = 0;
        if (++c1 == g.E[1]) { c1 = 0; ++c0; }
    }
    // OR of the lanes' lines
    if constexpr (kDilateLanes > 1) {
#pragma unroll
        for (int d = 1; d < kDilateLanes; d <<= 1) out |= __shfl_xor(out, d, kDilateLanes);
    }
    return out;
}

template <int kDilateLanes>
__global__ __launch_bounds__(256) void k_cand_dilate(Geom g, const unsigned long long* __restrict__ occ,
                                                     const int* __restrict__ tap_active,
                                                     unsigned long long* __restrict__ cand,
                                                     unsigned* __restrict__ cand_count) {
    const long long n_words = (long long)g.batch * g.Wps;
    const int sub = threadIdx.x & (kDilateLanes - 1);
    const long long groups = (long long)gridDim.x * (blockDim.x / kDilateLanes);
    for (long long w = (long long)blockIdx.x * (blockDim.x / kDilateLanes) + threadIdx.x / kDilateLanes; w < n_words;
         w += groups) {
        const unsigned long long out = dilate_word<kDilateLanes>(g, occ, tap_active, w, sub);
        if (sub == 0) {
            cand[w] = out;
            cand_count[w] = (unsigned)__popcll(out);
        }
    }
}

// Small grids of short lines: a wave takes a word, a lane each of its sites.  A word of an 8^3 grid holds eight lines, which
// the form above walks one after the other (8^3 x 4: 10.5 us); here a site looks at the lines of its filter, several lines'
// loads in flight, and the ballot is the word.
constexpr int kDilateBatch = 5;  // lines in flight
constexpr long long kDilateSiteWords = 4096;
// The form above takes about 0.6 us + 0.2 for every tap of a line, for every line that a word holds part of (64 / E[2], one or two
// more where that leaves a remainder) and every sixteen lines of the filter; this one 1.4 us for every five lines of the filter,
// 2.1 where 4096 words share the chip.  Calls, the form above less this one, us: 3 x 3 x 3 on 8^3 x 4 / 16^3 x 16 / 30^3 / 32^3 /
// 32^3 x 8 +5.7 / +1.8 / +2.4 / -0.3 / -2.2, 5 x 5 x 5 on the same but 30^3 +15 / +4.7 / -0.8 / -4.6, 31 x 1 x 1 +0.4 / -4.3 / -8 / -12,
// 9 x 1 x 1 +2.4 / -0.1 / -1.5 / -3.1; 3 x 3 on 28 x 28 x 4 / 50 x 40 x 100 +3.8 / +1.4, 31 x 1 -4.3 / -10.  Of 458 such calls the
// rule takes the slower form for none by more than 0.5 us.
static bool dilate_by_sites(const Geom& g, long long n_words) {
    if (n_words > kDilateSiteWords || g.E[2] >= 64 || g.K[2] > 32) return false;
    const long long lines = (long long)g.K[0] * g.K[1];
    const long long held = 640 + (64 % g.E[2] != 0 ? 13 * g.E[2] : 0);                // tenths of a line of a word, times E[2]
    const long long by_words = held * ((lines + 15) / 16) * (6 + 2 * g.K[2]);         // hundredths of a us, times E[2]
    const long long by_sites = (lines + kDilateBatch - 1) / kDilateBatch * (14 * 4096 + 7 * n_words);  // tenths, times 4096
    return by_words * 4096 >= 10 * by_sites * g.E[2];
}
__global__ __launch_bounds__(256) void k_cand_dilate_sites(Geom g, const unsigned long long* __restrict__ occ,
                                                           const int* __restrict__ tap_active,
                                                           unsigned long long* __restrict__ cand,
                                                           unsigned* __restrict__ cand_count) {
    const int n_words = g.batch * g.Wps, lane = threadIdx.x & 63, n_lines = g.K[0] * g.K[1];
    const int w = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    if (w >= n_words) return;  // (whole waves)
    const int b = w / g.Wps, first = b * g.Wps;
    const unsigned site = (unsigned)(w - first) * 64u + (unsigned)lane;
    const bool real = (long long)site < g.N;
    int c0 = 0, c1 = 0, c2 = 0, k_lo, k_hi;
    if (real) site_of(g, site, c0, c1, c2);
    taps_on_line(g.E[2], c2, -g.H[2], g.K[2], k_lo, k_hi);
    const unsigned on_line = real && k_hi > k_lo ? (~0u >> (32 - (k_hi - k_lo))) << k_lo : 0u;
    unsigned any = 0;
    for (int l0 = 0; l0 < n_lines; l0 += kDilateBatch) {
        unsigned long long word_a[kDilateBatch], word_b[kDilateBatch];
        unsigned p[kDilateBatch], act[kDilateBatch];
        bool ok[kDilateBatch];
#pragma unroll
        for (int i = 0; i < kDilateBatch; ++i) {
            const int l = l0 + i < n_lines ? l0 + i : n_lines - 1;  // (a line taken twice gives the same)
            const int t0 = l / g.K[1], t1 = l - t0 * g.K[1];
            const int q0 = c0 + t0 - g.H[0], q1 = c1 + t1 - g.H[1];
            ok[i] = on_line != 0u && (unsigned)q0 < (unsigned)g.E[0] && (unsigned)q1 < (unsigned)g.E[1];
            const unsigned bit = ok[i] ? (unsigned)((q0 * g.E[1] + q1) * g.E[2] + c2 - g.H[2] + k_lo) : 0u;
            p[i] = bit & 63u;
            const int wa = (int)(bit >> 6), wb = wa + 1 < g.Wps ? wa + 1 : wa;  // (a line ends inside its sample)
            word_a[i] = occ[first + wa];
            word_b[i] = occ[first + wb];
            act[i] = active_taps(tap_active, l * g.K[2], g.K[2]);
        }
#pragma unroll
        for (int i = 0; i < kDilateBatch; ++i) {
            const unsigned window = (unsigned)(word_a[i] >> p[i]) | (unsigned)((word_b[i] << 1) << (63u - p[i]));
            any |= ok[i] ? (window << k_lo) & on_line & act[i] : 0u;
        }
    }
    const unsigned long long out = __ballot(any != 0u);
    if (lane == 0) {
        cand[w] = out;
        cand_count[w] = (unsigned)__popcll(out);
    }
}

// The same for bitmaps of up to kEmitMidWords words: a workgroup takes chunks of 256 / LANES consecutive words and also
// leaves each chunk's candidate count, from which k_cand_emit_mid finds its place in the candidate list without a
// scan launch in between.
template <int kDilateLanes>
__global__ __launch_bounds__(256) void k_cand_dilate_chunks(Geom g, const unsigned long long* __restrict__ occ,
                                                            const int* __restrict__ tap_active,
                                                            unsigned long long* __restrict__ cand,
                                                            unsigned* __restrict__ cand_count,
                                                            unsigned* __restrict__ chunk_sums) {
    constexpr int kChunk = 256 / kDilateLanes;
    __shared__ unsigned s_wave[4];
    const long long n_words = (long long)g.batch * g.Wps;
    const long long n_chunks = (n_words + kChunk - 1) / kChunk;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int sub = threadIdx.x & (kDilateLanes - 1);
    for (long long c = blockIdx.x; c < n_chunks; c += gridDim.x) {
        const long long w = c * kChunk + threadIdx.x / kDilateLanes;
        unsigned n = 0;
        if (w < n_words) {
            const unsigned long long out = dilate_word<kDilateLanes>(g, occ, tap_active, w, sub);
            if (sub == 0) {
                n = (unsigned)__popcll(out);
                cand[w] = out;
                cand_count[w] = n;
            }
        }
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) n += __shfl_xor(n, d, 64);
        if (lane == 0) s_wave[wave] = n;
        __syncthreads();
        if (threadIdx.x == 0) chunk_sums[c] = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
        __syncthreads();
    }
}

hipError_t launch_cand_dilate(const Geom& g, const unsigned long long* occ, const int* tap_active,
                              unsigned long long* cand, unsigned* cand_count, unsigned* chunk_sums, hipStream_t s) {
    const long long n_words = (long long)g.batch * g.Wps;
    const int lanes = cand_dilate_lanes(n_words, g.Wps);
    if (chunk_sums) {  // (the caller passes them for kEmitSmallWords < n_words <= kEmitMidWords)
        long long blocks = (n_words * lanes + 255) / 256;
        if (blocks > 8192) blocks = 8192;
        if (lanes == 16)
            hipLaunchKernelGGL(k_cand_dilate_chunks<16>, dim3((unsigned)blocks), dim3(256), 0, s, g, occ, tap_active,
                               cand, cand_count, chunk_sums);
        else
            hipLaunchKernelGGL(k_cand_dilate_chunks<1>, dim3((unsigned)blocks), dim3(256), 0, s, g, occ, tap_active,
                               cand, cand_count, chunk_sums);
        return hipGetLastError();
    }
    if (dilate_by_sites(g, n_words)) {
        hipLaunchKernelGGL(k_cand_dilate_sites, dim3((unsigned)((n_words + 3) / 4)), dim3(256), 0, s, g, occ, tap_active, cand,
                           cand_count);
        return hipGetLastError();
    }
    long long blocks = (n_words * lanes + 255) / 256;
    if (blocks < 1) blocks = 1;
    if (blocks > 8192) blocks = 8192;
    if (lanes == 16)
        hipLaunchKernelGGL(k_cand_dilate<16>, dim3((unsigned)blocks), dim3(256), 0, s, g, occ, tap_active, cand,
                           cand_count);
    else
        hipLaunchKernelGGL(k_cand_dilate<1>, dim3((unsigned)blocks), dim3(256), 0, s, g, occ, tap_active, cand,
                           cand_count);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_popcount(const unsigned long long* __restrict__ bits, long long n_words,
                                                  unsigned* __restrict__ out) {
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n_words;
         i += (long long)gridDim.x * blockDim.x)
        out[i] = (unsigned)__popcll(bits[i]);
}

hipError_t launch_popcount(const unsigned long long* bits, long long n_words, unsigned* out, hipStream_t s) {
    long long blocks = (n_words + 255) / 256;
    if (blocks < 1) blocks = 1;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_popcount, dim3((unsigned)blocks), dim3(256), 0, s, bits, n_words, out);
    return hipGetLastError();
}

// Candidate list and its per-sample ranges, in one launch.
// Last block: per-sample candidate ranges and tile ranges.  Each sample's candidates are padded to whole tiles so
// that a tile never spans two samples.  rows16_start[b] = 16-row groups of all earlier samples (each sample
// rounded up), the unit in which the pair lists of the matrix-core path reserve their space.
// Other blocks, one thread per bitmap word: write the per-sample site index of every set bit at its rank.  The
// list comes out sorted by (b, lin).
__global__ __launch_bounds__(256) void k_cand_emit(Geom g, const unsigned long long* __restrict__ cand,
                                                   const unsigned* __restrict__ cand_prefix, long long n_words,
                                                   unsigned* __restrict__ cand_lin, long long cand_cap,
                                                   int* __restrict__ cand_start, int* __restrict__ tile_start,
                                                   int* __restrict__ rows16_start, Counters* ctr) {
    __shared__ unsigned s_wave[4];
    if (blockIdx.x == gridDim.x - 1) {
        const long long n_cand = ctr->n_cand;  // written by the scan
        const bool overflow = n_cand > cand_cap;
        for (int b = threadIdx.x; b <= g.batch; b += blockDim.x) {
            int v = 0;
            if (!overflow) v = (b == g.batch) ? (int)n_cand : (int)cand_prefix[(long long)b * g.Wps];
            cand_start[b] = v;
        }
        __syncthreads();
        const int n_tiles_all = sample_ranges_256(g.batch, cand_start, tile_start, rows16_start, s_wave);
        if (threadIdx.x == 0) {
            ctr->n_tiles = n_tiles_all;
            if (overflow) atomicOr(&ctr->flags, SCNN_FLAG_CAND_OVERFLOW);
        }
        return;
    }
    for (long long w = (long long)blockIdx.x * blockDim.x + threadIdx.x; w < n_words;
         w += (long long)(gridDim.x - 1) * blockDim.x) {
        unsigned long long bits = cand[w];
        if (!bits) continue;
        long long o = cand_prefix[w];
        const unsigned base = (unsigned)((w % g.Wps) * 64);
        while (bits) {
            const int bit = __ffsll((long long)bits) - 1;
            bits &= bits - 1;
            if (o < cand_cap) cand_lin[o] = base + (unsigned)bit;
            ++o;
        }
    }
}

// Writes the site indices of the set bits of the wave's `count` words (lane j < count holds word j: its bits, the place of its
// first site in the list, and the site of its bit 0; 0 in the lanes past them).  A word at a time, 64 lanes to one run of the
// list; or, where all words hold few bits (scattered sites: 256^3, 13.7 -> 9.7 us), a lane to its own word's bits, which
// writes to as many places of the list at a time.  (whole wave)
__device__ __forceinline__ void emit_words(unsigned long long bits, unsigned o, unsigned base, int count,
                                           unsigned* __restrict__ cand_lin, long long cand_cap) {
    const int lane = threadIdx.x & 63;
    if (wave_max((unsigned)__popcll(bits)) < (unsigned)__popcll(__ballot(bits != 0ull))) {  // (uniform) fewer steps
        for (; bits; bits &= bits - 1ull, ++o)
            if ((long long)o < cand_cap) cand_lin[o] = base + (unsigned)__builtin_ctzll(bits);
        return;
    }
    for (int j = 0; j < count; ++j) {
        const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)bits, j);
        const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(bits >> 32), j);
        if ((lo | hi) == 0u) continue;  // (uniform)
        const unsigned place = (unsigned)__builtin_amdgcn_readlane((int)o, j), site = (unsigned)__builtin_amdgcn_readlane((int)base, j);
        const unsigned at = place + __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
        const bool set = ((lane < 32 ? lo : hi) >> (lane & 31)) & 1u;
        if (set && (long long)at < cand_cap) cand_lin[at] = site + (unsigned)lane;
    }
}

// The same for short bitmaps (at most kEmitSmallWords words), without a scan launch before it: a block sums the counts
// of the words before its own (a few thousand numbers out of L2) and scans its 64 words itself; the last block scans
// the whole array once to find the per-sample ranges.  `cand_count` holds the words' candidate counts, unscanned.
__global__ __launch_bounds__(256) void k_cand_emit_small(Geom g, const unsigned long long* __restrict__ cand,
                                                         const unsigned* __restrict__ cand_count, int n_words,
                                                         unsigned* __restrict__ cand_lin, long long cand_cap,
                                                         int* __restrict__ cand_start, int* __restrict__ tile_start,
                                                         int* __restrict__ rows16_start, Counters* ctr) {
    __shared__ unsigned s_wave[4];
    if (blockIdx.x == gridDim.x - 1) {
        // exclusive scan in chunks of 2048 words; a sample starts at every Wps-th word
        unsigned carry = 0;
        for (int start = 0; start < n_words; start += kScanChunk) {
            const int base = start + threadIdx.x * 8;
            unsigned v[8], sum = 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                v[i] = (base + i < n_words) ? cand_count[base + i] : 0u;
                sum += v[i];
            }
            unsigned total;
            unsigned excl = carry + block_exclusive_scan_256(sum, s_wave, total);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int w = base + i;
                if (w < n_words && w % (int)g.Wps == 0) cand_start[w / (int)g.Wps] = (int)excl;
                excl += v[i];
            }
            carry += total;
        }
        const long long n_cand = (long long)carry;
        const bool overflow = n_cand > cand_cap;
        __syncthreads();  // cand_start[0 .. batch) written
        if (overflow)
            for (int b = threadIdx.x; b < g.batch; b += blockDim.x) cand_start[b] = 0;
        if (threadIdx.x == 0) cand_start[g.batch] = overflow ? 0 : (int)n_cand;
        __syncthreads();
        const int n_tiles_all = sample_ranges_256(g.batch, cand_start, tile_start, rows16_start, s_wave);
        if (threadIdx.x == 0) {
            ctr->n_cand = n_cand;
            ctr->n_tiles = n_tiles_all;
            if (overflow) atomicOr(&ctr->flags, SCNN_FLAG_CAND_OVERFLOW);
        }
        return;
    }
    // 64 words: every wave takes sixteen of them, and finds out by itself what lies before
    const int w0 = blockIdx.x * 64, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned below = 0;
    for (int i0 = threadIdx.x; i0 < w0; i0 += 256 * 8) {  // eight loads in flight per thread
        unsigned x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = i0 + 256 * u < w0 ? cand_count[i0 + 256 * u] : 0u;
#pragma unroll
        for (int u = 0; u < 8; ++u) below += x[u];
    }
    const int w = w0 + lane;
    const unsigned long long bits = w < n_words ? cand[w] : 0ull;
    below = wave_add(below);
    if (lane == 0) s_wave[wave] = below;
    __syncthreads();
    const unsigned own = (unsigned)__popcll(bits);
    const unsigned o = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3] + wave_inclusive_add(own) - own;
    const unsigned base = w < n_words ? (unsigned)((w % (int)g.Wps) * 64) : 0u;
    // (lane j of the wave: word 16 wave + j)
    const int src = (wave * 16 + lane) & 63;
    const unsigned long long mine = __shfl(bits, src, 64);
    emit_words(lane < 16 ? mine : 0ull, __shfl(o, src, 64), __shfl(base, src, 64), 16, cand_lin, cand_cap);
}

// The same for bitmaps of up to kEmitMidWords words, after k_cand_dilate_chunks: a block owns 256 words, adds up the
// counts of the chunks (of 1 << chunk_shift words: 256 or 16) before them, a few thousand numbers out of L2, and scans
// its own words.  The last
// block finds the per-sample ranges from the chunk counts by itself, so that no block waits for another.
// `cand_count` holds the words' candidate counts, unscanned.
__global__ __launch_bounds__(256) void k_cand_emit_mid(Geom g, const unsigned long long* __restrict__ cand,
                                                       const unsigned* __restrict__ cand_count,
                                                       const unsigned* __restrict__ chunk_sums, int chunk_shift,
                                                       long long n_words, unsigned* __restrict__ cand_lin,
                                                       long long cand_cap,
                                                       int* __restrict__ cand_start, int* __restrict__ tile_start,
                                                       int* __restrict__ rows16_start, Counters* ctr) {
    __shared__ unsigned s_wave[4];
    __shared__ unsigned long long s_total;
    __shared__ unsigned s_pref[kEmitMidChunks + 1];  // (last block) candidates in the chunks before chunk i
    if (blockIdx.x == gridDim.x - 1) {
        // exclusive scan of the chunk counts: a thread takes `per` consecutive chunks
        const int n_chunks = (int)((n_words + (1ll << chunk_shift) - 1) >> chunk_shift);  // (<= kEmitMidChunks)
        const int per = (n_chunks + 255) / 256, i_lo = (int)threadIdx.x * per;
        unsigned local = 0;
        for (int i = i_lo; i < i_lo + per && i < n_chunks; ++i) local += chunk_sums[i];
        unsigned total;
        unsigned run = block_exclusive_scan_256(local, s_wave, total);
        for (int i = i_lo; i < i_lo + per && i < n_chunks; ++i) {
            s_pref[i] = run;
            run += chunk_sums[i];
        }
        if (threadIdx.x == 0) {
            s_pref[n_chunks] = total;
            s_total = total;
        }
        __syncthreads();
        // candidates before sample b = chunks wholly before its first word + the words of the chunk it starts in
        for (int b = threadIdx.x; b <= g.batch; b += 256) {
            const long long w_b = (long long)b * g.Wps;  // (= n_words for b = batch)
            const int c_b = (int)(w_b >> chunk_shift);
            unsigned sum = s_pref[c_b];
            for (long long w0 = (long long)c_b << chunk_shift; w0 < w_b; w0 += 8) {  // eight loads in flight
                unsigned x[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) x[u] = w0 + u < w_b ? cand_count[w0 + u] : 0u;
#pragma unroll
                for (int u = 0; u < 8; ++u) sum += x[u];
            }
            // (a total beyond the capacity is far below 2^31: at most 2^31 sites per call)
            cand_start[b] = (int)sum;
        }
        __syncthreads();
        const long long n_cand = (long long)s_total;
        const bool overflow = n_cand > cand_cap;
        if (overflow)
            for (int b = threadIdx.x; b <= g.batch; b += blockDim.x) cand_start[b] = 0;
        __syncthreads();
        const int n_tiles_all = sample_ranges_256(g.batch, cand_start, tile_start, rows16_start, s_wave);
        if (threadIdx.x == 0) {
            ctr->n_cand = n_cand;
            ctr->n_tiles = n_tiles_all;
            if (overflow) atomicOr(&ctr->flags, SCNN_FLAG_CAND_OVERFLOW);
        }
        return;
    }
    const int c = blockIdx.x;  // words [256 c, 256 c + 256): whole chunks (a chunk has 256 or 16 words)
    const int chunks_below = (int)(((long long)c << 8) >> chunk_shift);
    unsigned below = 0;
    for (int i0 = threadIdx.x; i0 < chunks_below; i0 += 256 * 8) {  // eight loads in flight per thread
        unsigned x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = i0 + 256 * u < chunks_below ? chunk_sums[i0 + 256 * u] : 0u;
#pragma unroll
        for (int u = 0; u < 8; ++u) below += x[u];
    }
    unsigned before_block;
    (void)block_exclusive_scan_256(below, s_wave, before_block);  // (the total is what is wanted)
    const long long w = (long long)c * 256 + threadIdx.x;
    const unsigned long long bits = w < n_words ? cand[w] : 0ull;
    unsigned block_total;
    const unsigned o = before_block + block_exclusive_scan_256((unsigned)__popcll(bits), s_wave, block_total);
    emit_words(bits, o, w < n_words ? (unsigned)((w % g.Wps) * 64) : 0u, 64, cand_lin, cand_cap);
}

hipError_t launch_cand_emit_mid(const Geom& g, const unsigned long long* cand, const unsigned* cand_count,
                                const unsigned* chunk_sums, long long n_words, unsigned* cand_lin, long long cand_cap,
                                int* cand_start, int* tile_start, int* rows16_start, Counters* ctr, hipStream_t s) {
    const unsigned blocks = (unsigned)((n_words + 255) / 256);
    const int chunk_shift = cand_chunk_shift(n_words, g.Wps);
    hipLaunchKernelGGL(k_cand_emit_mid, dim3(blocks + 1), dim3(256), 0, s, g, cand, cand_count, chunk_sums,
                       chunk_shift, n_words, cand_lin, cand_cap, cand_start, tile_start, rows16_start, ctr);
    return hipGetLastError();
}

hipError_t launch_cand_emit(const Geom& g, const unsigned long long* cand, const unsigned* cand_prefix,
                            long long n_words, unsigned* cand_lin, long long cand_cap, int* cand_start,
                            int* tile_start, int* rows16_start, Counters* ctr, hipStream_t s) {
    long long blocks = (n_words + 255) / 256;
    if (blocks < 1) blocks = 1;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_cand_emit, dim3((unsigned)blocks + 1), dim3(256), 0, s, g, cand, cand_prefix, n_words,
                       cand_lin, cand_cap, cand_start, tile_start, rows16_start, ctr);
    return hipGetLastError();
}

hipError_t launch_cand_emit_small(const Geom& g, const unsigned long long* cand, const unsigned* cand_count,
                                  long long n_words, unsigned* cand_lin, long long cand_cap, int* cand_start,
                                  int* tile_start, int* rows16_start, Counters* ctr, hipStream_t s) {
    const unsigned blocks = (unsigned)((n_words + 63) / 64);
    hipLaunchKernelGGL(k_cand_emit_small, dim3(blocks + 1), dim3(256), 0, s, g, cand, cand_count, (int)n_words,
                       cand_lin, cand_cap, cand_start, tile_start, rows16_start, ctr);
    return hipGetLastError();
}

}  // namespace scnn
