// Back-propagation through the convolution (Algorithm 2, with the masks of Eq. 3).
//
// The paper walks the same loop nest as the forward pass and issues two atomic
// adds per multiply (one into bp_data, one into bp_filter).  Here both outputs
// are formed without value atomics:
//
//   bp_data[q, ic]      = sum over taps t, channels oc of  w[t, ic, oc] * g[q - delta_t, oc]     (x[q, ic] != 0)
//   bp_filter[t, ic, oc] = sum over input rows q of         x[q, ic]    * g[q - delta_t, oc]     (w[t, ic, oc] != 0)
//
// bp_data is the forward convolution of the gradient rows with the adjoint
// filter (taps negated, channels transposed), evaluated at the input's own
// sites only: the forward kernels are reused with the input rows as the list
// of output sites (gather form, fixed summation order in the vector kernel).
// bp_filter is a reduction over (input row, gradient row) pairs per tap: every
// workgroup (vector kernel) or wave (matrix-core kernel) sums a share of the
// tiles into a private partial filter in fp64 and stores it; a last kernel
// adds the partials in a fixed order, applies the mask and rounds to fp32 once.
#include "scnn_internal.h"

namespace scnn {


// ------------------------------------------------------------------ input rows as the list of output sites
// cand_lin[r] = site index of input row r; rows16_start[b] = 16-row groups of all earlier samples (the unit in
// which the pair lists reserve their space).  Rows outside the grid or out of order are reported.
__global__ __launch_bounds__(256) void k_bwd_sites(Geom g, const int32_t* __restrict__ coords, long long rows,
                                                   const int* __restrict__ cand_start,
                                                   unsigned* __restrict__ cand_lin, int* __restrict__ rows16_start,
                                                   Counters* ctr) {
    const int stride = 1 + g.ndim;
    for (long long r = (long long)blockIdx.x * blockDim.x + threadIdx.x; r < rows;
         r += (long long)gridDim.x * blockDim.x) {
        int b, c0, c1, c2;
        load_site(g, coords + r * stride, b, c0, c1, c2);
        unsigned lin = 0;
        if (site_in_grid(g, b, c0, c1, c2)) {
            lin = (unsigned)lin_of(g, c0, c1, c2);
            if (r > 0) {
                int pb, p0, p1, p2;
                load_site(g, coords + (r - 1) * stride, pb, p0, p1, p2);
                if (site_in_grid(g, pb, p0, p1, p2) &&
                    (long long)pb * g.Npad + lin_of(g, p0, p1, p2) >= (long long)b * g.Npad + lin)
                    atomicOr(&ctr->flags, SCNN_FLAG_UNSORTED);
            }
        } else {
            atomicOr(&ctr->flags, SCNN_FLAG_BAD_COORD);
        }
        cand_lin[r] = lin;
    }
    if (blockIdx.x == 0) {  // (whole block)
        __shared__ unsigned s_wave[4];
        (void)sample_ranges_256(g.batch, cand_start, nullptr, rows16_start, s_wave);
    }
}

hipError_t launch_bwd_sites(const Geom& g, const int32_t* coords, long long rows, const int* cand_start,
                            unsigned* cand_lin, int* rows16_start, Counters* ctr, hipStream_t s) {
    long long blocks = (rows + 255) / 256;
    if (blocks < 1) blocks = 1;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_bwd_sites, dim3((unsigned)blocks), dim3(256), 0, s, g, coords, rows, cand_start, cand_lin,
                       rows16_start, ctr);
    return hipGetLastError();
}

// ------------------------------------------------------------------ bp_data: planar tiles -> rows, masked by x != 0
// resp[tile][ic][row] holds the adjoint convolution at the input rows of the tile (Eq. 3, first line: the
// gradient reaches non-zero input values only).  Through LDS so that both sides coalesce.
__global__ __launch_bounds__(256) void k_bwd_data_write(Geom g, const float* __restrict__ resp,
                                                        const float* __restrict__ x, int c_in,
                                                        const int* __restrict__ cand_start,
                                                        const int* __restrict__ tile_start,
                                                        const Counters* __restrict__ ctr,
                                                        float* __restrict__ bp_data) {
    __shared__ float s_t[kTileRows][65];
    const int n_tiles = (int)ctr->n_tiles;
    // rows of x and bp_data start on 16-byte boundaries
    const bool vec4 = (c_in & 3) == 0 && ((((size_t)x) | ((size_t)bp_data)) & 15) == 0;
    for (int tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const int b = sample_of_tile(tile_start, g.batch, tile);
        const int first = cand_start[b] + (tile - tile_start[b]) * kTileRows;
        int nrows = cand_start[b + 1] - first;
        if (nrows > kTileRows) nrows = kTileRows;
        for (int cc = 0; cc < c_in; cc += 64) {
            const int cw = (c_in - cc) < 64 ? (c_in - cc) : 64;
            __syncthreads();
            for (int i = threadIdx.x; i < kTileRows * cw; i += 256) {
                const int c = i >> 7, r = i & 127;
                s_t[r][c] = resp[((size_t)tile * c_in + cc + c) * kTileRows + r];
            }
            __syncthreads();
            if (vec4) {  // four channels per thread: 16-byte loads of x and stores of bp_data
                const int q = cw >> 2;
                for (int i = threadIdx.x; i < nrows * q; i += 256) {
                    const int r = i / q, c = (i - r * q) * 4;
                    const size_t at = (size_t)(first + r) * c_in + cc + c;
                    const float4 xv = *reinterpret_cast<const float4*>(x + at);
                    float4 o;
                    o.x = xv.x != 0.0f ? s_t[r][c] : 0.0f;
                    o.y = xv.y != 0.0f ? s_t[r][c + 1] : 0.0f;
                    o.z = xv.z != 0.0f ? s_t[r][c + 2] : 0.0f;
                    o.w = xv.w != 0.0f ? s_t[r][c + 3] : 0.0f;
                    *reinterpret_cast<float4*>(bp_data + at) = o;
                }
            } else {
                for (int i = threadIdx.x; i < nrows * cw; i += 256) {
                    const int r = i / cw, c = i - r * cw;
                    const size_t at = (size_t)(first + r) * c_in + cc + c;
                    bp_data[at] = (x[at] != 0.0f) ? s_t[r][c] : 0.0f;
                }
            }
        }
    }
}

hipError_t launch_bwd_data_write(const Geom& g, const float* resp, const float* x, int c_in, const int* cand_start,
                                 const int* tile_start, const Counters* ctr, long long tiles_cap, float* bp_data,
                                 hipStream_t s) {
    long long blocks = tiles_cap < 1 ? 1 : (tiles_cap > 4096 ? 4096 : tiles_cap);
    hipLaunchKernelGGL(k_bwd_data_write, dim3((unsigned)blocks), dim3(256), 0, s, g, resp, x, c_in, cand_start,
                       tile_start, ctr, bp_data);
    return hipGetLastError();
}

// ------------------------------------------------------------------ bp_filter in fp64 (any shape)
// Per tap the contraction D[ic][oc] = sum over input rows q of x[q][ic] * g[q - delta_t][oc] (0 where the gradient has no
// row) on the fp64 matrix cores: v_mfma_f64_16x16x4_f64, the rows of a tile as K, four per instruction.  Work item =
// (slab, share of the tiles), a slab being one block of 16 input channels against up to 32 (tap, block of 16 output
// channels) slots, two to a wave.  The tile's values of x and its neighbour rows, looked up once per tile, are shared
// through LDS.  Inputs of the paper's own layers have a gradient row behind nearly every (row, tap), so the rows are not
// packed (27 taps of 47 k rows: 57 us packed, 53 not).  Bound by the latency of the look-ups and of the gathers (8 -> 16
// channels, 47 k rows, 27 taps: 319 k instructions, 10 us of matrix time).  So sixteen waves are held to 64 registers, two
// workgroups to a CU: x is read from LDS at the product and eight gathers are in flight, their masks in one register: 33 us;
// 53 with x and sixteen gathers in registers, one workgroup to a CU (40 with four masked gathers, 46 with eight; a few
// registers of the look-up spill); 167 with a thread per filter element that read both operands of every product.  Calls,
// us, before and after: 8->8, 27 taps, 12 k rows 52 / 50, 125 taps, 126 k rows 474 / 432; 24->24, 27 taps, 126 k rows
// 458 / 393; one tap, 47 k rows, 100->100 232 / 156.  Partial sums of a share are stored (no atomics), zero included.
typedef double f64x4 __attribute__((ext_vector_type(4)));
// W waves of two (tap, block of 16 output channels) slots each; nt taps and no blocks to a slab, nt * no <= 2 W (MULTI:
// no may be more than 1).
template <int W, int MULTI>
__global__ __launch_bounds__(64 * W, W == 16 ? 8 : 4) void k_bwd_filter_f64(Geom g, const unsigned long long* __restrict__ occ,
                                                        const unsigned* __restrict__ occ_prefix, long long g_rows,
                                                        const float* __restrict__ gf, int c_out,
                                                        const float* __restrict__ x, int c_in,
                                                        const int* __restrict__ tap_active /* adjoint tap order */,
                                                        const unsigned* __restrict__ cand_lin,
                                                        const int* __restrict__ cand_start,
                                                        const int* __restrict__ tile_start,
                                                        const Counters* __restrict__ ctr, int nt, int no, int n_icb,
                                                        int n_og, int n_slabs, int n_chunks,
                                                        double* __restrict__ fpart) {
    constexpr int NT = 64 * W, F = 8;  // (F: gathers in flight)
    __shared__ int s_nbr[kTileRows][2 * W + 1];
    __shared__ int s_site[kTileRows][3];
    __shared__ float s_x[kTileRows][17];
    const int n_tiles = (int)ctr->n_tiles;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = lane & 15, kq = lane >> 4;
    const int slab = (int)(blockIdx.x % (unsigned)n_slabs), chunk = (int)(blockIdx.x / (unsigned)n_slabs);
    const int blk = slab % (n_icb * n_og), t_lo = slab / (n_icb * n_og) * nt;
    const int t_hi = (t_lo + nt < g.T ? t_lo + nt : g.T) - 1;
    const int ic0 = blk / n_og * 16, oc0 = blk % n_og * no * 16;
    // the wave's slots: tap t_lo + tap[j], output channels col[j] .. col[j] + 15 (those past the layer's are dropped)
    int tap[2], col[2];
    bool on[2];
    f64x4 acc[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int slot = MULTI ? __builtin_amdgcn_readfirstlane(wave + W * j) : wave + W * j;
        const int block = MULTI ? slot / nt : 0;
        tap[j] = slot - block * nt;
        col[j] = oc0 + block * 16;
        on[j] = t_lo + tap[j] <= t_hi && (!MULTI || (block < no && col[j] < c_out));
        acc[j] = f64x4{0.0, 0.0, 0.0, 0.0};
    }

    const int a_lo = g.T - 1 - t_hi, a_hi = g.T - 1 - t_lo;  // adjoint taps [a_lo, a_hi]
    const unsigned act = active_taps(tap_active, a_lo, a_hi - a_lo + 1);
    for (int tile = chunk; tile < n_tiles; tile += n_chunks) {
        const int b = sample_of_tile(tile_start, g.batch, tile);
        const int first = cand_start[b] + (tile - tile_start[b]) * kTileRows;
        int nrows = cand_start[b + 1] - first;
        if (nrows > kTileRows) nrows = kTileRows;
        __syncthreads();  // readers of the previous tile are done
#pragma unroll
        for (int i = threadIdx.x; i < kTileRows * 16; i += NT) {
            const int r = i >> 4, c = i & 15;
            s_x[r][c] = r < nrows && ic0 + c < c_in ? x[(size_t)(first + r) * c_in + ic0 + c] : 0.0f;
        }
        if (threadIdx.x < kTileRows) {
            int c0 = 0, c1 = 0, c2 = 0;
            if (threadIdx.x < nrows) site_of(g, cand_lin[first + threadIdx.x], c0, c1, c2);
            s_site[threadIdx.x][0] = c0;
            s_site[threadIdx.x][1] = c1;
            s_site[threadIdx.x][2] = c2;
        }
        __syncthreads();
        // The gradient row of (row, tap t) sits at site - delta_t = site + delta of the mirrored tap T-1-t, so the
        // look-ups run over the mirrored (adjoint) tap indices, per filter line: the taps of a line look at
        // adjacent sites and share one pair of bitmap words.  tap_active is in adjoint order already.
        {
            const int l_first = a_lo / g.K[2];
            const int n_seg = a_hi / g.K[2] - l_first + 1;
            for (int i = threadIdx.x; i < kTileRows * n_seg; i += NT) {
                const int r = i & (kTileRows - 1), l = l_first + (i >> 7);
                const int aa = a_lo > l * g.K[2] ? a_lo : l * g.K[2];
                const int ab = (a_hi + 1) < (l + 1) * g.K[2] ? (a_hi + 1) : (l + 1) * g.K[2];
                const int t0 = l / g.K[1], t1 = l - t0 * g.K[1];
                int* dst = &s_nbr[r][0];
                lookup_line(g, occ, occ_prefix, g_rows, r < nrows, b, s_site[r][0], s_site[r][1], s_site[r][2], t0,
                            t1, aa - l * g.K[2], ab - aa, act >> (aa - a_lo),
                            [&](int k, int n) { dst[g.T - 1 - (aa + k) - t_lo] = n; });
            }
        }
        __syncthreads();
        if (g_rows < 1) continue;  // (every product is 0; the gathers below read row 0 for an absent neighbour)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (!on[j]) continue;
            // (a column past the layer's reads its last one; nothing is stored for it)
            const float* gcol = gf + (col[j] + m < c_out ? col[j] + m : c_out - 1);
#pragma unroll 1
            for (int s0 = 0; 4 * s0 < nrows; s0 += F) {
                float gv[F];
                unsigned there = 0;
#pragma unroll
                for (int s = 0; s < F; ++s) {
                    const int n = s_nbr[4 * (s0 + s) + kq][tap[j]];
                    gv[s] = gcol[(size_t)(n < 0 ? 0 : n) * c_out];
                    there |= n < 0 ? 0u : 1u << s;
                }
#pragma unroll
                for (int s = 0; s < F; ++s) {
                    // no gradient row: the product is 0 * 0 whatever the rows hold (an infinity or NaN belongs to the
                    // pairs that exist)
                    const bool pair = there & (1u << s);
                    acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(pair ? (double)s_x[4 * (s0 + s) + kq][m] : 0.0,
                                                                  pair ? (double)gv[s] : 0.0, acc[j], 0, 0, 0);
                }
            }
        }
    }
    // element v of a lane: input channel 4 v + kq, output channel m of the block
    double* out = fpart + (size_t)chunk * g.T * c_in * c_out;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        if (!on[j]) continue;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int ic = ic0 + 4 * v + kq;
            if (ic < c_in && col[j] + m < c_out)
                out[((size_t)(t_lo + tap[j]) * c_in + ic) * c_out + col[j] + m] = acc[j][v];
        }
    }
}

// ------------------------------------------------------------------ bp_filter, vector kernel (long filters, few channels)
// Work item = (block of 256 consecutive filter elements in [t][ic][oc] order, share of the tiles).  A thread owns
// one element and walks the rows of its tiles: row q contributes x[q, ic] * g[q - delta_t, oc] when the gradient
// has a row at q - delta_t.  The neighbour rows of a tile are looked up once per tap and shared through LDS.
// fp64 throughout; the partial sum of the share is stored (no atomics), zero included.
// Where a 16 x 16 block of channels holds at most 16 products the matrix form above does sixteen times the work of this
// one and is slower once there are more than two slabs of taps: 125 taps, 47 k / 126 k rows, call in us, this / that:
// 1->8 141 / 304 against 196 / 425, 1->16 242 / 504 against 264 / 552, 3->5 222 / 463 against 251 / 528; 49 taps, 31 k
// rows of 2-D: 73 against 84, 90 against 98, 102 against 111; but 1->1, 125 taps, on 12 k rows 134 against 90.
constexpr int kBwdTapChunk = 32;  // taps whose neighbour rows are staged in LDS at a time
__global__ __launch_bounds__(256) void k_bwd_filter_valu(Geom g, const unsigned long long* __restrict__ occ,
                                                         const unsigned* __restrict__ occ_prefix, long long g_rows,
                                                         const float* __restrict__ gf, int c_out,
                                                         const float* __restrict__ x, int c_in,
                                                         const int* __restrict__ tap_active /* adjoint tap order */,
                                                         const unsigned* __restrict__ cand_lin,
                                                         const int* __restrict__ cand_start,
                                                         const int* __restrict__ tile_start,
                                                         const Counters* __restrict__ ctr, int n_eb, int n_chunks,
                                                         double* __restrict__ fpart) {
    __shared__ int s_nbr[kTileRows][kBwdTapChunk + 1];
    __shared__ int s_site[kTileRows][3];
    const int n_tiles = (int)ctr->n_tiles;
    const int cc = c_in * c_out;
    const long long n_elem = (long long)g.T * cc;
    const int eb = (int)(blockIdx.x % (unsigned)n_eb), chunk = (int)(blockIdx.x / (unsigned)n_eb);
    const long long e = (long long)eb * 256 + threadIdx.x;
    const bool valid = e < n_elem;
    const int t_e = valid ? (int)(e / cc) : -1;
    const int ic = valid ? (int)((e % cc) / c_out) : 0, oc = valid ? (int)(e % c_out) : 0;
    const int t_lo = (int)(((long long)eb * 256) / cc);
    long long e_hi = (long long)eb * 256 + 255;
    if (e_hi > n_elem - 1) e_hi = n_elem - 1;
    const int t_hi = (int)(e_hi / cc);
    double acc = 0.0;

    for (int tile = chunk; tile < n_tiles; tile += n_chunks) {
        const int b = sample_of_tile(tile_start, g.batch, tile);
        const int first = cand_start[b] + (tile - tile_start[b]) * kTileRows;
        int nrows = cand_start[b + 1] - first;
        if (nrows > kTileRows) nrows = kTileRows;
        __syncthreads();  // readers of s_site / s_nbr of the previous tile are done
        if (threadIdx.x < kTileRows) {
            int c0 = 0, c1 = 0, c2 = 0;
            if (threadIdx.x < nrows) site_of(g, cand_lin[first + threadIdx.x], c0, c1, c2);
            s_site[threadIdx.x][0] = c0;
            s_site[threadIdx.x][1] = c1;
            s_site[threadIdx.x][2] = c2;
        }
        for (int tc = t_lo; tc <= t_hi; tc += kBwdTapChunk) {
            __syncthreads();
            // The gradient row of (row, tap t) sits at site - delta_t = site + delta of the mirrored tap T-1-t, so the
            // look-ups run over the mirrored (adjoint) tap indices, per filter line: the taps of a line look at
            // adjacent sites and share one pair of bitmap words.  tap_active is in adjoint order already.
            {
                const int t_last = (tc + kBwdTapChunk - 1) < t_hi ? (tc + kBwdTapChunk - 1) : t_hi;
                const int a_lo = g.T - 1 - t_last, a_hi = g.T - 1 - tc;  // adjoint taps [a_lo, a_hi]
                const unsigned act = active_taps(tap_active, a_lo, a_hi - a_lo + 1);
                const int l_first = a_lo / g.K[2];
                const int n_seg = a_hi / g.K[2] - l_first + 1;
                for (int i = threadIdx.x; i < kTileRows * n_seg; i += 256) {
                    const int r = i & (kTileRows - 1), l = l_first + (i >> 7);
                    const int aa = a_lo > l * g.K[2] ? a_lo : l * g.K[2];
                    const int ab = (a_hi + 1) < (l + 1) * g.K[2] ? (a_hi + 1) : (l + 1) * g.K[2];
                    const int t0 = l / g.K[1], t1 = l - t0 * g.K[1];
                    int* dst = &s_nbr[r][0];
                    lookup_line(g, occ, occ_prefix, g_rows, r < nrows, b, s_site[r][0], s_site[r][1], s_site[r][2], t0,
                                t1, aa - l * g.K[2], ab - aa, act >> (aa - a_lo),
                                [&](int k, int n) { dst[g.T - 1 - (aa + k) - tc] = n; });
                }
            }
            __syncthreads();
            if (valid && t_e >= tc && t_e < tc + kBwdTapChunk) {
                const int tt = t_e - tc;
                // eight rows at a time, their loads independent of one another; the sum keeps the row order
                for (int r0 = 0; r0 < nrows; r0 += 8) {
                    float xv[8], gv[8];
                    bool on[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int r = r0 + u;
                        const int n = r < nrows ? s_nbr[r][tt] : -1;
                        on[u] = n >= 0;
                        xv[u] = x[(size_t)(first + (r < nrows ? r : 0)) * c_in + ic];
                        gv[u] = on[u] ? gf[(size_t)n * c_out + oc] : 0.0f;  // (no gradient row: nothing is read)
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        if (on[u]) acc = fma((double)xv[u], (double)gv[u], acc);
                }
            }
        }
    }
    if (valid) fpart[(size_t)chunk * n_elem + e] = acc;
}

// How bp_filter outside the matrix-core lists is cut.  waves = 0: the vector kernel, `slabs` blocks of 256 elements.
// Taps x blocks of output channels of at most 8 take four waves and everything in one slab (1 x 1, 47 k rows: 24->24 118
// -> 53 us a call, 100->100 1300 -> 156 with all blocks of channels in the workgroup that looks the rows up; 9 taps 24->24
// 160 -> 98); but a workgroup per block where these do not fill the chip (one 28 x 28 image, 24->24: 50 us against 57).
struct BwdF64Shape {
    int waves, nt, no, n_icb, n_og;
    long long slabs;
};
static BwdF64Shape bwd_f64_shape(const Geom& g, int c_in, int c_out, long long tiles_cap) {
    BwdF64Shape s;
    if (g.T > 48 && c_in * c_out <= 16 && tiles_cap > 64) {
        s = BwdF64Shape{0, 0, 0, 0, 0, ((long long)g.T * c_in * c_out + 255) / 256};
        return s;
    }
    const int n_ocb = (c_out + 15) / 16;
    s.waves = (long long)g.T * n_ocb <= 8 ? 4 : 16;
    s.nt = g.T < 2 * s.waves ? g.T : 2 * s.waves;
    s.n_icb = (c_in + 15) / 16;
    const long long groups = (long long)((g.T + s.nt - 1) / s.nt) * s.n_icb;
    s.no = 2 * s.waves / s.nt < n_ocb ? 2 * s.waves / s.nt : n_ocb;
    if (groups * n_ocb * tiles_cap <= device_cu_count()) s.no = 1;
    s.n_og = (n_ocb + s.no - 1) / s.no;
    s.slabs = groups * s.n_og;
    return s;
}

hipError_t launch_bwd_filter_f64(const Geom& g, const unsigned long long* occ, const unsigned* occ_prefix,
                                 long long g_rows, const float* gf, int c_out, const float* x, int c_in,
                                 const int* tap_active, const unsigned* cand_lin, const int* cand_start,
                                 const int* tile_start, const Counters* ctr, long long tiles_cap, int n_chunks,
                                 double* fpart, hipStream_t s) {
    const BwdF64Shape p = bwd_f64_shape(g, c_in, c_out, tiles_cap);
    const dim3 grid((unsigned)(p.slabs * n_chunks)), block((unsigned)(p.waves ? 64 * p.waves : 256));
#define SCNN_BWD_F64(W, MULTI)                                                                                        \
    hipLaunchKernelGGL((k_bwd_filter_f64<W, MULTI>), grid, block, 0, s, g, occ, occ_prefix, g_rows, gf, c_out, x, c_in, \
                       tap_active, cand_lin, cand_start, tile_start, ctr, p.nt, p.no, p.n_icb, p.n_og, (int)p.slabs,  \
                       n_chunks, fpart)
    if (p.waves == 0)
        hipLaunchKernelGGL(k_bwd_filter_valu, grid, block, 0, s, g, occ, occ_prefix, g_rows, gf, c_out, x, c_in,
                           tap_active, cand_lin, cand_start, tile_start, ctr, (int)p.slabs, n_chunks, fpart);
    else if (p.waves == 4)
        SCNN_BWD_F64(4, 1);
    else if (p.no > 1)
        SCNN_BWD_F64(16, 1);
    else
        SCNN_BWD_F64(16, 0);
#undef SCNN_BWD_F64
    return hipGetLastError();
}

// ------------------------------------------------------------------ bp_filter, matrix-core kernel
// Uses the pair lists of the adjoint convolution: per tile of 128 input rows and per adjoint tap t', blocks of 16
// (local input row, gradient row) pairs.  For one tap the filter gradient is the contraction
//     D[ic][oc] += sum over pairs  x[q(pair)][ic] * g[p(pair)][oc],
// i.e. a [C_in x pairs] . [pairs x C_out] product whose long dimension is the pair list: the pairs are the K
// dimension of v_mfma_f32_16x16x4_f32, four per instruction.  A wave owns one (tap, 16*MT input channels,
// 16*NT output channels) slab and a contiguous share of the tiles; it keeps the slab in registers for its whole
// life: fp32 matrix-core sums over the (at most 128) pairs of one tile, added to an fp64 copy after each tile.
// Lane (jj = lane & 15, gq = lane >> 4) feeds pair 4*gq + j of a block in step j (the order of the pairs inside a
// sum is free), input channels jj*MT + i and output channels jj*NT + i of the slab, so that its operands are one
// 8- or 16-byte load per pair at a 32-bit offset from a wave-uniform base: three vector instructions of address
// arithmetic per pair.  Only the last block of a tap can hold list padding (local row 128), so only that block
// pays for masking.
//
// What bounds it: the fp32 matrix instructions (128 x 8 clocks of a SIMD per block at 32 x 64 channels) and the latency
// of the gathers behind them.  128^3 x 4, 32 -> 64 channels, 25 G multiply-adds: 291 us (164 at the rate that a large fp32
// product reaches here) -> 266 us with the blocks of a share as one stream across tiles and the padding masked at the
// multiplication.  Splitting the operands into bf16 thirds takes 60 vector instructions per eight values, more issue
// time than the fp32 products it would replace.
//
// All slabs of one share of the tiles run on the same XCD (workgroup i runs on XCD i % 8), so that the share's
// input rows and gradient rows are fetched into that XCD's L2 once for all taps.
template <int MT, int NT>
struct BwdOperands {
    float av[4][MT], bv[4][NT];
    bool live[4];  // of a tap's last block in a tile: not list padding
};

template <int MT, int NT, bool MASKED>
__device__ __forceinline__ void bwd_filter_load(const uint4 ent, const char* __restrict__ xt,
                                                const char* __restrict__ gl, unsigned cin4, unsigned cout4,
                                                unsigned xlane, unsigned glane, BwdOperands<MT, NT>& o) {
    const unsigned en[4] = {ent.x, ent.y, ent.z, ent.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const unsigned row = en[j] >> kPairRowShift;
        // the 24-bit multiply reads the low 24 bits of its operands: the gradient row of the pair, as it is
        const unsigned goff = __umul24(en[j], cout4) + glane;
        unsigned xoff = __umul24(row, cin4) + xlane;
        if constexpr (MASKED) {
            o.live[j] = row < (unsigned)kTileRows;
            xoff = o.live[j] ? xoff : xlane;
        }
        if constexpr (MT == 1) {
            o.av[j][0] = *(const float*)(xt + xoff);
        } else {
            const float2 t2 = *(const float2*)(xt + xoff);
            o.av[j][0] = t2.x;
            o.av[j][1] = t2.y;
        }
        if constexpr (NT == 1) {
            o.bv[j][0] = *(const float*)(gl + goff);
        } else if constexpr (NT == 2) {
            const float2 t2 = *(const float2*)(gl + goff);
            o.bv[j][0] = t2.x;
            o.bv[j][1] = t2.y;
        } else {
            const float4 t4 = *(const float4*)(gl + goff);
            o.bv[j][0] = t4.x;
            o.bv[j][1] = t4.y;
            o.bv[j][2] = t4.z;
            o.bv[j][3] = t4.w;
        }
    }
}

template <int MT, int NT>
__device__ __forceinline__ void bwd_filter_mma(const BwdOperands<MT, NT>& o, f32x4 (&acc)[MT][NT]) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int a = 0; a < MT; ++a)
#pragma unroll
            for (int c = 0; c < NT; ++c)
                acc[a][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(o.av[j][a], o.bv[j][c], acc[a][c], 0, 0, 0);
}

template <int MT, int NT>
__global__ __launch_bounds__(256) void k_bwd_filter_mfma(int taps, int c_in, int c_out, const float* __restrict__ x,
                                                         const float* __restrict__ gf,
                                                         const unsigned* __restrict__ pairs,
                                                         const unsigned short* __restrict__ tap_first,
                                                         const uint2* __restrict__ tile_hdr,
                                                         const int* __restrict__ cand_start,
                                                         const int* __restrict__ tile_start, int batch,
                                                         const Counters* __restrict__ ctr, int n_chunks,
                                                         int groups /* workgroups per share */,
                                                         double* __restrict__ fpart) {
    const int lane = threadIdx.x & 63;
    const int jj = lane & 15, gq = lane >> 4;
    const int n_icb = c_in / (16 * MT), n_ocb = c_out / (16 * NT);
    const int slabs = taps * n_icb * n_ocb;
    const int xcd = blockIdx.x % kXcds, j_in_xcd = blockIdx.x / kXcds;
    const int chunk = (j_in_xcd / groups) * kXcds + xcd;
    const int slab = __builtin_amdgcn_readfirstlane((j_in_xcd % groups) * 4 + (int)(threadIdx.x >> 6));
    if (chunk >= n_chunks || slab >= slabs) return;
    const int ta = slab / (n_icb * n_ocb);  // adjoint tap
    const int icb = (slab / n_ocb) % n_icb, ocb = slab % n_ocb;
    const int n_tiles = (int)ctr->n_tiles;
    // contiguous share of the tiles
    const int tile_lo = (int)((long long)chunk * n_tiles / n_chunks);
    const int tile_hi = (int)((long long)(chunk + 1) * n_tiles / n_chunks);
    const unsigned cin4 = (unsigned)c_in * 4u, cout4 = (unsigned)c_out * 4u;
    const unsigned xlane = (unsigned)(icb * 16 * MT + jj * MT) * 4u, glane = (unsigned)(ocb * 16 * NT + jj * NT) * 4u;
    const char* __restrict__ gl = (const char*)gf;

    double acc64[MT][NT][4];
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int c = 0; c < NT; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc64[a][c][v] = 0.0;

    int b = tile_lo < tile_hi ? sample_of_tile(tile_start, batch, tile_lo) : 0;
    int b_end = tile_start[b + 1];  // first tile of the next sample
    // The share's blocks of this tap as one stream: pair entries are fetched two blocks ahead of the multiplication and
    // operands one (two register sets that swap roles, so that nothing is copied), across tiles too: a tile has about
    // three blocks of a tap, and a pipeline filled anew for each of them left the matrix pipe idle a third of the time.
    int tile = tile_lo - 1;         // tile of the block handed out last
    unsigned blk = 0, blk_end = 0;  // its next block and its end
    unsigned nb0 = 0, nb1 = 0;      // block range of this tap in the next tile, read one tile ahead
    const char* xt = (const char*)x;
    auto read_range = [&](int t) {
        if (t < tile_hi) {
            const unsigned short* tf = tap_first + (size_t)t * (taps + 1) + ta;
            const unsigned h = tile_hdr[t].x;
            nb0 = h + tf[0];
            nb1 = h + tf[1];
        }
    };
    uint4 ent;
    bool ahead = true, ent_last = false;  // a block is waiting in ent; it is its tile's last
    auto next = [&] {
        while (blk >= blk_end) {
            if (++tile >= tile_hi) {
                ahead = false;
                return;
            }
            blk = nb0;
            blk_end = nb1;
            read_range(tile + 1);
            while (tile >= b_end) {  // next sample (samples without rows have no tiles)
                ++b;
                b_end = tile_start[b + 1];
            }
            xt = (const char*)(x + (size_t)(cand_start[b] + (tile - tile_start[b]) * kTileRows) * c_in);
        }
        ent = *(const uint4*)(pairs + (size_t)blk * 16 + gq * 4);
        ent_last = ++blk >= blk_end;
    };
    auto issue = [&](BwdOperands<MT, NT>& dst) {
        const bool last = ent_last;
        if (last)
            bwd_filter_load<MT, NT, true>(ent, xt, gl, cin4, cout4, xlane, glane, dst);
        else
            bwd_filter_load<MT, NT, false>(ent, xt, gl, cin4, cout4, xlane, glane, dst);
        next();
        return last;
    };
    f32x4 acc[MT][NT];
    auto clear = [&] {
#pragma unroll
        for (int a = 0; a < MT; ++a)
#pragma unroll
            for (int c = 0; c < NT; ++c) acc[a][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    auto multiply = [&](BwdOperands<MT, NT>& o, bool last) {
        if (last) {  // (here and not after the loads, which would be waited for one by one)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int a = 0; a < MT; ++a) o.av[j][a] = o.live[j] ? o.av[j][a] : 0.0f;
        }
        bwd_filter_mma<MT, NT>(o, acc);
        if (last) {
#pragma unroll
            for (int a = 0; a < MT; ++a)
#pragma unroll
                for (int c = 0; c < NT; ++c)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        acc64[a][c][v] = fma((double)acc[a][c][v], 1.0, acc64[a][c][v]);  // full-rate form of the add
            clear();
        }
    };
    clear();
    read_range(tile_lo);
    next();
    if (ahead) {
        BwdOperands<MT, NT> opa, opb;
        bool last_a = issue(opa), last_b = false;
        for (;;) {
            const bool more_b = ahead;
            if (more_b) last_b = issue(opb);
            multiply(opa, last_a);
            if (!more_b) break;
            const bool more_a = ahead;
            if (more_a) last_a = issue(opa);
            multiply(opb, last_b);
            if (!more_a) break;
        }
    }
    // result element (a, c, v) of this lane: input channel (4*gq + v)*MT + a, output channel jj*NT + c of the slab
    const int t = taps - 1 - ta;  // tap of the filter itself
    double* out = fpart + ((size_t)chunk * taps + t) * c_in * c_out;
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int ic = icb * 16 * MT + (4 * gq + v) * MT + a;
#pragma unroll
            for (int c = 0; c < NT; ++c) out[(size_t)ic * c_out + ocb * 16 * NT + jj * NT + c] = acc64[a][c][v];
        }
}

// The gradient values are addressed with 32-bit byte offsets.
bool bwd_filter_mfma_supported(int c_in, int c_out, long long g_rows) {
    return c_in % 16 == 0 && c_out % 16 == 0 && g_rows * c_out * 4 < (1ll << 32);
}

// waves per share of the tiles
static int bwd_filter_slabs(const Geom& g, int c_in, int c_out) {
    const int mt = (c_in % 32 == 0) ? 2 : 1, nt = (c_out % 64 == 0) ? 4 : (c_out % 32 == 0 ? 2 : 1);
    return g.T * (c_in / (16 * mt)) * (c_out / (16 * nt));
}

int bwd_filter_chunks(const Geom& g, int c_in, int c_out, long long tiles_cap, bool mfma) {
    long long chunks;
    if (mfma) {
        const int slabs = bwd_filter_slabs(g, c_in, c_out);
        // all waves resident at once (two per SIMD), the same number of shares on every XCD
        chunks = (device_cu_count() * 8) / ((slabs + 3) / 4 * 4) / kXcds * kXcds;
        if (chunks < kXcds) chunks = kXcds;
        if (chunks > 256) chunks = 256;
    } else {
        // every share's partial filter is stored and added up again
        const BwdF64Shape p = bwd_f64_shape(g, c_in, c_out, tiles_cap);
        if (p.waves == 0) {
            chunks = (4096 + p.slabs - 1) / p.slabs;
            if (chunks > 512) chunks = 512;
        } else {
            chunks = ((p.waves == 4 ? 4 : 2) * device_cu_count() + p.slabs - 1) / p.slabs;
        }
    }
    if (chunks > tiles_cap) chunks = tiles_cap;
    if (chunks < 1) chunks = 1;
    return (int)chunks;
}

hipError_t launch_bwd_filter_mfma(const Geom& g, const float* x, int c_in, const float* gf, int c_out,
                                  const unsigned* pairs, const unsigned short* tap_first, const uint2* tile_hdr,
                                  const int* cand_start, const int* tile_start, const Counters* ctr, int n_chunks,
                                  double* fpart, hipStream_t s) {
    const int groups = (bwd_filter_slabs(g, c_in, c_out) + 3) / 4;
    const unsigned blocks = (unsigned)(kXcds * groups * ((n_chunks + kXcds - 1) / kXcds));
#define SCNN_BWD_CASE(MT_, NT_)                                                                                   \
    hipLaunchKernelGGL((k_bwd_filter_mfma<MT_, NT_>), dim3(blocks), dim3(256), 0, s, g.T, c_in, c_out, x, gf, pairs, \
                       tap_first, tile_hdr, cand_start, tile_start, g.batch, ctr, n_chunks, groups, fpart)
    if (c_in % 32 == 0) {
        if (c_out % 64 == 0) SCNN_BWD_CASE(2, 4); else if (c_out % 32 == 0) SCNN_BWD_CASE(2, 2); else SCNN_BWD_CASE(2, 1);
    } else {
        if (c_out % 64 == 0) SCNN_BWD_CASE(1, 4); else if (c_out % 32 == 0) SCNN_BWD_CASE(1, 2); else SCNN_BWD_CASE(1, 1);
    }
#undef SCNN_BWD_CASE
    return hipGetLastError();
}

// ------------------------------------------------------------------ bp_filter: add the partials, mask, round
// Eq. 3, second line: a weight that is exactly zero (pruned) receives no gradient.
// Also writes the call's status words: {input rows, gradient rows, flags, 0}.
constexpr int kFinishParts = 16;
__global__ __launch_bounds__(64 * kFinishParts) void k_bwd_filter_finish(const double* __restrict__ fpart, int n_chunks,
                                                                         long long n_elem, const float* __restrict__ w,
                                                                         float* __restrict__ bp_filter,
                                                                         const Counters* __restrict__ ctr,
                                                                         long long nnz_in, long long g_rows,
                                                                         long long* __restrict__ info) {
    // 64 elements per workgroup; sixteen threads per element each add a sixteenth of the partials (ascending, eight
    // loads in flight), then those sums are added in ascending order: the order of the additions never depends on
    // timing.  (Four threads with one load in flight each took 20.6 us for
    // 293 shares of 3456 elements; this takes 6.2 for 372.)
    __shared__ double s_q[kFinishParts][64];
    const int el = threadIdx.x & 63, q = threadIdx.x >> 6;
    const long long e = (long long)blockIdx.x * 64 + el;
    double sum = 0.0;
    const bool live = e < n_elem && w[e] != 0.0f;
    if (live) {
        const int c0 = (int)((long long)q * n_chunks / kFinishParts), c1 = (int)((long long)(q + 1) * n_chunks / kFinishParts);
#pragma unroll 8
        for (int c = c0; c < c1; ++c) sum += fpart[(size_t)c * n_elem + e];
    }
    s_q[q][el] = sum;
    __syncthreads();
    if (q == 0 && e < n_elem) {
#pragma unroll
        for (int i = 1; i < kFinishParts; ++i) sum += s_q[i][el];
        bp_filter[e] = (float)sum;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        info[0] = nnz_in;
        info[1] = g_rows;
        info[2] = (long long)ctr->flags;
        info[3] = 0;
    }
}

hipError_t launch_bwd_filter_finish(const double* fpart, int n_chunks, long long n_elem, const float* w,
                                    float* bp_filter, const Counters* ctr, long long nnz_in, long long g_rows,
                                    long long* info, hipStream_t s) {
    hipLaunchKernelGGL(k_bwd_filter_finish, dim3((unsigned)((n_elem + 63) / 64)), dim3(64 * kFinishParts), 0, s, fpart,
                       n_chunks, n_elem, w, bp_filter, ctr, nnz_in, g_rows, info);
    return hipGetLastError();
}

}  // namespace scnn
