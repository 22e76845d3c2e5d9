// Convolution proper (Algorithm 1, steps 5-9 and 13-14), output-stationary.
//
// The paper scatters every input entry into a dense per-(sample, channel)
// buffer with atomic adds.  Here each candidate output site instead gathers
// its present neighbours: for tap delta the neighbour of p is q = p + delta,
// found through the occupancy bitmap (the inverse of get_update_id).  Sums are
// therefore formed in a fixed order (tap ascending, input channel ascending),
// need no atomics and no r^d value buffer, and are bit-reproducible.
//
// Accumulation is in fp64 with one rounding to fp32 per response: a response is
// a sum of hundreds of signed products that largely cancel, and an fp32 running
// sum leaves an absolute error of a few 1e-6 on the small ones -- more than the
// 1e-6 the layer's results are held to.  On gfx950 the fp64 vector FMA issues at
// the rate of the (unpacked) fp32 one, so the wider sum costs registers only.
//
// Responses are written as tiles of kTileRows candidate sites in a planar
// layout  resp[tile][oc][row]  so that the per-channel selection that follows
// streams contiguous segments.
#include <type_traits>

#include "scnn_internal.h"

namespace scnn {

constexpr int kTapChunk = 32;  // taps whose neighbour rows are staged in LDS at a time
constexpr int kOcBlock = 16;   // output channels accumulated per thread

// Streaming form of the vector kernel, for layers with many more work items than workgroup slots: little shared
// memory and moderate registers, so that many waves per compute unit hide each other's memory latency.  A thread
// walks its taps; per tap it fetches CH input channels with one vector load and takes the weights through scalar
// loads, two channels' worth at a time.  Neighbour rows are looked up per filter line (adjacent sites share one
// pair of bitmap words).
// Work item = (tile, block of 32 output channels); thread = (row, 16 channels).  When the block holds only 16
// channels the second half of the workgroup takes every other tap (partial sums added through LDS, fixed order).
// OCB = 8: layers of at most 8 output channels (the first block of the paper's networks, on its largest grid) keep
// 8 accumulators per thread instead of 16 half-idle ones; on such layers the kernel is bound by FMA issue.
// Runs only when the layer has more than `min_items` work items (a device-side count).
template <int CH /* the largest of 8, 4, 2, 1 that divides C_in and suits the alignment of the values */,
          int OCB /* output channels per thread: 16, or 8 for layers of at most 8 channels (then always split) */>
__global__ __launch_bounds__(256) void k_conv_valu_stream(Geom g, const unsigned long long* __restrict__ occ,
                                                          const unsigned* __restrict__ occ_prefix, long long nnz_in,
                                                          const float* __restrict__ feats, int c_in,
                                                          const double* __restrict__ wp, int c_out, int c_out_pad,
                                                          const float* __restrict__ bias,
                                                          const int* __restrict__ tap_active,
                                                          const unsigned* __restrict__ cand_lin,
                                                          const int* __restrict__ cand_start,
                                                          const int* __restrict__ tile_start,
                                                          const Counters* __restrict__ ctr, long long min_items,
                                                          float* __restrict__ resp) {
    // s_nbr doubles as the buffer of the second half's partial sums (16 doubles per row fit in 33 ints)
    __shared__ __align__(8) int s_nbr[kTileRows][kTapChunk + 2];
    __shared__ int s_site[kTileRows][3];
    static_assert(sizeof(int) * (kTapChunk + 2) >= sizeof(double) * (kOcBlock + 1), "a row of partial sums fits");

    const int n_tiles = (int)ctr->n_tiles;
    const int n_chunks = (c_out_pad + 2 * kOcBlock - 1) / (2 * kOcBlock);
    const long long n_items = (long long)n_tiles * n_chunks;
    if (n_items <= min_items) return;  // the latency-oriented kernel takes small layers
    const int row = threadIdx.x & (kTileRows - 1);
    const int half = __builtin_amdgcn_readfirstlane(threadIdx.x >> 7);  // which 16-channel block of the chunk

    for (long long item = blockIdx.x; item < n_items; item += gridDim.x) {
        const int tile = (int)(item / n_chunks);
        const int chunk = (int)(item - (long long)tile * n_chunks);
        const int b = sample_of_tile(tile_start, g.batch, tile);
        const int first = cand_start[b] + (tile - tile_start[b]) * kTileRows;
        int nrows = cand_start[b + 1] - first;
        if (nrows > kTileRows) nrows = kTileRows;
        const bool split = chunk * 2 * kOcBlock + kOcBlock >= c_out_pad;
        const int oc0 = chunk * 2 * kOcBlock + (split ? 0 : half * kOcBlock);

        __syncthreads();  // previous item's readers of s_site / s_nbr are done
        if (threadIdx.x < kTileRows) {
            int c0 = 0, c1 = 0, c2 = 0;
            if (threadIdx.x < nrows) site_of(g, cand_lin[first + threadIdx.x], c0, c1, c2);
            s_site[threadIdx.x][0] = c0;
            s_site[threadIdx.x][1] = c1;
            s_site[threadIdx.x][2] = c2;
        }

        double acc[OCB];
#pragma unroll
        for (int o = 0; o < OCB; ++o) acc[o] = 0.0;

        for (int tc = 0; tc < g.T; tc += kTapChunk) {
            const int tmax = (g.T - tc) < kTapChunk ? (g.T - tc) : kTapChunk;
            const unsigned act = active_taps(tap_active, tc, tmax);
            __syncthreads();
            // element i = line segment * 128 + row: the chunk's taps are cut into runs that share (t0, t1); a run's
            // neighbours are adjacent sites and are resolved from one pair of bitmap words
            {
                const int l_first = tc / g.K[2];
                const int n_seg = (tc + tmax - 1) / g.K[2] - l_first + 1;
                for (int i = threadIdx.x; i < kTileRows * n_seg; i += 256) {
                    const int r = i & (kTileRows - 1), l = l_first + (i >> 7);
                    const int ta = tc > l * g.K[2] ? tc : l * g.K[2];
                    const int tb = (tc + tmax) < (l + 1) * g.K[2] ? (tc + tmax) : (l + 1) * g.K[2];
                    const int t0 = l / g.K[1], t1 = l - t0 * g.K[1];
                    int* dst = &s_nbr[r][ta - tc];
                    lookup_line(g, occ, occ_prefix, nnz_in, r < nrows, b, s_site[r][0], s_site[r][1], s_site[r][2], t0,
                                t1, ta - l * g.K[2], tb - ta, act >> (ta - tc), [&](int k, int n) { dst[k] = n; });
                }
            }
            __syncthreads();
            if (oc0 < c_out_pad && row < nrows) {
                for (int tt = split ? half : 0; tt < tmax; tt += split ? 2 : 1) {
                    const int n = s_nbr[row][tt];
                    if (n < 0) continue;
                    const float* __restrict__ x = feats + (size_t)n * c_in;
                    const double* __restrict__ wt = wp + ((size_t)(tc + tt) * c_in) * c_out_pad + oc0;
                    for (int ic0 = 0; ic0 < c_in; ic0 += CH) {
                        float xv[CH];
                        if constexpr (CH == 8) {
                            const float4 u = *(const float4*)(x + ic0), v = *(const float4*)(x + ic0 + 4);
                            xv[0] = u.x; xv[1] = u.y; xv[2] = u.z; xv[3] = u.w;
                            xv[4] = v.x; xv[5] = v.y; xv[6] = v.z; xv[7] = v.w;
                        } else if constexpr (CH == 4) {
                            const float4 u = *(const float4*)(x + ic0);
                            xv[0] = u.x; xv[1] = u.y; xv[2] = u.z; xv[3] = u.w;
                        } else if constexpr (CH == 2) {
                            const float2 u = *(const float2*)(x + ic0);
                            xv[0] = u.x; xv[1] = u.y;
                        } else {
                            xv[0] = x[ic0];
                        }
                        // two channels' weights (64 scalar registers) in flight at a time: more would spill
#pragma unroll
                        for (int j2 = 0; j2 < CH; j2 += 2) {
                            const double* __restrict__ wr = wt + (size_t)(ic0 + j2) * c_out_pad;
                            double wa[OCB], wb[OCB];
#pragma unroll
                            for (int o = 0; o < OCB; ++o) wa[o] = wr[o];
                            if constexpr (CH > 1) {
#pragma unroll
                                for (int o = 0; o < OCB; ++o) wb[o] = wr[c_out_pad + o];
                            }
                            const double xa = (double)xv[j2];
#pragma unroll
                            for (int o = 0; o < OCB; ++o) acc[o] = fma(xa, wa[o], acc[o]);
                            if constexpr (CH > 1) {
                                const double xb = (double)xv[j2 + 1];
#pragma unroll
                                for (int o = 0; o < OCB; ++o) acc[o] = fma(xb, wb[o], acc[o]);
                            }
                            // keeps the compiler from hoisting the next pair's scalar loads above this point
                            asm volatile("" ::: "memory");
                        }
                    }
                }
            }
        }
        if (split) {  // even taps (first half) + odd taps (second half)
            double* s_acc = reinterpret_cast<double*>(&s_nbr[row][0]);
            __syncthreads();  // the last chunk's neighbour rows have been read
            if (half == 1) {
#pragma unroll
                for (int o = 0; o < OCB; ++o) s_acc[o] = acc[o];
            }
            __syncthreads();
            if (half == 0) {
#pragma unroll
                for (int o = 0; o < OCB; ++o) acc[o] += s_acc[o];
            }
        }
        if (oc0 < c_out_pad && (!split || half == 0)) {
#pragma unroll
            for (int o = 0; o < OCB; ++o) {
                const int oc = oc0 + o;
                if (oc < c_out) {
                    float v = (row < nrows) ? (float)acc[o] : 0.0f;
                    if (bias && v != 0.0f) v += bias[oc];
                    resp[((size_t)tile * c_out + oc) * kTileRows + row] = v;
                }
            }
        }
    }
}

// One input channel (the first layer of every network), or eight: a neighbour costs few values and multiply-adds, so what
// the forms above spend per tap and wave, whether a lane has the neighbour or not, is nearly all of their time.  Here a
// thread owns a site and walks the neighbours that it has, lowest tap first, several in flight, with the weights of its tap
// from LDS: a wave takes as many rounds as its richest site has neighbours (three of 27 taps on scattered sites, about
// half of them on surfaces).  The sums are fp64 and in tap order.  One input and eight output channels, against the forms
// above: 256^3 scattered, 1.7 M sites, 104 -> 35 us; 28 x 28 x 1024 29 -> 17.5; one 28 x 28 image 9.8 -> 5.3.  By density
// (share of occupied input sites; the stage by events), 1 -> 8 and 1 -> 16 on 128^3: 0.02 58 -> 25 and 68 -> 29, 0.3 126 ->
// 60 and 150 -> 77, all occupied 128 -> 78 and 154 -> 105; 16^3, 32 tiles: 14.7 -> 8.3 and 15.2 -> 9.4, 14.6 -> 10.9 and
// 14.9 -> 12.9, all occupied 14.7 -> 12.8 and 15.1 -> 15.6, the one place where it is the slower.
// Eight input channels are bound by the weights' way out of LDS (512 bytes a lane and neighbour): 128^3 x 4, 8 -> 8,
// 91 -> 57 us.  By density, 0.02 / 0.3 / all: 32^3 x 4 26 / 52 / 51 -> 13 / 23 / 30, 64^3 x 4, 2 k tiles, - / 44 / 45 -> - /
// 31 / 42; surfaces of 0.05 to 0.2 on 64^3 x 8 0.72 to 1.01 times.  It loses where the forms above do their best: with at
// most 256 tiles in use (surfaces on 40^3 x 4, 189 tiles, 304 of capacity, 21.7 against 24.0; 16^3 x 8, all occupied, 21.9
// against 25.3) and, with nearly all of 27 neighbours there, as a surface's gradient rows are, up to 512 (adjoint, 40^3 x 4,
// 300 tiles, 27.3 against 30.0; 512 tiles 27.2 against 29.8, 640 42.7 against 31.7): hence the line at twice the 32-row
// form's items, and at its items for at most nine taps (28 x 28 x 64, all occupied, 16.4 -> 13.5; adjoint, 28 x 28 x 200,
// 26.4 -> 15.5) and inputs of less than a row per six candidates (16^3 x 8, 0.06 occupied, 21.6 -> 14.3).  Past it only the
// adjoint on 1040 to 1250 tiles is slower, by 1.05 to 1.1.  Sixteen output channels double that bound, and on the dense
// surfaces that follow a pooling lose to the streaming form (64^3 x 4: 57 -> 80 us); they keep the forms above.
// Tiles: a workgroup's two are neighbours (SPREAD = 0), which share most of the rows they gather; two that the whole launch
// lies between take 1.02 to 1.35 times as long.  The adjoint convolution is followed by a filter gradient that gathers the
// same rows, tile i on XCD i % 8: there the tiles are spread likewise, so that it finds them in its L2 (8 -> 1 channels'
// layer, 40^3 x 4, 141 k rows: filter gradient 132 -> 102 us, 104 behind the streaming form).  (An argument instead of an
// instance took sixteen more registers of 1 -> 16 and 10 % of its time.)
constexpr int kOneLines = 9;  // filter lines at most (and 32 taps)
constexpr long long kOneBlocks = 256 * 16;
template <int CI /* input channels: 1 or 8 */, int OCB /* output channels at most: 8 or 16 */, int SPREAD>
__global__ __launch_bounds__(256) void k_conv_valu_one(Geom g, const unsigned long long* __restrict__ occ,
                                                       const unsigned* __restrict__ occ_prefix, long long nnz_in,
                                                       const float* __restrict__ feats, const double* __restrict__ wp,
                                                       int c_out, int c_out_pad, const float* __restrict__ bias,
                                                       const int* __restrict__ tap_active,
                                                       const unsigned* __restrict__ cand_lin,
                                                       const int* __restrict__ cand_start,
                                                       const int* __restrict__ tile_start,
                                                       const Counters* __restrict__ ctr, float* __restrict__ resp) {
    constexpr int U = CI == 1 ? 4 : 2;  // neighbours in flight
    constexpr int WS = CI * OCB + 2;  // (lanes at different taps read different banks)
    __shared__ __align__(16) double s_w[32 * WS];
    __shared__ unsigned s_row[kOneLines][256];  // row of the first occupied site on the thread's window of each line
    __shared__ unsigned char s_line[32], s_k[32];  // line of a tap and its place there
    const int T = g.T, K1 = g.K[1], K2 = g.K[2], n_lines = g.K[0] * K1;
    const int tid = threadIdx.x, n_tiles = (int)ctr->n_tiles;
    const unsigned act = active_taps(tap_active, 0, T);
    for (int i = tid; i < T * CI * OCB; i += 256)
        s_w[i / (CI * OCB) * WS + i % (CI * OCB)] = wp[(size_t)(i / OCB) * c_out_pad + i % OCB];
    if (tid < T) {
        s_line[tid] = (unsigned char)(tid / K2);
        s_k[tid] = (unsigned char)(tid % K2);
    }
    __syncthreads();
    const int first_tile = SPREAD ? (int)blockIdx.x + (tid >> 7) * (int)gridDim.x : (int)blockIdx.x * 2 + (tid >> 7);
    for (int tile = first_tile; tile < n_tiles; tile += (int)gridDim.x * 2) {  // (uniform in the wave)
        const int b = sample_of_tile(tile_start, g.batch, tile), r = tid & (kTileRows - 1);
        const int cand = cand_start[b] + (tile - tile_start[b]) * kTileRows + r;
        const bool live = cand < cand_start[b + 1];
        int c0 = 0, c1 = 0, c2 = 0;
        if (live) site_of(g, cand_lin[cand], c0, c1, c2);
        // ---- occupancy of the sites that the taps look at: bit t = tap t's (lookup_line, all lines' loads in flight)
        const int q2s = c2 - g.H[2];
        int k_lo, k_hi;
        taps_on_line(g.E[2], c2, -g.H[2], K2, k_lo, k_hi);
        const unsigned w_last = (unsigned)g.batch * (unsigned)g.Wps - 1u;
        const unsigned on_line = live && k_hi > k_lo ? (~0u >> (32 - (k_hi - k_lo))) << k_lo : 0u;
        unsigned raw = 0;
        constexpr int LB = 3;  // lines whose loads are in flight together
        for (int line0 = 0; line0 < n_lines; line0 += LB) {
            unsigned long long word_a[LB], word_b[LB];
            unsigned pre_a[LB], pre_b[LB], p[LB];
            bool ok[LB];
#pragma unroll
            for (int i = 0; i < LB; ++i) {
                const int line = line0 + i < n_lines ? line0 + i : n_lines - 1;
                const int t0 = line / K1, t1 = line - t0 * K1;
                const int q0 = c0 + t0 - g.H[0], q1 = c1 + t1 - g.H[1];
                ok[i] = on_line != 0u && (unsigned)q0 < (unsigned)g.E[0] && (unsigned)q1 < (unsigned)g.E[1];
                const unsigned bit = ok[i] ? (unsigned)((q0 * g.E[1] + q1) * g.E[2] + q2s + k_lo) : 0u;
                p[i] = bit & 63u;
                const unsigned w0 = (unsigned)b * (unsigned)g.Wps + (bit >> 6);
                const unsigned wa = w0 < w_last ? w0 : w_last, wb = wa < w_last ? wa + 1u : wa;
                word_a[i] = occ[wa];
                word_b[i] = occ[wb];
                pre_a[i] = occ_prefix[wa];
                pre_b[i] = occ_prefix[wb];
            }
#pragma unroll
            for (int i = 0; i < LB; ++i) {
                const int line = line0 + i < n_lines ? line0 + i : n_lines - 1;  // (a line taken twice gives the same)
                const unsigned window = (unsigned)(word_a[i] >> p[i]) | (unsigned)((word_b[i] << 1) << (63u - p[i]));
                raw |= (ok[i] ? (window << k_lo) & on_line : 0u) << (line * K2);
                s_row[line][tid] = word_a[i] ? pre_a[i] + (unsigned)__popcll(word_a[i] & ((1ull << p[i]) - 1ull)) : pre_b[i];
            }
        }
        // ---- its neighbours, four at a time
        double acc[OCB];
#pragma unroll
        for (int o = 0; o < OCB; ++o) acc[o] = 0.0;
        const unsigned line_mask = K2 >= 32 ? ~0u : (1u << K2) - 1u;
        for (unsigned m = raw & act; m != 0u;) {
            int t[U];
            float x[U][CI];
#pragma unroll
            for (int j = 0; j < U; ++j) {
                t[j] = -1;
                if (m != 0u) {
                    const int tap = __builtin_ctz(m), line = s_line[tap], kk = s_k[tap];
                    m &= m - 1u;
                    const unsigned row = s_row[line][tid] + (unsigned)__popc((raw >> (tap - kk)) & line_mask & ((1u << kk) - 1u));
                    if (row < (unsigned)nnz_in) {  // (only an unsorted input can trip this guard)
                        t[j] = tap;
                        if constexpr (CI == 1) {
                            x[j][0] = feats[row];
                        } else {
                            const float4 u = *(const float4*)(feats + (size_t)row * CI), v = *(const float4*)(feats + (size_t)row * CI + 4);
                            x[j][0] = u.x; x[j][1] = u.y; x[j][2] = u.z; x[j][3] = u.w;
                            x[j][4] = v.x; x[j][5] = v.y; x[j][6] = v.z; x[j][7] = v.w;
                        }
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < U; ++j)
                if (t[j] >= 0) {
                    const double2* wr = (const double2*)(s_w + t[j] * WS);
#pragma unroll
                    for (int ic = 0; ic < CI; ++ic) {
                        const double xd = (double)x[j][ic];
#pragma unroll
                        for (int o = 0; o < OCB / 2; ++o) {
                            const double2 w = wr[ic * (OCB / 2) + o];
                            acc[2 * o] = fma(xd, w.x, acc[2 * o]);
                            acc[2 * o + 1] = fma(xd, w.y, acc[2 * o + 1]);
                        }
                    }
                }
        }
        float* dst = resp + (size_t)tile * c_out * kTileRows + r;
#pragma unroll
        for (int o = 0; o < OCB; ++o) {
            if (o >= c_out) break;
            float v = (float)acc[o];
            if (bias && v != 0.0f) v += bias[o];
            dst[(size_t)o * kTileRows] = v;
        }
    }
}

// Eight input channels on middling layers, where k_conv_valu_one's workgroups are one round of the chip and a call waits for
// the richest site of 64 in each: here four lanes share a site (its lines' look-ups, then every fourth neighbour; their sums
// added at the end), a wave takes sixteen sites at a time, and persistent workgroups, each XCD on a run of consecutive tiles,
// put the weights into LDS once.  It issues a third more vector instructions (each lane knows its site), so larger layers keep
// the other form.  Calls, 8 -> 8, 27 taps, against it: 32^3 x 4, sites in use from 0.03 occupied to all, 59 / 77 / 85 us ->
// 57 / 74 / 82, on surfaces 67 -> 56; 40^3 x 4, 2 k tiles, 76 / 101 / 112 -> 74 / 100 / 111, surfaces 87 -> 76; 64^3 x 2
// 95 / 134 / 413 -> 97 / 134 / 418, surfaces 110 -> 101; 64^3 x 4, 8 k tiles, 110 / 175 / 512 -> 116 / 185 / 522; with nine
// taps (100 x 100 x 16) 46 / 60 / 63 -> 44 / 61 / 66.  The nine-layer 32^3 network 595 -> 568.
constexpr long long kEightTiles = 3072;  // of capacity, at most
constexpr int kEightPerCu = 3;           // workgroups that run at once (80 registers)
constexpr int kEightThreads = 512;       // a tile: four lanes a site, sixteen sites a wave
__device__ __forceinline__ unsigned quad_swap1(unsigned x) { return (unsigned)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xf, 0xf, true); }
__device__ __forceinline__ unsigned quad_swap2(unsigned x) { return (unsigned)__builtin_amdgcn_mov_dpp((int)x, 0x4E, 0xf, 0xf, true); }
__device__ __forceinline__ double quad_swap1(double x) {
    return __hiloint2double((int)quad_swap1((unsigned)__double2hiint(x)), (int)quad_swap1((unsigned)__double2loint(x)));
}
__device__ __forceinline__ double quad_swap2(double x) {
    return __hiloint2double((int)quad_swap2((unsigned)__double2hiint(x)), (int)quad_swap2((unsigned)__double2loint(x)));
}
__global__ __launch_bounds__(kEightThreads, 6) void k_conv_valu_eight(Geom g, const unsigned long long* __restrict__ occ,
                                                         const unsigned* __restrict__ occ_prefix, long long nnz_in,
                                                         const float* __restrict__ feats, const double* __restrict__ wp,
                                                         int c_out, int c_out_pad, const float* __restrict__ bias,
                                                         const int* __restrict__ tap_active,
                                                         const unsigned* __restrict__ cand_lin,
                                                         const int* __restrict__ cand_start,
                                                         const int* __restrict__ tile_start,
                                                         const Counters* __restrict__ ctr, float* __restrict__ resp) {
    constexpr int CI = 8, OCB = 8, NT = kEightThreads, U = 2;  // U: neighbours in flight
    constexpr int WS = CI * OCB + 2;                           // (lanes at different taps read different banks)
    __shared__ __align__(16) double s_w[32 * WS];
    __shared__ unsigned s_row[NT / 64][kOneLines][16];  // row of the first occupied site on the site's window of each line
    __shared__ unsigned char s_line[32], s_k[32];       // line of a tap and its place there
    const int T = g.T, K1 = g.K[1], K2 = g.K[2], n_lines = g.K[0] * K1;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), j = tid & 3, q = (tid & 63) >> 2;
    const int n_tiles = (int)ctr->n_tiles;
    // XCD x (workgroups x, x + 8, ..) takes a run of consecutive tiles
    const int per = (n_tiles + kXcds - 1) / kXcds, base = ((int)blockIdx.x % kXcds) * per;
    const int first = base + (int)blockIdx.x / kXcds, last = min(base + per, n_tiles), step = (int)gridDim.x / kXcds;
    if (first >= last) return;
    const unsigned act = active_taps(tap_active, 0, T);
    {
        constexpr int NW = (32 * CI * OCB + NT - 1) / NT;
        double weight[NW];  // (all of a thread's loads in flight together)
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            const int e = tid + i * NT;
            weight[i] = e < T * CI * OCB ? wp[(size_t)(e / OCB) * c_out_pad + e % OCB] : 0.0;
        }
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            const int e = tid + i * NT;
            if (e < T * CI * OCB) s_w[e / (CI * OCB) * WS + e % (CI * OCB)] = weight[i];
        }
    }
    if (tid < T) {
        s_line[tid] = (unsigned char)(tid / K2);
        s_k[tid] = (unsigned char)(tid % K2);
    }
    __syncthreads();
    const unsigned line_mask = K2 >= 32 ? ~0u : (1u << K2) - 1u;
    for (int tile = first; tile < last; tile += step) {
        const int b = sample_of_tile(tile_start, g.batch, tile), r = wave * 16 + q;
        const int cand = cand_start[b] + (tile - tile_start[b]) * kTileRows + r;
        const bool live = cand < cand_start[b + 1];
        int c0 = 0, c1 = 0, c2 = 0;
        if (live) site_of(g, cand_lin[cand], c0, c1, c2);
        // ---- occupancy of the sites that the taps look at: bit t = tap t's (lookup_line, a lane every fourth line)
        const int q2s = c2 - g.H[2];
        int k_lo, k_hi;
        taps_on_line(g.E[2], c2, -g.H[2], K2, k_lo, k_hi);
        const unsigned w_last = (unsigned)g.batch * (unsigned)g.Wps - 1u;
        const unsigned on_line = live && k_hi > k_lo ? (~0u >> (32 - (k_hi - k_lo))) << k_lo : 0u;
        unsigned raw = 0;
        {
            constexpr int LB = (kOneLines + 3) / 4;
            unsigned long long word_a[LB], word_b[LB];
            unsigned pre_a[LB], pre_b[LB], p[LB];
            bool ok[LB];
#pragma unroll
            for (int i = 0; i < LB; ++i) {
                const int line = j + 4 * i;
                const int t0 = line / K1, t1 = line - t0 * K1;
                const int q0 = c0 + t0 - g.H[0], q1 = c1 + t1 - g.H[1];
                ok[i] = line < n_lines && on_line != 0u && (unsigned)q0 < (unsigned)g.E[0] && (unsigned)q1 < (unsigned)g.E[1];
                const unsigned bit = ok[i] ? (unsigned)((q0 * g.E[1] + q1) * g.E[2] + q2s + k_lo) : 0u;
                p[i] = bit & 63u;
                const unsigned w0 = (unsigned)b * (unsigned)g.Wps + (bit >> 6);
                const unsigned wa = w0 < w_last ? w0 : w_last, wb = wa < w_last ? wa + 1u : wa;
                word_a[i] = occ[wa];
                word_b[i] = occ[wb];
                pre_a[i] = occ_prefix[wa];
                pre_b[i] = occ_prefix[wb];
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // (the last tile's rows have been read)
#pragma unroll
            for (int i = 0; i < LB; ++i) {
                const int line = j + 4 * i;
                if (line >= n_lines) continue;
                const unsigned window = (unsigned)(word_a[i] >> p[i]) | (unsigned)((word_b[i] << 1) << (63u - p[i]));
                raw |= (ok[i] ? (window << k_lo) & on_line : 0u) << (line * K2);
                s_row[wave][line][q] = word_a[i] ? pre_a[i] + (unsigned)__popcll(word_a[i] & ((1ull << p[i]) - 1ull)) : pre_b[i];
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        raw |= quad_swap1(raw);
        raw |= quad_swap2(raw);
        // ---- the site's neighbours, every fourth to a lane, several in flight
        double acc[OCB];
#pragma unroll
        for (int o = 0; o < OCB; ++o) acc[o] = 0.0;
        unsigned m = raw & act;
        auto drop = [&](bool yes) { m = yes ? m & (m - 1u) : m; };
        drop(j > 0);
        drop(j > 1);
        drop(j > 2);
        while (m != 0u) {
            int t[U];
            float x[U][CI];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                t[u] = -1;
                if (m != 0u) {
                    const int tap = __builtin_ctz(m), line = s_line[tap], kk = s_k[tap];
                    const unsigned row = s_row[wave][line][q] + (unsigned)__popc((raw >> (tap - kk)) & line_mask & ((1u << kk) - 1u));
                    drop(true); drop(true); drop(true); drop(true);
                    if (row < (unsigned)nnz_in) {  // (only an unsorted input can trip this guard)
                        t[u] = tap;
                        const float4 a = *(const float4*)(feats + (size_t)row * CI), c = *(const float4*)(feats + (size_t)row * CI + 4);
                        x[u][0] = a.x; x[u][1] = a.y; x[u][2] = a.z; x[u][3] = a.w;
                        x[u][4] = c.x; x[u][5] = c.y; x[u][6] = c.z; x[u][7] = c.w;
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (t[u] >= 0) {
                    const double2* wr = (const double2*)(s_w + t[u] * WS);
#pragma unroll
                    for (int ic = 0; ic < CI; ++ic) {
                        const double xd = (double)x[u][ic];
#pragma unroll
                        for (int o = 0; o < OCB / 2; ++o) {
                            const double2 w = wr[ic * (OCB / 2) + o];
                            acc[2 * o] = fma(xd, w.x, acc[2 * o]);
                            acc[2 * o + 1] = fma(xd, w.y, acc[2 * o + 1]);
                        }
                    }
                }
        }
        // ---- the four lanes' sums: lane j ends with channels 4 (j & 1) + (j & 2) and the one after
        double half[4], sum[2];
#pragma unroll
        for (int o = 0; o < 4; ++o) {
            const double mine = (j & 1) ? acc[o + 4] : acc[o], other = (j & 1) ? acc[o] : acc[o + 4];
            half[o] = mine + quad_swap1(other);
        }
#pragma unroll
        for (int o = 0; o < 2; ++o) {
            const double mine = (j & 2) ? half[o + 2] : half[o], other = (j & 2) ? half[o] : half[o + 2];
            sum[o] = mine + quad_swap2(other);
        }
        const int o0 = 4 * (j & 1) + (j & 2);
        float* dst = resp + ((size_t)tile * c_out + o0) * kTileRows + r;
#pragma unroll
        for (int o = 0; o < 2; ++o)
            if (o0 + o < c_out) {
                float v = (float)sum[o];
                if (bias && v != 0.0f) v += bias[o0 + o];
                dst[(size_t)o * kTileRows] = v;
            }
    }
}

// Response tiles of a layer without input rows (candidate sites cannot exist either; kept for completeness).
__global__ __launch_bounds__(256) void k_conv_valu_empty(int c_out, const Counters* __restrict__ ctr,
                                                         float* __restrict__ resp) {
    const size_t n = (size_t)ctr->n_tiles * c_out * kTileRows;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        resp[i] = 0.0f;
}

typedef double f64x4 __attribute__((ext_vector_type(4)));

// Latency-oriented form of the vector kernel, for layers with at most `max_items` work items (about one per
// workgroup slot of the chip: the regime of the paper's own narrow networks on small grids).
// Work item = (tile, block of 32 output channels); thread = (row, 16 channels).  When the block has only 16
// channels (C_out <= 16, or the last block), the second half of the workgroup would idle: it then takes every
// other tap of the same 16 channels instead and the two partial sums are added through LDS (even taps + odd taps,
// a fixed order).
// What bounds a small layer is memory latency, not arithmetic, so nothing in the inner loop waits on global memory:
// the neighbour rows of a chunk of taps are looked up per filter line (adjacent sites share one pair of bitmap
// words), and the neighbours' values are gathered into LDS cooperatively (CH channels of TG taps at a time, every
// load independent of every other), together with the group's weights, one round ahead of the multiply-add phase
// that reads both from there.
// With CH >= 4 the multiply-add phase runs on the fp64 matrix cores instead (v_mfma_f64_16x16x4_f64, same fp64
// products and sums): wave w then owns rows 32 w .. 32 w + 31 and all of the chunk's channels, and the results go
// through LDS to the (row, 16 channels) threads that write them.  Reading a (tap, channel)'s 16 weights as an LDS
// broadcast per lane, as the thread-per-row form does, costs the LDS four times the cycles the FMAs take.
template <int CH /* input channels per gather: the largest of 8, 4, 2, 1 that divides C_in */>
__global__ __launch_bounds__(256) void k_conv_valu(Geom g, const unsigned long long* __restrict__ occ,
                                                   const unsigned* __restrict__ occ_prefix, long long nnz_in,
                                                   const float* __restrict__ feats, int c_in,
                                                   const double* __restrict__ wp, int c_out, int c_out_pad,
                                                   const float* __restrict__ bias,
                                                   const int* __restrict__ tap_active,
                                                   const unsigned* __restrict__ cand_lin,
                                                   const int* __restrict__ cand_start,
                                                   const int* __restrict__ tile_start,
                                                   const Counters* __restrict__ ctr, long long max_items,
                                                   float* __restrict__ resp) {
    constexpr int TG = (64 / CH) < kTapChunk ? (64 / CH) : kTapChunk;  // taps per gather
    constexpr int XS = TG * CH + 4;                                     // row stride of the gathered values
    __shared__ int s_nbr[kTileRows][kTapChunk + 1];
    __shared__ int s_site[kTileRows][3];
    __shared__ __align__(16) float s_x[kTileRows][XS];
    __shared__ __align__(16) double s_w[2][TG * CH][kOcBlock];  // the group's weights, per 16-channel block
    // partial sums of the second half when it shares the taps; reuses the gather buffer after the last group
    static_assert(sizeof(float) * XS >= sizeof(double) * (kOcBlock + 1), "gather rows hold a row of partial sums");
    double (*s_acc)[kOcBlock + 1] = reinterpret_cast<double (*)[kOcBlock + 1]>(&s_x[0][0]);

    const int n_tiles = (int)ctr->n_tiles;
    const int n_chunks = (c_out_pad + 2 * kOcBlock - 1) / (2 * kOcBlock);
    const long long n_items = (long long)n_tiles * n_chunks;
    if (n_items > max_items) return;  // the streaming kernel takes large layers
    const int row = threadIdx.x & (kTileRows - 1);
    const int half = __builtin_amdgcn_readfirstlane(threadIdx.x >> 7);  // which 16-channel block of the chunk

    for (long long item = blockIdx.x; item < n_items; item += gridDim.x) {
        const int tile = (int)(item / n_chunks);
        const int chunk = (int)(item - (long long)tile * n_chunks);
        const int b = sample_of_tile(tile_start, g.batch, tile);
        const int first = cand_start[b] + (tile - tile_start[b]) * kTileRows;
        int nrows = cand_start[b + 1] - first;
        if (nrows > kTileRows) nrows = kTileRows;
        // the chunk's second 16-channel block does not exist: both halves work on the first one, taps interleaved
        const bool split = chunk * 2 * kOcBlock + kOcBlock >= c_out_pad;
        const int oc0 = chunk * 2 * kOcBlock + (split ? 0 : half * kOcBlock);

        __syncthreads();  // previous item's readers of the shared arrays are done
        if (threadIdx.x < kTileRows) {
            int c0 = 0, c1 = 0, c2 = 0;
            if (threadIdx.x < nrows) site_of(g, cand_lin[first + threadIdx.x], c0, c1, c2);
            s_site[threadIdx.x][0] = c0;
            s_site[threadIdx.x][1] = c1;
            s_site[threadIdx.x][2] = c2;
        }

        double acc[kOcBlock];
#pragma unroll
        for (int o = 0; o < kOcBlock; ++o) acc[o] = 0.0;
        // matrix-core form (CH >= 4): wave w owns rows 32 w .. 32 w + 31 as two 16-row groups, times the chunk's
        // 16-channel blocks; lane (m, kq) holds output channel m of rows kq, 4 + kq, 8 + kq, 12 + kq of a group
        f64x4 macc[2][2];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int c = 0; c < 2; ++c) macc[a][c] = f64x4{0.0, 0.0, 0.0, 0.0};
        const int mi = threadIdx.x & 15, kq = (threadIdx.x >> 4) & 3;
        const int wrow = (threadIdx.x >> 6) * 32;  // first row of the wave

        for (int tc = 0; tc < g.T; tc += kTapChunk) {
            const int tmax = (g.T - tc) < kTapChunk ? (g.T - tc) : kTapChunk;
            const unsigned act = active_taps(tap_active, tc, tmax);
            __syncthreads();
            // ---- neighbour rows of (row, tap): element i = line segment * 128 + row; the chunk's taps are cut into
            //      runs that share (t0, t1), whose neighbours are resolved from one pair of bitmap words
            {
                const int l_first = tc / g.K[2];
                const int n_seg = (tc + tmax - 1) / g.K[2] - l_first + 1;
                for (int i = threadIdx.x; i < kTileRows * n_seg; i += 256) {
                    const int r = i & (kTileRows - 1), l = l_first + (i >> 7);
                    const int ta = tc > l * g.K[2] ? tc : l * g.K[2];
                    const int tb = (tc + tmax) < (l + 1) * g.K[2] ? (tc + tmax) : (l + 1) * g.K[2];
                    const int t0 = l / g.K[1], t1 = l - t0 * g.K[1];
                    int* dst = &s_nbr[r][ta - tc];
                    lookup_line(g, occ, occ_prefix, nnz_in, r < nrows, b, s_site[r][0], s_site[r][1], s_site[r][2], t0,
                                t1, ta - l * g.K[2], tb - ta, act >> (ta - tc), [&](int k, int n) { dst[k] = n; });
                }
            }
            // ---- rounds = (block of CH input channels) x (group of TG taps).  The global loads of round q + 1 (the
            //      neighbours' values and the group's weights) are in flight while round q multiplies.
            constexpr int GB = (kTileRows * TG) / 256;                   // (row, tap) pairs a thread gathers
            constexpr int WB = (2 * TG * CH * kOcBlock + 255) / 256;     // weights a thread stages
            const int n_tg = (tmax + TG - 1) / TG;
            const int n_rounds = (c_in / CH) * n_tg;
            float xv[GB][CH];
            double wv[WB];
            auto fetch = [&](int q) {
                const int ic0 = (q / n_tg) * CH, tg0 = (q % n_tg) * TG;
                const int tg_n = (tmax - tg0) < TG ? (tmax - tg0) : TG;
#pragma unroll
                for (int m = 0; m < GB; ++m) {
                    const int e = threadIdx.x + m * 256;
                    const int r = e & (kTileRows - 1), tg = e >> 7;
                    const int n = (tg < tg_n) ? s_nbr[r][tg0 + tg] : -1;
                    const float* __restrict__ xp = feats + (size_t)(n < 0 ? 0 : n) * c_in + ic0;
                    if constexpr (CH == 8) {
                        const float4 u = *(const float4*)xp, v = *(const float4*)(xp + 4);
                        xv[m][0] = u.x; xv[m][1] = u.y; xv[m][2] = u.z; xv[m][3] = u.w;
                        xv[m][4] = v.x; xv[m][5] = v.y; xv[m][6] = v.z; xv[m][7] = v.w;
                    } else if constexpr (CH == 4) {
                        const float4 u = *(const float4*)xp;
                        xv[m][0] = u.x; xv[m][1] = u.y; xv[m][2] = u.z; xv[m][3] = u.w;
                    } else if constexpr (CH == 2) {
                        const float2 u = *(const float2*)xp;
                        xv[m][0] = u.x; xv[m][1] = u.y;
                    } else {
                        xv[m][0] = xp[0];
                    }
                    // a site without this neighbour multiplies zeros: the multiply-add phase has no per-row branch
#pragma unroll
                    for (int j = 0; j < CH; ++j) xv[m][j] = n < 0 ? 0.0f : xv[m][j];
                }
                // the group's weights: element e = (hb, tg * CH + j, o) <- w[tap tg][ic0 + j][16 * hb + o of the chunk]
#pragma unroll
                for (int m = 0; m < WB; ++m) {
                    const int e = threadIdx.x + m * 256;
                    const int o = e & (kOcBlock - 1), tj = (e >> 4) % (TG * CH), hb = e / (TG * CH * kOcBlock);
                    const int tg = tj / CH, j = tj - tg * CH;
                    const int oc = chunk * 2 * kOcBlock + hb * kOcBlock + o;
                    const bool ok = e < 2 * TG * CH * kOcBlock && tg < tg_n && oc < c_out_pad;
                    const size_t at = ok ? ((size_t)(tc + tg0 + tg) * c_in + ic0 + j) * c_out_pad + oc : 0;
                    const double v = wp[at];
                    wv[m] = ok ? v : 0.0;
                }
            };
            auto commit = [&]() {
#pragma unroll
                for (int m = 0; m < GB; ++m) {
                    const int e = threadIdx.x + m * 256;
                    const int r = e & (kTileRows - 1), tg = e >> 7;
#pragma unroll
                    for (int j = 0; j < CH; ++j) s_x[r][tg * CH + j] = xv[m][j];
                }
#pragma unroll
                for (int m = 0; m < WB; ++m) {
                    const int e = threadIdx.x + m * 256;
                    if (e < 2 * TG * CH * kOcBlock) (&s_w[0][0][0])[e] = wv[m];
                }
            };
            __syncthreads();  // s_nbr complete
            fetch(0);
            for (int q = 0; q < n_rounds; ++q) {
                const int tg0 = (q % n_tg) * TG;
                const int tg_n = (tmax - tg0) < TG ? (tmax - tg0) : TG;
                __syncthreads();  // the previous round's readers of s_x / s_w are done
                commit();
                __syncthreads();
                if (q + 1 < n_rounds) fetch(q + 1);
                if constexpr (CH >= 4) {
                    // ---- multiply-add on the matrix cores in fp64: per tap and four input channels, the wave's 32
                    //      rows' values (A, 16 x 4 per row group; zeros where a row lacks the neighbour) times the
                    //      weights (B, 4 x 16 per channel block)
                    unsigned live = 0;
#pragma unroll
                    for (int tg = 0; tg < TG; ++tg) {
                        const bool has = tg < tg_n && s_nbr[wrow + (threadIdx.x & 31)][tg0 + tg] >= 0;
                        if (__ballot(has) != 0ull) live |= 1u << tg;
                    }
                    for (int tg = 0; tg < tg_n; ++tg) {
                        if (!((live >> tg) & 1u)) continue;
#pragma unroll
                        for (int jb = 0; jb < CH / 4; ++jb) {
                            const int tj = tg * CH + jb * 4 + kq;
                            const double a0 = (double)s_x[wrow + mi][tj], a1 = (double)s_x[wrow + 16 + mi][tj];
                            const double b0 = s_w[0][tj][mi];
                            macc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, macc[0][0], 0, 0, 0);
                            macc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, macc[1][0], 0, 0, 0);
                            if (!split) {
                                const double b1 = s_w[1][tj][mi];
                                macc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, macc[0][1], 0, 0, 0);
                                macc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, macc[1][1], 0, 0, 0);
                            }
                        }
                    }
                    continue;
                }
                // ---- multiply-add: values and weights from LDS (the weights are a broadcast read).  A tap is skipped
                //      when no row of the wave has that neighbour; the weights of input channel j + 1 are read while
                //      channel j multiplies (the fences keep the compiler from sinking the reads to their uses).
                if (oc0 < c_out_pad) {
                    const int hb = split ? 0 : half;
                    unsigned live = 0;
#pragma unroll
                    for (int tg = 0; tg < TG; ++tg) {
                        const bool has = tg < tg_n && s_nbr[row][tg0 + tg] >= 0;
                        if (__ballot(has) != 0ull) live |= 1u << tg;
                    }
                    auto read_w = [&](double (&dst)[kOcBlock], int tj) {
                        const double2* p = reinterpret_cast<const double2*>(&s_w[hb][tj][0]);
#pragma unroll
                        for (int o = 0; o < kOcBlock / 2; ++o) {
                            const double2 v = p[o];
                            dst[2 * o] = v.x;
                            dst[2 * o + 1] = v.y;
                        }
                    };
                    auto mul_add = [&](float x, const double (&wr)[kOcBlock]) {
                        const double xd = (double)x;
#pragma unroll
                        for (int o = 0; o < kOcBlock; ++o) acc[o] = fma(xd, wr[o], acc[o]);
                    };
                    for (int tg = split ? half : 0; tg < tg_n; tg += split ? 2 : 1) {
                        if (!((live >> tg) & 1u)) continue;
                        float xf[CH];
                        if constexpr (CH >= 4) {
#pragma unroll
                            for (int j = 0; j < CH; j += 4) {
                                const float4 u = *reinterpret_cast<const float4*>(&s_x[row][tg * CH + j]);
                                xf[j] = u.x; xf[j + 1] = u.y; xf[j + 2] = u.z; xf[j + 3] = u.w;
                            }
                        } else {
#pragma unroll
                            for (int j = 0; j < CH; ++j) xf[j] = s_x[row][tg * CH + j];
                        }
                        double wa[kOcBlock], wb[kOcBlock];
                        read_w(wa, tg * CH);
#pragma unroll
                        for (int j = 0; j < CH; j += 2) {
                            if (j + 1 < CH) read_w(wb, tg * CH + j + 1);
                            __builtin_amdgcn_sched_barrier(0);
                            mul_add(xf[j], wa);
                            __builtin_amdgcn_sched_barrier(0);
                            if (j + 1 < CH) {
                                if (j + 2 < CH) read_w(wa, tg * CH + j + 2);
                                __builtin_amdgcn_sched_barrier(0);
                                mul_add(xf[j + 1], wb);
                                __builtin_amdgcn_sched_barrier(0);
                            }
                        }
                    }
                }
            }
        }
        if constexpr (CH >= 4) {
            // ---- results to LDS (over the gather buffer), so that a thread can write a row's channels as below
            static_assert(XS >= 2 * kOcBlock + 1, "a gather row holds a row of results");
            __syncthreads();  // the last round's values have been read
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int c = 0; c < 2; ++c)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        s_x[wrow + a * 16 + 4 * v + kq][c * kOcBlock + mi] = (float)macc[a][c][v];
            __syncthreads();
            if (oc0 < c_out_pad && (!split || half == 0)) {
#pragma unroll
                for (int o = 0; o < kOcBlock; ++o) {
                    const int oc = oc0 + o;
                    if (oc < c_out) {
                        float v = (row < nrows) ? s_x[row][(split ? 0 : half) * kOcBlock + o] : 0.0f;
                        if (bias && v != 0.0f) v += bias[oc];
                        resp[((size_t)tile * c_out + oc) * kTileRows + row] = v;
                    }
                }
            }
            continue;
        }
        if (split) {  // even taps (first half) + odd taps (second half)
            __syncthreads();  // the last group's values have been read
            if (half == 1) {
#pragma unroll
                for (int o = 0; o < kOcBlock; ++o) s_acc[row][o] = acc[o];
            }
            __syncthreads();
            if (half == 0) {
#pragma unroll
                for (int o = 0; o < kOcBlock; ++o) acc[o] += s_acc[row][o];
            }
        }
        if (oc0 < c_out_pad && (!split || half == 0)) {
#pragma unroll
            for (int o = 0; o < kOcBlock; ++o) {
                const int oc = oc0 + o;
                if (oc < c_out) {
                    float v = (row < nrows) ? (float)acc[o] : 0.0f;
                    if (bias && v != 0.0f) v += bias[oc];
                    resp[((size_t)tile * c_out + oc) * kTileRows + row] = v;
                }
            }
        }
    }
}

// The same kernel shape for the smallest layers (a few hundred tiles: the deep, pooled layers of the paper's
// networks; narrow ones of up to a thousand), where 128-row work items would leave most of the chip idle.  Work item = (quarter of a tile = 32 rows,
// block of 32 output channels).  The four waves of the workgroup share the taps (wave w takes taps w, w + 4, ...);
// A round covers all taps of the chunk for CH input channels, so that a 3^d filter over 24 channels takes three
// rounds.  CH >= 4: a wave multiplies its taps for all 32 rows and channels on the fp64 matrix cores
// (v_mfma_f64_16x16x4_f64) and the four waves' partial sums are added through LDS in the order of the waves.
// CH = 2: the two halves of a wave take the two 16-channel blocks, or, when there is only one, every other input
// channel, with fp64 FMAs; the eight partial sums per output are added through LDS in a fixed order.
// For the matrix cores a round's weights lie in LDS as the fp32 numbers that they are and are widened at the product: with eight
// channels and two blocks an item takes 70 KB, two workgroups to a compute unit (103 KB and one with fp64 weights): 56 x 56 x 4,
// calls in us, before and after: 16 -> 24 54 / 48, 16 -> 64 66 / 58, 25 taps, 24 -> 24 70 / 58, 16 -> 64 87 / 69; the same time
// where one round of workgroups is enough.  Three to a unit with one block (168 registers, some spilled) gains 5 % or loses 3,
// as the rounds fall: not taken.
// NB = 1: items of one 16-channel block, half the weights to load: 16^3 x 4, 16 -> 16, 512 items, call 71 -> 59 us, 8 -> 8
// 61 -> 53, 8^3 x 4, 24 -> 24 (two blocks, 160 items) 64 -> 56 (against two blocks and one workgroup to a unit).
template <int CH /* 8, 4 or 2 */, int NB /* 16-channel blocks of a work item: 2, or 1 */>
__global__ __launch_bounds__(256, 2) void k_conv_valu_small(Geom g, const unsigned long long* __restrict__ occ,
                                                         const unsigned* __restrict__ occ_prefix, long long nnz_in,
                                                         const float* __restrict__ feats, int c_in,
                                                         const double* __restrict__ wp, int c_out, int c_out_pad,
                                                         const float* __restrict__ bias,
                                                         const int* __restrict__ tap_active,
                                                         const unsigned* __restrict__ cand_lin,
                                                         const int* __restrict__ cand_start,
                                                         const int* __restrict__ tile_start,
                                                         const Counters* __restrict__ ctr, float* __restrict__ resp) {
    constexpr int R = 32;                    // rows per work item
    constexpr int Q = kTileRows / R;         // work items per tile and channel block
    constexpr int XS = kTapChunk * CH + 4;   // row stride of the gathered values
    constexpr int GB = (R * kTapChunk) / 256;                     // (row, tap) pairs a thread gathers per round
    constexpr int WB = (NB * kTapChunk * CH * kOcBlock) / 256;    // weights a thread stages per round
    // One block of memory: the round's weights per 16-channel block, then the gathered values, whose padding holds the rows'
    // sites; after the last round the partial sums of the waves (CH = 2: of the eight (wave, half) pairs).
    using WT = std::conditional_t<(CH >= 4), float, double>;
    constexpr int kWBytes = NB * kTapChunk * CH * kOcBlock * (int)sizeof(WT);
    constexpr int kXBytes = R * XS * 4;
    constexpr int kRedBytes = (CH >= 4 ? 4 * R * (NB * kOcBlock + 1) : 8 * R * (kOcBlock + 1)) * 8;
    __shared__ __align__(16) unsigned char s_mem[kWBytes + kXBytes > kRedBytes ? kWBytes + kXBytes : kRedBytes];
    __shared__ int s_nbr[kTapChunk][R];
    WT (*s_w)[kTapChunk * CH][kOcBlock] = reinterpret_cast<WT (*)[kTapChunk * CH][kOcBlock]>(&s_mem[0]);
    float (*s_x)[XS] = reinterpret_cast<float (*)[XS]>(&s_mem[kWBytes]);
    double (*s_red)[R][kOcBlock + 1] = reinterpret_cast<double (*)[R][kOcBlock + 1]>(&s_mem[0]);
    auto site = [&](int r) { return reinterpret_cast<int*>(&s_x[r][kTapChunk * CH]); };

    const int n_tiles = (int)ctr->n_tiles;
    const int n_chunks = (c_out_pad + NB * kOcBlock - 1) / (NB * kOcBlock);
    const long long n_items = (long long)n_tiles * n_chunks * Q;
    const int row = threadIdx.x & (R - 1);
    const int sl = threadIdx.x >> 5;          // (wave, half of the wave)
    const int lh = sl & 1;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    for (long long item = blockIdx.x; item < n_items; item += gridDim.x) {
        const int quarter = (int)(item % Q);
        const long long tc_item = item / Q;
        const int tile = (int)(tc_item / n_chunks);
        const int chunk = (int)(tc_item - (long long)tile * n_chunks);
        const int b = sample_of_tile(tile_start, g.batch, tile);
        const int first = cand_start[b] + (tile - tile_start[b]) * kTileRows + quarter * R;
        int nrows = cand_start[b + 1] - first;
        if (nrows > R) nrows = R;
        if (nrows < 0) nrows = 0;
        // the chunk's second 16-channel block does not exist: the halves of a wave share the input channels
        const bool split = NB == 1 || chunk * NB * kOcBlock + kOcBlock >= c_out_pad;
        const int hb = split ? 0 : lh;

        double acc[kOcBlock];
#pragma unroll
        for (int o = 0; o < kOcBlock; ++o) acc[o] = 0.0;
        // matrix-core form (CH >= 4): [16-row group][16-channel block]; lane (m, kq) holds output channel m of rows
        // kq, 4 + kq, 8 + kq, 12 + kq (the fp64 instruction's result layout)
        f64x4 macc[2][NB];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int c = 0; c < NB; ++c) macc[a][c] = f64x4{0.0, 0.0, 0.0, 0.0};
        const int mi = threadIdx.x & 15, kq = (threadIdx.x >> 4) & 3;

        __syncthreads();  // previous item's readers of the shared arrays are done
        if (nrows > 0) {  // (uniform) a quarter without rows only writes its zeros
            if (threadIdx.x < R) {
                int c0 = 0, c1 = 0, c2 = 0;
                if (threadIdx.x < nrows) site_of(g, cand_lin[first + threadIdx.x], c0, c1, c2);
                site(threadIdx.x)[0] = c0;
                site(threadIdx.x)[1] = c1;
                site(threadIdx.x)[2] = c2;
            }
            for (int tc = 0; tc < g.T; tc += kTapChunk) {
                const int tmax = (g.T - tc) < kTapChunk ? (g.T - tc) : kTapChunk;
                const int n_rounds = c_in / CH;
                float xv[GB][CH];
                WT wv[WB];
                // the round's weights: element e = (block hb, tap tg, channel j, o) <- w[tc + tg][ic0 + j][16 hb + o]
                auto fetch_w = [&](int q) {
                    const int ic0 = q * CH;
#pragma unroll
                    for (int m = 0; m < WB; ++m) {
                        const int e = threadIdx.x + m * 256;
                        const int o = e & (kOcBlock - 1), tj = (e >> 4) % (kTapChunk * CH);
                        const int hbw = e / (kTapChunk * CH * kOcBlock);
                        const int tg = tj / CH, j = tj - tg * CH;
                        const int oc = chunk * NB * kOcBlock + hbw * kOcBlock + o;
                        const bool ok = tg < tmax && oc < c_out_pad;
                        const size_t at = ok ? ((size_t)(tc + tg) * c_in + ic0 + j) * c_out_pad + oc : 0;
                        const WT v = (WT)wp[at];  // (an fp32 number, whatever it is held in)
                        wv[m] = ok ? v : (WT)0;
                    }
                };
                // the neighbours' values; a site without the neighbour multiplies zeros
                auto fetch_x = [&](int q) {
                    const int ic0 = q * CH;
#pragma unroll
                    for (int m = 0; m < GB; ++m) {
                        const int e = threadIdx.x + m * 256;
                        const int r = e & (R - 1), tg = e >> 5;
                        const int n = (tg < tmax) ? s_nbr[tg][r] : -1;
                        const float* __restrict__ xp = feats + (size_t)(n < 0 ? 0 : n) * c_in + ic0;
                        if constexpr (CH == 8) {
                            const float4 u = *(const float4*)xp, v = *(const float4*)(xp + 4);
                            xv[m][0] = u.x; xv[m][1] = u.y; xv[m][2] = u.z; xv[m][3] = u.w;
                            xv[m][4] = v.x; xv[m][5] = v.y; xv[m][6] = v.z; xv[m][7] = v.w;
                        } else if constexpr (CH == 4) {
                            const float4 u = *(const float4*)xp;
                            xv[m][0] = u.x; xv[m][1] = u.y; xv[m][2] = u.z; xv[m][3] = u.w;
                        } else {
                            const float2 u = *(const float2*)xp;
                            xv[m][0] = u.x; xv[m][1] = u.y;
                        }
#pragma unroll
                        for (int j = 0; j < CH; ++j) xv[m][j] = n < 0 ? 0.0f : xv[m][j];
                    }
                };
                auto commit = [&]() {
#pragma unroll
                    for (int m = 0; m < GB; ++m) {
                        const int e = threadIdx.x + m * 256;
                        const int r = e & (R - 1), tg = e >> 5;
#pragma unroll
                        for (int j = 0; j < CH; ++j) s_x[r][tg * CH + j] = xv[m][j];
                    }
#pragma unroll
                    for (int m = 0; m < WB; ++m) (&s_w[0][0][0])[threadIdx.x + m * 256] = wv[m];
                };
                const unsigned act = active_taps(tap_active, tc, tmax);
                fetch_w(0);  // does not depend on the neighbours: in flight during the look-ups
                __syncthreads();  // the sites are written; the previous chunk's readers of s_nbr are done
                {
                    const int l_first = tc / g.K[2];
                    const int n_seg = (tc + tmax - 1) / g.K[2] - l_first + 1;
                    for (int i = threadIdx.x; i < R * n_seg; i += 256) {
                        const int r = i & (R - 1), l = l_first + (i >> 5);
                        const int ta = tc > l * g.K[2] ? tc : l * g.K[2];
                        const int tb = (tc + tmax) < (l + 1) * g.K[2] ? (tc + tmax) : (l + 1) * g.K[2];
                        const int t0 = l / g.K[1], t1 = l - t0 * g.K[1];
                        int* dst = &s_nbr[ta - tc][r];
                        lookup_line(g, occ, occ_prefix, nnz_in, r < nrows, b, site(r)[0], site(r)[1], site(r)[2],
                                    t0, t1, ta - l * g.K[2], tb - ta, act >> (ta - tc),
                                    [&](int k, int n) { dst[k * R] = n; });
                    }
                }
                __syncthreads();  // s_nbr complete
                fetch_x(0);
                // taps of the chunk that some row of this wave has
                unsigned live = 0;
                for (int tg = wave; tg < tmax; tg += 4)
                    if (__ballot(s_nbr[tg][row] >= 0) != 0ull) live |= 1u << tg;
                for (int q = 0; q < n_rounds; ++q) {
                    __syncthreads();  // the previous round's readers of s_x / s_w are done
                    commit();
                    __syncthreads();
                    if (q + 1 < n_rounds) {
                        fetch_w(q + 1);
                        fetch_x(q + 1);
                    }
                    if constexpr (CH >= 4) {
                        // ---- multiply-add on the matrix cores in fp64: per tap and four input channels, the 32
                        //      rows' values (A, 16 x 4 per row group; zeros where a row lacks the neighbour) times
                        //      the weights (B, 4 x 16 per channel block).  Two 8-byte operand reads feed 1024
                        //      multiply-adds, where the vector form reads 128 bytes of weights per lane for 16.
                        for (int tg = wave; tg < tmax; tg += 4) {
                            if (!((live >> tg) & 1u)) continue;
#pragma unroll
                            for (int jb = 0; jb < CH / 4; ++jb) {
                                const int tj = tg * CH + jb * 4 + kq;
                                const double a0 = (double)s_x[mi][tj], a1 = (double)s_x[16 + mi][tj];
                                const double b0 = (double)s_w[0][tj][mi];
                                macc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, macc[0][0], 0, 0, 0);
                                macc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, macc[1][0], 0, 0, 0);
                                if constexpr (NB > 1)
                                    if (!split) {
                                        const double b1 = (double)s_w[1][tj][mi];
                                        macc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, macc[0][1], 0, 0, 0);
                                        macc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, macc[1][1], 0, 0, 0);
                                    }
                            }
                        }
                        continue;
                    }
                    // ---- multiply-add, weights of the next input channel read while this one multiplies
                    auto read_w = [&](double (&dst)[kOcBlock], int tj) {
                        const double2* p = reinterpret_cast<const double2*>(&s_w[hb][tj][0]);
#pragma unroll
                        for (int o = 0; o < kOcBlock / 2; ++o) {
                            const double2 v = p[o];
                            dst[2 * o] = v.x;
                            dst[2 * o + 1] = v.y;
                        }
                    };
                    auto mul_add = [&](float x, const double (&wr)[kOcBlock]) {
                        const double xd = (double)x;
#pragma unroll
                        for (int o = 0; o < kOcBlock; ++o) acc[o] = fma(xd, wr[o], acc[o]);
                    };
                    // channel of step i: every channel, or every other one starting at this half's
                    const int jmul = split ? 2 : 1, jadd = split ? lh : 0;
                    const int n_steps = split ? CH / 2 : CH;
                    for (int tg = wave; tg < tmax; tg += 4) {
                        if (!((live >> tg) & 1u)) continue;
                        double wa[kOcBlock], wb[kOcBlock];
                        const float* xr = &s_x[row][tg * CH + jadd];
                        read_w(wa, tg * CH + jadd);
                        for (int i = 0; i < n_steps; i += 2) {
                            const float xa = xr[i * jmul];
                            float xb = 0.0f;
                            if (i + 1 < n_steps) {
                                xb = xr[(i + 1) * jmul];
                                read_w(wb, tg * CH + (i + 1) * jmul + jadd);
                            }
                            __builtin_amdgcn_sched_barrier(0);
                            mul_add(xa, wa);
                            __builtin_amdgcn_sched_barrier(0);
                            if (i + 1 < n_steps) {
                                if (i + 2 < n_steps) read_w(wa, tg * CH + (i + 2) * jmul + jadd);
                                __builtin_amdgcn_sched_barrier(0);
                                mul_add(xb, wb);
                                __builtin_amdgcn_sched_barrier(0);
                            }
                        }
                    }
                }
            }
        }
        __syncthreads();  // the last round's weights have been read
        if constexpr (CH >= 4) {
            // ---- the four waves' partial sums (one per tap slice), added in the order of the waves
            double (*s_rm)[R][NB * kOcBlock + 1] = reinterpret_cast<double (*)[R][NB * kOcBlock + 1]>(&s_mem[0]);
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int c = 0; c < NB; ++c)
#pragma unroll
                    for (int v = 0; v < 4; ++v) s_rm[wave][a * 16 + 4 * v + kq][c * kOcBlock + mi] = macc[a][c][v];
            __syncthreads();
            const int per = split ? 2 : 4;  // channels per thread: 16 or 32 channels over 8 thread groups
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (i >= per) break;
                const int c = sl * per + i;  // channel within the chunk
                const int oc = chunk * NB * kOcBlock + c;
                if (oc >= c_out) continue;
                double sum = 0.0;
#pragma unroll
                for (int k = 0; k < 4; ++k) sum += s_rm[k][row][c];
                float v = (row < nrows) ? (float)sum : 0.0f;
                if (bias && v != 0.0f) v += bias[oc];
                resp[((size_t)tile * c_out + oc) * kTileRows + quarter * R + row] = v;
            }
            continue;
        }
        // ---- the eight partial sums of an output, added in a fixed order (wave 0 .. 3, first half then second)
#pragma unroll
        for (int o = 0; o < kOcBlock; ++o) s_red[sl][row][o] = acc[o];
        __syncthreads();
        {
            const int per = split ? 2 : 4;  // channels per thread: 16 or 32 channels over 8 thread groups
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (i >= per) break;
                const int c = sl * per + i;               // channel within the chunk
                const int hbo = c >> 4, o = c & (kOcBlock - 1);
                const int oc = chunk * NB * kOcBlock + c;
                if (oc >= c_out) continue;
                double sum = 0.0;
                if (split) {
#pragma unroll
                    for (int k = 0; k < 8; ++k) sum += s_red[k][row][o];
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k) sum += s_red[2 * k + hbo][row][o];
                }
                float v = (row < nrows) ? (float)sum : 0.0f;
                if (bias && v != 0.0f) v += bias[oc];
                resp[((size_t)tile * c_out + oc) * kTileRows + quarter * R + row] = v;
            }
        }
    }
}

// Workgroups of the streaming kernel.  About six are resident per CU; a grid of 8 per CU ran a third of them in a
// second, badly filled round (128^3 stack 2.05 ms, paper runtime shape r = 256: convolution 155 us), 6 per CU fits
// exactly (2.02 ms, 137 us), and 32 per CU, about one work item per workgroup on these layers, balances best
// (1.99 ms, 123 us; 64 and 128 per CU the same).
constexpr int kStreamBlocks = 256 * 32;

// Layers with at most this many work items run the latency-oriented kernel, larger ones the streaming kernel.
constexpr long long kValuLatencyItems = 1024;
// Layers whose workspace holds more than this many work items run the streaming kernel alone.
constexpr long long kValuStreamOnlyItems = 8 * kValuLatencyItems;
// Layers whose workspace holds at most this many work items (a bound the host knows) run the 32-row form.
constexpr long long kValuSmallItems = 256;

hipError_t launch_conv_valu(const Geom& g, const unsigned long long* occ, const unsigned* occ_prefix,
                            long long nnz_in, const float* feats, int c_in, const double* wp, int c_out,
                            int c_out_pad, const float* bias, const int* tap_active, const unsigned* cand_lin,
                            const int* cand_start, const int* tile_start, const Counters* ctr, long long tiles_cap,
                            int spread, float* resp, hipStream_t s) {
    if (nnz_in <= 0) {  // no input row: every response tile is zero (the gather would have no row to point at)
        hipLaunchKernelGGL(k_conv_valu_empty, dim3(256 * 8), dim3(256), 0, s, c_out, ctr, resp);
        return hipGetLastError();
    }
    // (between one and two times the 32-row form's items only where a site has few neighbours: see above)
    const bool few = g.T <= 9 || nnz_in * 6 <= tiles_cap * kTileRows;
    const bool eight = c_in == 8 && c_out <= 8 && ((uintptr_t)feats & 15) == 0 &&
                       tiles_cap > (few ? 1 : 2) * kValuSmallItems;
    if ((c_in == 1 || eight) && c_out <= 16 && g.T <= 32 && g.K[0] * g.K[1] <= kOneLines) {
        long long blocks = (tiles_cap + 1) / 2;
        if (spread) blocks = round_up(blocks, kXcds);
        if (blocks > kOneBlocks) blocks = kOneBlocks;
#define SCNN_VALU_ONE(CI_, OCB_, SPREAD_)                                                                                     \
    hipLaunchKernelGGL((k_conv_valu_one<CI_, OCB_, SPREAD_>), dim3((unsigned)blocks), dim3(256), 0, s, g, occ, occ_prefix, nnz_in, \
                       feats, wp, c_out, c_out_pad, bias, tap_active, cand_lin, cand_start, tile_start, ctr, resp)
        if (c_in == 1 && c_out <= 8) {
            if (spread) SCNN_VALU_ONE(1, 8, 1); else SCNN_VALU_ONE(1, 8, 0);
        } else if (c_in == 1) {
            if (spread) SCNN_VALU_ONE(1, 16, 1); else SCNN_VALU_ONE(1, 16, 0);
        } else if (!spread && g.T > 9 && tiles_cap <= kEightTiles) {
            const long long most = (long long)device_cu_count() * kEightPerCu;
            blocks = round_up(tiles_cap < most ? tiles_cap : most, kXcds);
            hipLaunchKernelGGL(k_conv_valu_eight, dim3((unsigned)blocks), dim3(kEightThreads), 0, s, g, occ, occ_prefix, nnz_in,
                               feats, wp, c_out, c_out_pad, bias, tap_active, cand_lin, cand_start, tile_start, ctr, resp);
        } else {
            if (spread) SCNN_VALU_ONE(8, 8, 1); else SCNN_VALU_ONE(8, 8, 0);
        }
#undef SCNN_VALU_ONE
        return hipGetLastError();
    }
    // Which kernel runs is decided by the number of work items, which only the device knows.  The host knows an
    // upper bound (tiles_cap): when that is small the latency-oriented kernel is launched alone; otherwise both
    // are launched and the one whose regime it is not returns at once (a few microseconds).
    // Vector loads of CH channels need the row start aligned to them.
    const int align_ch = (int)((((uintptr_t)feats) & 15) == 0 ? 8 : ((((uintptr_t)feats) & 7) == 0 ? 2 : 1));
    int ch = 1;
    if (c_in % 8 == 0 && align_ch >= 8) ch = 8;
    else if (c_in % 4 == 0 && align_ch >= 8) ch = 4;
    else if (c_in % 2 == 0 && align_ch >= 2) ch = 2;
    const int n_chunks = (c_out_pad + 2 * kOcBlock - 1) / (2 * kOcBlock);
    // Far above the latency kernel's regime only the streaming kernel is launched (it takes any number of items; a
    // layer whose workspace is that much larger than its data runs slower on it, a large layer saves a launch).
    const bool stream_only = tiles_cap * n_chunks > kValuStreamOnlyItems;
    const bool both = !stream_only && tiles_cap * n_chunks > kValuLatencyItems;
    // .. or, with items of one block, more, where sites miss at least half of their neighbours (a wave skips the taps that none of
    // its rows has): four channels a gather, or sixteen input channels and more with a cube of taps.  Surfaces and level sets of
    // a tenth and four tenths of the sites, calls, us, against the forms below: 20^3 x 6, 16 -> 16 63 / 67 -> 47 / 61, 4 -> 16
    // 47 / 51 -> 41 / 47; 24^3 x 8, 860 tiles, 24 -> 16 96 / 134 -> 83 / 116; 32^3 x 4 16 -> 8 84 / 116 -> 84 / 109; all
    // occupied 78 -> 81 (24^3 x 4, 16 -> 8) and 122 -> 136 (32^3 x 4); 8 -> 16 55 / 63 / 65 -> 52 / 62 / 72; nine taps, 80 x 80
    // x 12, 16 -> 16, 54 / 61 / 74 -> 57 / 69 / 88.  Four channels a gather gain on every filter (9 to 125 taps 0.98 to 2.0 times
    // as fast).  With eight, 27 and 125 taps gain 0.94 to 1.4 times; of filters longer one way only some groups of 32 taps are
    // full: 5 x 3 x 3 0.82 to 1.18, 5 x 5 0.88 to 1.20, 9 x 9 0.86 to 1.33 (56 x 73 x 16, 24 -> 16 182 -> 200 us), 7 x 7 0.89 to 1.25.
    const bool cube = g.K[0] == g.K[1] && g.K[1] == g.K[2];
    const bool thin = c_out_pad <= kOcBlock && g.T > 9 && (ch == 4 || (ch == 8 && c_in >= 16 && cube)) &&
                      nnz_in * 2 <= tiles_cap * kTileRows && tiles_cap <= 4 * kValuSmallItems;
    if ((tiles_cap * n_chunks <= kValuSmallItems || thin) && ch >= 2) {  // cannot hold more than a thousand tiles
        // One 16-channel block per item where the layer has no more, or where that many workgroups still run at once (two to a
        // compute unit): 40 x 40 x 4, 16 -> 24, 520 items, keeps two blocks
        const long long items = tiles_cap * (c_out_pad / kOcBlock) * (kTileRows / 32);
        const bool one_block = c_out_pad <= kOcBlock || items <= 2 * device_cu_count();
        const int blocks = (int)(one_block ? items : tiles_cap * n_chunks * (kTileRows / 32));
#define SCNN_VALU_SMALL(CH_)                                                                                            \
    do {                                                                                                                \
        if (one_block)                                                                                                  \
            hipLaunchKernelGGL((k_conv_valu_small<CH_, 1>), dim3(blocks), dim3(256), 0, s, g, occ, occ_prefix, nnz_in,  \
                               feats, c_in, wp, c_out, c_out_pad, bias, tap_active, cand_lin, cand_start, tile_start,   \
                               ctr, resp);                                                                              \
        else                                                                                                            \
            hipLaunchKernelGGL((k_conv_valu_small<CH_, 2>), dim3(blocks), dim3(256), 0, s, g, occ, occ_prefix, nnz_in,  \
                               feats, c_in, wp, c_out, c_out_pad, bias, tap_active, cand_lin, cand_start, tile_start,   \
                               ctr, resp);                                                                              \
    } while (0)
        if (ch == 8) SCNN_VALU_SMALL(8);
        else if (ch == 4) SCNN_VALU_SMALL(4);
        else SCNN_VALU_SMALL(2);
#undef SCNN_VALU_SMALL
        return hipGetLastError();
    }
#define SCNN_VALU_CASE(CH_)                                                                                          \
    do {                                                                                                             \
        const long long stream_min = stream_only ? -1 : kValuLatencyItems;                                           \
        if ((both || stream_only) && c_out <= 8)                                                                     \
            hipLaunchKernelGGL((k_conv_valu_stream<CH_, 8>), dim3(kStreamBlocks), dim3(256), 0, s, g, occ,           \
                               occ_prefix, nnz_in, feats, c_in, wp, c_out, c_out_pad, bias, tap_active, cand_lin,    \
                               cand_start, tile_start, ctr, stream_min, resp);                                       \
        else if (both || stream_only)                                                                                \
            hipLaunchKernelGGL((k_conv_valu_stream<CH_, 16>), dim3(kStreamBlocks), dim3(256), 0, s, g, occ,          \
                               occ_prefix, nnz_in, feats, c_in, wp, c_out, c_out_pad, bias, tap_active, cand_lin,    \
                               cand_start, tile_start, ctr, stream_min, resp);                                       \
        if (!stream_only)                                                                                            \
            hipLaunchKernelGGL(k_conv_valu<CH_>, dim3(256 * 8), dim3(256), 0, s, g, occ, occ_prefix, nnz_in, feats,  \
                               c_in, wp, c_out, c_out_pad, bias, tap_active, cand_lin, cand_start, tile_start, ctr,  \
                               kValuLatencyItems, resp);                                                             \
    } while (0)
    if (ch == 8) SCNN_VALU_CASE(8);
    else if (ch == 4) SCNN_VALU_CASE(4);
    else if (ch == 2) SCNN_VALU_CASE(2);
    else SCNN_VALU_CASE(1);
#undef SCNN_VALU_CASE
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Matrix-core path for wide channels (C_in a multiple of 32, C_out a multiple
// of 16 up to 64): the gathered neighbour block of one tap really is a dense
// [pairs x C_in] . [C_in x C_out] contraction.
//
// Only about a third of a surface candidate's taps have a neighbour, and which
// ones varies from site to site, so zero-padding absent neighbours would waste
// most of the matrix cores.  Instead, per tile of 128 candidate sites and per
// tap, the present (output row, input row) pairs are packed into blocks of 16
// (k_pair_build, a light kernel that runs at high occupancy and leaves the
// lists in global memory); k_conv_mfma then runs one fp32 MFMA chain per block
// and per 32 input channels and adds the 16 x 16 results to the tile's
// accumulators in LDS.  Those accumulators are fp64 (native LDS ds_add_f64):
// the fp32 matrix cores only ever sum 32 products of a single tap, the long
// cancelling sum over channels and taps is carried in double and rounded to
// fp32 once.
//
// A wave multiplies its blocks against a whole filter tap (all C_out channels):
// an input row is fetched once per pair and a tap's weights once per round of
// up to three blocks, which keeps the L1 traffic well below what the matrix
// cores could consume.  Waves of a workgroup share the tile's accumulators
// through the LDS atomic, so the order of the fp64 additions is not fixed.
// ---------------------------------------------------------------------------

constexpr unsigned kPadPair = (unsigned)kTileRows << kPairRowShift;  // list padding: dummy accumulator row, input row 0
constexpr int kStageBlocks = 208;                 // 16-pair blocks staged in LDS at a time by the contraction

// Pair lists of all tiles live in one global array of 16-entry blocks; a tile's blocks are contiguous, in
// ascending (tap, output row) order.  tile_hdr[tile] = {first block, block count};
// block_tap[block] = tap | (index of the block within its tap) << 8.
// A tile's space is reserved in closed form, at most ceil(rows / 16) blocks per active tap, so a tile starts at
// (active taps) * (16-row groups of all earlier tiles); unused blocks of a reservation are simply never read.
// One wave builds one tile (lanes = output rows lane and lane + 64) and walks the taps in order, so that it needs
// neither barriers nor a scan; the taps are looked up kPairTapGroup at a time to overlap their loads.
constexpr int kPairTapGroup = 5;
constexpr int kPairTapWords = 8;  // of 32 taps (block_tap holds a tap in one byte)
__global__ __launch_bounds__(256) void k_pair_build(Geom g, const unsigned long long* __restrict__ occ,
                                                    const unsigned* __restrict__ occ_prefix, long long nnz_in,
                                                    const int* __restrict__ tap_active,
                                                    const int* __restrict__ tap_coord,
                                                    const unsigned* __restrict__ cand_lin,
                                                    const int* __restrict__ cand_start,
                                                    const int* __restrict__ tile_start,
                                                    const int* __restrict__ rows16_start, Counters* ctr,
                                                    unsigned* __restrict__ pairs, unsigned short* __restrict__ block_tap,
                                                    uint2* __restrict__ tile_hdr, long long block_cap,
                                                    unsigned short* __restrict__ tap_first) {
    constexpr int G = kPairTapGroup;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned long long lt_mask = (1ull << lane) - 1ull;
    const int n_tiles = (int)ctr->n_tiles;
    __shared__ unsigned s_act[kPairTapWords + 1];  // bit t of the whole: tap t has a non-zero weight
    int active = 0;                                // how many have
    for (int w = 0; w <= kPairTapWords; ++w) {
        const unsigned a = w * 32 < g.T ? active_taps(tap_active, w * 32, g.T - w * 32 < 32 ? g.T - w * 32 : 32) : 0u;
        active += __popc(a);
        if (threadIdx.x == 0) s_act[w] = a;
    }
    __syncthreads();

    const int waves = (int)gridDim.x * 4;
    for (int tile = (int)blockIdx.x * 4 + wave; tile < n_tiles; tile += waves) {
        const int b = sample_of_tile(tile_start, g.batch, tile);
        const int lt = tile - tile_start[b];
        const int first = cand_start[b] + lt * kTileRows;
        int nrows = cand_start[b + 1] - first;
        if (nrows > kTileRows) nrows = kTileRows;
        int sc[2][3];  // sites of rows lane and lane + 64
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            sc[h][0] = sc[h][1] = sc[h][2] = 0;
            if (h * 64 + lane < nrows) site_of(g, cand_lin[first + h * 64 + lane], sc[h][0], sc[h][1], sc[h][2]);
        }
        const long long tile_base = (long long)active * (rows16_start[b] + lt * (kTileRows / 16));
        if (tile_base + (long long)active * ((nrows + 15) >> 4) > block_cap) {
            // cannot happen with the documented workspace size
            if (lane == 0) {
                atomicOr(&ctr->flags, SCNN_FLAG_CAND_OVERFLOW);
                tile_hdr[tile] = make_uint2(0u, 0u);
            }
            if (tap_first)
                for (int t = lane; t <= g.T; t += 64) tap_first[(size_t)tile * (g.T + 1) + t] = 0;
            continue;
        }
        unsigned blk = (unsigned)tile_base;  // next free block
        // Taps are walked in order as segments of up to G taps of one filter line (t0, t1): the neighbours of a
        // segment are adjacent sites, resolved from one pair of bitmap words per row.  Two segments per step keep
        // sixteen loads in flight per lane.
        const int n_sub = (g.K[2] + G - 1) / G;
        const int n_seg = g.K[0] * g.K[1] * n_sub;
        for (int sg0 = 0; sg0 < n_seg; sg0 += 2) {
            unsigned nbr[2][G][2];
            int seg_tap[2], seg_cnt[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int sg = sg0 + u < n_seg ? sg0 + u : n_seg - 1;
                const int line = sg / n_sub, t2_lo = (sg - line * n_sub) * G;
                const int t0l = line / g.K[1], t1l = line - t0l * g.K[1];
                int cnt = g.K[2] - t2_lo;
                if (cnt > G) cnt = G;
                if (sg0 + u >= n_seg) cnt = 0;
                seg_tap[u] = line * g.K[2] + t2_lo;
                seg_cnt[u] = cnt;
                const unsigned long long act2 =
                    (unsigned long long)s_act[(seg_tap[u] >> 5) + 1] << 32 | s_act[seg_tap[u] >> 5];
                const unsigned act = (unsigned)(act2 >> (seg_tap[u] & 31));
#pragma unroll
                for (int h = 0; h < 2; ++h) {
#pragma unroll
                    for (int k = 0; k < G; ++k) nbr[u][k][h] = 0xffffffffu;
                    lookup_line(g, occ, occ_prefix, nnz_in, cnt > 0 && h * 64 + lane < nrows, b, sc[h][0], sc[h][1],
                                sc[h][2], t0l, t1l, t2_lo, cnt, act,
                                [&](int k, int n) { nbr[u][k][h] = (unsigned)n; });
                }
            }
            // ---- pack: each tap's present pairs in ascending output row, padded to whole blocks of 16 with
            //      entries that point at the dummy accumulator row
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int m = 0; m < G; ++m) {
                    if (m >= seg_cnt[u]) continue;
                    const int t = seg_tap[u] + m;
                    const unsigned long long m0 = __ballot(nbr[u][m][0] != 0xffffffffu),
                                             m1 = __ballot(nbr[u][m][1] != 0xffffffffu);
                    const int c0 = __popcll(m0), cnt = c0 + __popcll(m1);
                    const int nblk = (cnt + 15) >> 4;
                    unsigned* pl = pairs + (size_t)blk * 16;
                    if (nbr[u][m][0] != 0xffffffffu)
                        pl[__popcll(m0 & lt_mask)] = ((unsigned)lane << kPairRowShift) | nbr[u][m][0];
                    if (nbr[u][m][1] != 0xffffffffu)
                        pl[c0 + __popcll(m1 & lt_mask)] = ((unsigned)(64 + lane) << kPairRowShift) | nbr[u][m][1];
                    if (lane < 16 && cnt + lane < nblk * 16) pl[cnt + lane] = kPadPair;
                    if (lane < nblk) block_tap[blk + lane] = (unsigned short)(t | (lane << 8));
                    // optional: where each tap's blocks start within the tile (entry T = the tile's block count)
                    if (tap_first && lane == 0) tap_first[(size_t)tile * (g.T + 1) + t] = (unsigned short)(blk - (unsigned)tile_base);
                    blk += (unsigned)nblk;
                }
        }
        if (lane == 0) {
            tile_hdr[tile] = make_uint2((unsigned)tile_base, blk - (unsigned)tile_base);
            if (tap_first) tap_first[(size_t)tile * (g.T + 1) + g.T] = (unsigned short)(blk - (unsigned)tile_base);
        }
    }
}

hipError_t launch_pair_build(const Geom& g, const unsigned long long* occ, const unsigned* occ_prefix,
                             long long nnz_in, const int* tap_active, const int* tap_coord,
                             const unsigned* cand_lin, const int* cand_start, const int* tile_start,
                             const int* rows16_start, Counters* ctr, unsigned* pairs, unsigned short* block_tap,
                             uint2* tile_hdr, long long block_cap, long long tiles_cap, unsigned short* tap_first,
                             hipStream_t s) {
    long long blocks = (tiles_cap + 3) / 4;  // one wave per tile
    if (blocks < 1) blocks = 1;
    if (blocks > 256 * 8) blocks = 256 * 8;
    hipLaunchKernelGGL(k_pair_build, dim3((unsigned)blocks), dim3(256), 0, s, g, occ, occ_prefix, nnz_in, tap_active,
                       tap_coord, cand_lin, cand_start, tile_start, rows16_start, ctr, pairs, block_tap, tile_hdr,
                       block_cap, tap_first);
    return hipGetLastError();
}

constexpr int kConvWaves = 4;  // waves per workgroup of the contraction kernel

__host__ __device__ inline size_t conv_mfma_lds_bytes(int c_out) {
    return (size_t)(kTileRows + 1) * (c_out + 1) * sizeof(double)   // accumulators + one dummy row
           + (size_t)kStageBlocks * 16 * sizeof(unsigned)            // staged pair blocks
           + (size_t)kStageBlocks * sizeof(unsigned short)           // tap / position of each staged block
           + (size_t)kStageBlocks * sizeof(unsigned)                 // round list
           + (kConvWaves + 1 + 2) * sizeof(int);
}

// Operands of one round = up to RB consecutive 16-pair blocks of ONE tap, fetched one round ahead of their use.
template <int KC, int NB, int RB>
struct RoundRegs {
    f32x4 a[RB][KC][2];     // A operand: lane holds x[in(pair 16j + jj)][kc*32 + 8*gq .. + 8)
    f32x4 b[KC][NB][2];     // B operand: lane holds w[tap][kc*32 + 8*gq + s][16*cb + jj], s = 0..7
    unsigned oaddr[RB][4];  // LDS byte address of accumulator (row of result row 4*gq + v, channel jj)
};

// Work split: each wave of the workgroup takes a contiguous share of the rounds.  A wave multiplies its blocks against the whole
// filter tap (all C_out channels), so an input row is fetched once per pair and a tap's weights once per round;
// the price is that two waves may add to the same accumulator, which the LDS fp64 atomic makes safe but not
// ordered: the fp64 sum can differ in its last bits from run to run.
// HALF: C_in = 16 (KC = 1): a lane's K slot gq stands for the four channels 4 gq .. 4 gq + 3 instead of eight, so a
// block takes four matrix instructions per 16 output channels and the second halves of the operands stay unused
// (the filter is prepared in the same 8-floats-per-lane layout, upper four zero).
// only_odd: launched behind k_conv_mfma_split for the calls that it leaves (ctr->odd); leaves the others at once.
template <int KC /* C_in / 32 */, int NB /* C_out / 16 */, int HALF = 0>
__global__ __launch_bounds__(kConvWaves * 64) void k_conv_mfma(int taps, long long nnz_in, int only_odd,
                                                               const float* __restrict__ feats,
                                                               const float* __restrict__ wb,
                                                               const float* __restrict__ bias,
                                                               const unsigned* __restrict__ pairs,
                                                               const unsigned short* __restrict__ block_tap,
                                                               const uint2* __restrict__ tile_hdr,
                                                               Counters* __restrict__ ctr,
                                                               float* __restrict__ resp) {
    static_assert(!HALF || KC == 1, "the half chunk stands alone");
    if (only_odd && ctr->odd == 0) return;
    constexpr int C_IN = HALF ? 16 : KC * 32, C_OUT = NB * 16, CS = C_OUT + 1 /* padded accumulator row */;
    constexpr int RB = (KC * NB <= 4) ? 3 : ((KC * NB <= 8) ? 2 : 1);  // blocks per round
    constexpr int NT = kConvWaves * 64;
    static_assert(kStageBlocks % 4 == 0 && kStageBlocks <= 256, "stage size");
    extern __shared__ __align__(16) unsigned char smem[];
    double* s_c = (double*)smem;                                               // [129][CS]; row 128 absorbs padding
    unsigned* s_flat = (unsigned*)(s_c + (kTileRows + 1) * CS);                // [kStageBlocks][16] packed pairs
    unsigned short* s_btap = (unsigned short*)(s_flat + kStageBlocks * 16);    // [kStageBlocks]
    unsigned* s_rmeta = (unsigned*)(s_btap + kStageBlocks);  // [kStageBlocks] first block | blocks << 8 | tap << 16
    int* s_wlo = (int*)(s_rmeta + kStageBlocks);  // [kConvWaves + 1] first round of each wave; the last = all rounds
    int* s_next = s_wlo + kConvWaves + 1;         // [2] the workgroup's next tile (alternating slots)

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int jj = lane & 15, gq = lane >> 4;
    const unsigned long long lt_mask = (1ull << lane) - 1ull;
    const int n_tiles = (int)ctr->n_tiles;
    // LDS byte address of this lane's channel in accumulator row 0 (a generic pointer to LDS carries the LDS
    // address in its low 32 bits); accumulator addresses are formed once per block, at load time
    const unsigned lane_off = (unsigned)(size_t)s_c + (unsigned)jj * (unsigned)sizeof(double);

    // XCD-aware tile order: workgroup i runs on XCD i % kXcds; give each XCD one contiguous span of tiles so that
    // the input rows shared by neighbouring tiles stay in that XCD's L2.  Within its span a workgroup starts with
    // the tile of its slot and then draws tiles, in ascending order, from the span's counter (then from the other
    // spans' counters): tiles differ in work, and a fixed assignment would leave workgroups idle at the end.
    const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds, per_xcd = gridDim.x / kXcds;
    const int span = (n_tiles + kXcds - 1) / kXcds;
    const int tile_end = (xcd + 1) * span < n_tiles ? (xcd + 1) * span : n_tiles;

    for (int i = threadIdx.x; i < kTileRows * CS; i += NT) s_c[i] = 0.0;  // the dummy row needs no reset
    // The stage buffer only ever holds entries written by the pair builder (or these zeros), so whatever a clamped
    // read past the end of a tile's list finds there names a valid input row.
    for (int i = threadIdx.x; i < kStageBlocks * 16; i += NT) s_flat[i] = 0u;

    int parity = 0;
    for (int tile = xcd * span + slot < tile_end ? xcd * span + slot : -1; tile >= 0; parity ^= 1) {
        const uint2 hdr = tile_hdr[tile];
        for (unsigned s0 = 0; s0 < hdr.y; s0 += kStageBlocks) {
            const int n_blocks = (int)((hdr.y - s0) < (unsigned)kStageBlocks ? (hdr.y - s0) : (unsigned)kStageBlocks);
            __syncthreads();  // previous stage consumed (and, for the first stage, the accumulators are zero)
            {   // ---- stage this tile's next blocks: a contiguous copy, 16 bytes per thread and step
                const uint4* src = (const uint4*)(pairs + (size_t)(hdr.x + s0) * 16);
                uint4* dst = (uint4*)s_flat;
                for (int i = threadIdx.x; i < n_blocks * 4; i += NT) dst[i] = src[i];
                for (int i = threadIdx.x; i < n_blocks; i += NT) s_btap[i] = block_tap[hdr.x + s0 + i];
            }
            __syncthreads();
            // ---- round list: a round = up to RB consecutive blocks of one tap.  It starts at every RB-th block of
            //      a tap's run (and at the start of the stage); entry = first block | blocks << 8 | tap << 16.
            //      Wave w takes the rounds that start in the w-th quarter of the stage's blocks: contiguous, and
            //      within one round of an even share of the blocks.
            if (wave == 0) {
                int base = 0;
                int lo[kConvWaves];
#pragma unroll
                for (int w = 0; w < kConvWaves; ++w) lo[w] = 0;
                for (int i0 = 0; i0 < n_blocks; i0 += 64) {
                    const int i = i0 + lane;
                    unsigned bt[RB];
#pragma unroll
                    for (int d = 0; d < RB; ++d) bt[d] = s_btap[(i + d) < n_blocks ? (i + d) : n_blocks - 1];
                    const bool start = i < n_blocks && (i == 0 || ((bt[0] >> 8) % RB) == 0);
                    int nb = 1;
#pragma unroll
                    for (int d = 1; d < RB; ++d)
                        if (nb == d && i + d < n_blocks && ((bt[d] >> 8) % RB) != 0) nb = d + 1;
                    const unsigned long long m = __ballot(start);
                    if (start)
                        s_rmeta[base + __popcll(m & lt_mask)] = (unsigned)i | (unsigned)nb << 8 | (bt[0] & 0xffu) << 16;
                    base += __popcll(m);
#pragma unroll
                    for (int w = 1; w < kConvWaves; ++w)  // rounds that start before the w-th share of the blocks
                        lo[w] += __popcll(__ballot(start && i * kConvWaves < w * n_blocks));
                }
                if (lane == 0) {
#pragma unroll
                    for (int w = 0; w < kConvWaves; ++w) s_wlo[w] = lo[w];
                    s_wlo[kConvWaves] = base;
                }
            }
            __syncthreads();
            const int r_lo = __builtin_amdgcn_readfirstlane(s_wlo[wave]);
            const int my_rounds = __builtin_amdgcn_readfirstlane(s_wlo[wave + 1]) - r_lo;
            if (my_rounds > 0) {
                // The wave's pipeline, per round: list entry (LDS) -> pair entries of its blocks (LDS) -> operands
                // (global) -> compute.  Each step is issued a full round before its result is needed, so that no
                // LDS or memory round trip sits between two rounds' matrix instructions.  All reads of a round are
                // unconditional, so that their number is fixed: a round past the end repeats the wave's last one
                // (never computed), a block past a round's end repeats list entries and is never computed.
                struct Entries {
                    unsigned in[RB];  // pair jj of each block (its input row)
                    uint4 out[RB];    // pairs 4*gq .. 4*gq + 3 of each block (their result rows)
                };
                auto meta_at = [&](int j) { return s_rmeta[r_lo + (j < my_rounds ? j : my_rounds - 1)]; };
                auto read_entries = [&](unsigned meta, Entries& E) {
                    const int first = (int)(meta & 0xffu);
#pragma unroll
                    for (int k = 0; k < RB; ++k) {
                        const int blk = (first + k) < kStageBlocks ? (first + k) : kStageBlocks - 1;
                        E.in[k] = s_flat[16 * blk + jj];
                        E.out[k] = *(const uint4*)(s_flat + 16 * blk + 4 * gq);
                    }
                };
                auto load_round = [&](unsigned meta, const Entries& E, RoundRegs<KC, NB, RB>& R) {
                    int tt = (int)((meta >> 16) & 0xffu);
                    tt = tt < taps ? tt : taps - 1;
                    const f32x4* wt = (const f32x4*)(wb + ((size_t)tt * KC * NB * 64 + lane) * 8);
#pragma unroll
                    for (int kc = 0; kc < KC; ++kc)
#pragma unroll
                        for (int cb = 0; cb < NB; ++cb) {
                            R.b[kc][cb][0] = wt[(kc * NB + cb) * 128];
                            if constexpr (!HALF) R.b[kc][cb][1] = wt[(kc * NB + cb) * 128 + 1];
                        }
#pragma unroll
                    for (int k = 0; k < RB; ++k) {
                        const unsigned in = E.in[k] & kPairInMask;
                        const f32x4* src = (const f32x4*)(feats + (size_t)in * C_IN + (HALF ? 4 : 8) * gq);
#pragma unroll
                        for (int kc = 0; kc < KC; ++kc) {
                            R.a[k][kc][0] = src[kc * 8];
                            if constexpr (!HALF) R.a[k][kc][1] = src[kc * 8 + 1];
                        }
                        // (a stale entry past the end of the list may name any row, but such a block is not computed)
                        R.oaddr[k][0] = (E.out[k].x >> kPairRowShift) * (unsigned)(CS * sizeof(double)) + lane_off;
                        R.oaddr[k][1] = (E.out[k].y >> kPairRowShift) * (unsigned)(CS * sizeof(double)) + lane_off;
                        R.oaddr[k][2] = (E.out[k].z >> kPairRowShift) * (unsigned)(CS * sizeof(double)) + lane_off;
                        R.oaddr[k][3] = (E.out[k].w >> kPairRowShift) * (unsigned)(CS * sizeof(double)) + lane_off;
                    }
                };
                // A block = NB independent fp32 MFMA chains per 32 input channels (one per 16 output channels); the
                // 16 x 16 results (rows = pairs 4*gq + v, column = channel 16*cb + jj) are added to the fp64
                // accumulators.  Padding pairs land in the dummy row.  Blocks are guarded one by one (uniform
                // branches) rather than through per-count variants, which the compiler would merge again through
                // scratch memory.
                auto compute_round = [&](unsigned meta, const RoundRegs<KC, NB, RB>& R) {
                    const int nb = (int)((meta >> 8) & 0xffu);  // 1 .. RB
#pragma unroll
                    for (int k = 0; k < RB; ++k) {
                        if (k == 0 || k < nb) {  // (a round has at least one block)
#pragma unroll
                            for (int kc = 0; kc < KC; ++kc) {
                                f32x4 acc[NB];
#pragma unroll
                                for (int cb = 0; cb < NB; ++cb) {
                                    f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                                    for (int s = 0; s < 4; ++s)
                                        c = __builtin_amdgcn_mfma_f32_16x16x4f32(R.a[k][kc][0][s], R.b[kc][cb][0][s], c, 0, 0, 0);
                                    if constexpr (!HALF) {
#pragma unroll
                                        for (int s = 0; s < 4; ++s)
                                            c = __builtin_amdgcn_mfma_f32_16x16x4f32(R.a[k][kc][1][s], R.b[kc][cb][1][s], c, 0, 0, 0);
                                    }
                                    acc[cb] = c;
                                }
#pragma unroll
                                for (int cb = 0; cb < NB; ++cb)
#pragma unroll
                                    for (int v = 0; v < 4; ++v)
                                        __hip_atomic_fetch_add(
                                            (__attribute__((address_space(3))) double*)(size_t)R.oaddr[k][v] + cb * 16,
                                            (double)acc[cb][v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                            }
                        }
                    }
                };
                RoundRegs<KC, NB, RB> r0, r1;
                Entries ent;
                unsigned m0 = __builtin_amdgcn_readfirstlane(meta_at(0));
                unsigned m1 = __builtin_amdgcn_readfirstlane(meta_at(1));
                unsigned m_ahead = meta_at(2);
                read_entries(m0, ent);
                load_round(m0, ent, r0);
                read_entries(m1, ent);
                // Let these first reads land before the loop: inside it, every value read from LDS is used only
                // after a round's worth of accumulator updates has been issued behind the read, so the wait for
                // it (the LDS queue is in order) does not wait for those updates.
                asm volatile("" : "+v"(m_ahead));
#pragma unroll
                for (int k = 0; k < RB; ++k)
                    asm volatile("" : "+v"(ent.in[k]), "+v"(ent.out[k].x), "+v"(ent.out[k].y), "+v"(ent.out[k].z),
                                 "+v"(ent.out[k].w));
                for (int j = 0; j < my_rounds; j += 2) {
                    // here: r0 = operands of round j (list entry m0), ent = pair entries of round j + 1 (m1),
                    //       m_ahead = list entry of round j + 2
                    load_round(m1, ent, r1);
                    const unsigned m2 = __builtin_amdgcn_readfirstlane(m_ahead);
                    read_entries(m2, ent);
                    m_ahead = meta_at(j + 3);
                    compute_round(m0, r0);
                    if (j + 1 >= my_rounds) break;
                    load_round(m2, ent, r0);
                    const unsigned m3 = __builtin_amdgcn_readfirstlane(m_ahead);
                    read_entries(m3, ent);
                    m_ahead = meta_at(j + 4);
                    compute_round(m1, r1);
                    m0 = m2;
                    m1 = m3;
                }
            }
        }
        // Draw the next tile: from the own span, and once that is used up from the other spans, so that no XCD ends
        // before the others.  The last wave does it when its share of the tile is done: it has the smallest share
        // on average and would otherwise only wait at the barrier, which hides the atomic's round trip.
        if (threadIdx.x == NT - 64) {
            int t = -1;
            for (int d = 0; d < kXcds && t < 0; ++d) {
                const int x = (xcd + d) % kXcds;
                const int end_x = (x + 1) * span < n_tiles ? (x + 1) * span : n_tiles;
                if (x * span + per_xcd >= end_x) continue;  // (a span with no tiles to draw)
                const int cand = x * span + per_xcd + (int)atomicAdd(&ctr->conv_ticket[x * kTicketStride], 1u);
                if (cand < end_x) t = cand;
            }
            s_next[parity] = t;
        }
        __syncthreads();
        const int next_tile = s_next[parity];
        // ---- epilogue: one rounding to fp32, bias on the non-zero entries, planar store; the accumulators are
        //      reset on the way.  A lane takes one row, a wave one channel at a time: consecutive rows lie
        //      CS doubles apart, i.e. 2 banks (mod 64), so the 64 reads of a wave spread over all LDS banks, and
        //      the wave's stores form one contiguous 256-byte run of the planar tile.
        {
            constexpr int OCW = (C_OUT + kConvWaves - 1) / kConvWaves, H = kTileRows / 64;
            double acc[OCW][H];
#pragma unroll
            for (int j = 0; j < OCW; ++j) {  // all reads first: one LDS latency for the lot
                const int oc = (wave + j * kConvWaves) < C_OUT ? (wave + j * kConvWaves) : C_OUT - 1;
#pragma unroll
                for (int h = 0; h < H; ++h) acc[j][h] = s_c[(h * 64 + lane) * CS + oc];
            }
#pragma unroll
            for (int j = 0; j < OCW; ++j) {
                const int oc = wave + j * kConvWaves;
                if (C_OUT % kConvWaves == 0 || oc < C_OUT) {
                    // (the weights stand in as a readable address when there is no bias)
                    const float bl = (bias ? bias : wb)[oc];
                    const float bv = bias ? bl : 0.0f;
#pragma unroll
                    for (int h = 0; h < H; ++h) {
                        const int r = h * 64 + lane;
                        s_c[r * CS + oc] = 0.0;
                        float x = (float)acc[j][h];
                        if (x != 0.0f) x += bv;
                        resp[((size_t)tile * C_OUT + oc) * kTileRows + r] = x;
                    }
                }
            }
        }
        tile = next_tile;
    }
}

template <int KC, int NB, int HALF = 0>
static hipError_t launch_conv_mfma_t(int taps, long long nnz_in, int only_odd, const float* feats, const float* wb, const float* bias,
                                     const unsigned* pairs, const unsigned short* block_tap, const uint2* tile_hdr,
                                     Counters* ctr, float* resp, hipStream_t s) {
    const size_t lds = conv_mfma_lds_bytes(NB * 16);
    // (set on every launch: the attribute belongs to the current device's copy of the kernel, and a flag remembering
    // that it was set would have to be kept per device and guarded between threads for the sake of a microsecond)
    hipError_t e = hipFuncSetAttribute((const void*)k_conv_mfma<KC, NB, HALF>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    int per_cu = (int)((160 * 1024) / lds);
    if (per_cu < 1) per_cu = 1;
    if (per_cu > 4) per_cu = 4;    // 16 waves per CU
    const int grid = (device_cu_count() * per_cu + kXcds - 1) / kXcds * kXcds;  // one span of tiles per XCD
    hipLaunchKernelGGL((k_conv_mfma<KC, NB, HALF>), dim3(grid), dim3(kConvWaves * 64), lds, s, taps, nnz_in, only_odd, feats, wb,
                       bias, pairs, block_tap, tile_hdr, ctr, resp);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The same contraction on the bf16 matrix cores, both operands as three bf16 numbers each (split3; the rows split after
// the load, the filter beforehand): the forward pass's pair-list kernel.  A block's 32 channels take 384 clocks of
// matrix time per 64 output channels instead of 1024, the sums of two chunks are added in fp64 registers before they go
// to the accumulators (half the LDS atomics), and the weights of one chunk at a time are held in registers.  256^3, 64->64
// channels, 125 taps, 1.3 M candidates: call 3.96 -> 2.50 ms, now bound by the weights and rows that vector memory
// returns (a round's chunk asks for 12 + 4 KB for at most two blocks); error against 64 bits 1.08e-7 -> 4.6e-8 of the
// result's norm, on rows with a sixth of their entries 5.4e-8 -> 3.8e-8.
// The adjoint convolution of the backward pass takes it too: 128^3 x 4, 32 -> 64 channels, 202 k rows: 327 -> 280 us, 23 of
// which the look over the gradient rows' values takes back (call 652 -> 604 us); bound by the gathers, 5 TB/s of rows.
// Sixteen input channels keep the fp32 kernel above, and the adjoint that of 32 -> 32 and 32 -> 16 (see carve_bwd).
// Operands of one 32-channel chunk of a round (up to RB consecutive 16-pair blocks of ONE tap), fetched one chunk ahead
// of their use.
template <int NB, int RB>
struct ChunkRegs {
    u32x4 a[RB][2];   // input rows in fp32: lane holds x[in(pair 16j + jj)][32 kc + 8 gq .. + 8), its 16-byte halves in
                      // the order (jj odd: upper first)
    u32x4 b[3][NB];   // filter in bf16 thirds (split3): lane holds w[tap][32 kc + 8 gq + i][16 cb + jj], i = 0..7
};

// Values that the parts do not hold (ctr->odd): the forward call's instances multiply them by the loop for them below; those
// of the adjoint convolution (LEAVE_ODD), where one tiny gradient is enough and is nothing unusual, leave the whole call to
// k_conv_mfma, launched behind them, which leaves the others.
template <int KC /* C_in / 32 */, int NB /* C_out / 16 */, int LEAVE_ODD>
__global__ __launch_bounds__(kConvWaves * 64, NB == 4 ? 2 : 1) void k_conv_mfma_split(int taps, long long nnz_in,
                                                               const float* __restrict__ feats,
                                                               const u32x4* __restrict__ ws,
                                                               const float* __restrict__ w,
                                                               const float* __restrict__ bias,
                                                               const unsigned* __restrict__ pairs,
                                                               const unsigned short* __restrict__ block_tap,
                                                               const uint2* __restrict__ tile_hdr,
                                                               Counters* __restrict__ ctr,
                                                               float* __restrict__ resp) {
    constexpr int C_IN = KC * 32, C_OUT = NB * 16, CS = C_OUT + 1 /* padded accumulator row */;
    constexpr int RB = NB <= 2 ? 3 : 2;  // blocks per round
    constexpr int NBP = NB > 2 ? 4 : 2;  // blocks of output channels in the filter's layout
    constexpr int NT = kConvWaves * 64;
    static_assert(kStageBlocks % 4 == 0 && kStageBlocks <= 256, "stage size");
    extern __shared__ __align__(16) unsigned char smem[];
    double* s_c = (double*)smem;                                               // [129][CS]; row 128 absorbs padding
    unsigned* s_flat = (unsigned*)(s_c + (kTileRows + 1) * CS);                // [kStageBlocks][16] packed pairs
    unsigned short* s_btap = (unsigned short*)(s_flat + kStageBlocks * 16);    // [kStageBlocks]
    unsigned* s_rmeta = (unsigned*)(s_btap + kStageBlocks);  // [kStageBlocks] first block | blocks << 8 | tap << 16
    int* s_wlo = (int*)(s_rmeta + kStageBlocks);  // [kConvWaves + 1] first round of each wave; the last = all rounds
    int* s_next = s_wlo + kConvWaves + 1;         // [2] the workgroup's next tile (alternating slots)

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int jj = lane & 15, gq = lane >> 4;
    const unsigned long long lt_mask = (1ull << lane) - 1ull;
    const int n_tiles = (int)ctr->n_tiles;
    bool odd = __builtin_amdgcn_readfirstlane(ctr->odd) != 0;
    if constexpr (LEAVE_ODD) {
        if (odd) return;
        odd = false;
    }
    // LDS byte address of this lane's channel in accumulator row 0 (a generic pointer to LDS carries the LDS
    // address in its low 32 bits); accumulator addresses are formed once per block, at load time
    const unsigned lane_off = (unsigned)(size_t)s_c + (unsigned)jj * (unsigned)sizeof(double);

    // XCD-aware tile order: workgroup i runs on XCD i % kXcds; give each XCD one contiguous span of tiles so that
    // the input rows shared by neighbouring tiles stay in that XCD's L2.  Within its span a workgroup starts with
    // the tile of its slot and then draws tiles, in ascending order, from the span's counter (then from the other
    // spans' counters): tiles differ in work, and a fixed assignment would leave workgroups idle at the end.
    const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds, per_xcd = gridDim.x / kXcds;
    const int span = (n_tiles + kXcds - 1) / kXcds;
    const int tile_end = (xcd + 1) * span < n_tiles ? (xcd + 1) * span : n_tiles;

    for (int i = threadIdx.x; i < kTileRows * CS; i += NT) s_c[i] = 0.0;  // the dummy row needs no reset
    // The stage buffer only ever holds entries written by the pair builder (or these zeros), so whatever a clamped
    // read past the end of a tile's list finds there names a valid input row.
    for (int i = threadIdx.x; i < kStageBlocks * 16; i += NT) s_flat[i] = 0u;

    int parity = 0;
    for (int tile = xcd * span + slot < tile_end ? xcd * span + slot : -1; tile >= 0; parity ^= 1) {
        const uint2 hdr = tile_hdr[tile];
        for (unsigned s0 = 0; s0 < hdr.y; s0 += kStageBlocks) {
            const int n_blocks = (int)((hdr.y - s0) < (unsigned)kStageBlocks ? (hdr.y - s0) : (unsigned)kStageBlocks);
            __syncthreads();  // previous stage consumed (and, for the first stage, the accumulators are zero)
            {   // ---- stage this tile's next blocks: a contiguous copy, 16 bytes per thread and step
                const uint4* src = (const uint4*)(pairs + (size_t)(hdr.x + s0) * 16);
                uint4* dst = (uint4*)s_flat;
                for (int i = threadIdx.x; i < n_blocks * 4; i += NT) dst[i] = src[i];
                for (int i = threadIdx.x; i < n_blocks; i += NT) s_btap[i] = block_tap[hdr.x + s0 + i];
            }
            __syncthreads();
            // ---- round list: a round = up to RB consecutive blocks of one tap.  It starts at every RB-th block of
            //      a tap's run (and at the start of the stage); entry = first block | blocks << 8 | tap << 16.
            //      Wave w takes the rounds that start in the w-th quarter of the stage's blocks: contiguous, and
            //      within one round of an even share of the blocks.
            if (wave == 0) {
                int base = 0;
                int lo[kConvWaves];
#pragma unroll
                for (int w = 0; w < kConvWaves; ++w) lo[w] = 0;
                for (int i0 = 0; i0 < n_blocks; i0 += 64) {
                    const int i = i0 + lane;
                    unsigned bt[RB];
#pragma unroll
                    for (int d = 0; d < RB; ++d) bt[d] = s_btap[(i + d) < n_blocks ? (i + d) : n_blocks - 1];
                    const bool start = i < n_blocks && (i == 0 || ((bt[0] >> 8) % RB) == 0);
                    int nb = 1;
#pragma unroll
                    for (int d = 1; d < RB; ++d)
                        if (nb == d && i + d < n_blocks && ((bt[d] >> 8) % RB) != 0) nb = d + 1;
                    const unsigned long long m = __ballot(start);
                    if (start)
                        s_rmeta[base + __popcll(m & lt_mask)] = (unsigned)i | (unsigned)nb << 8 | (bt[0] & 0xffu) << 16;
                    base += __popcll(m);
#pragma unroll
                    for (int w = 1; w < kConvWaves; ++w)  // rounds that start before the w-th share of the blocks
                        lo[w] += __popcll(__ballot(start && i * kConvWaves < w * n_blocks));
                }
                if (lane == 0) {
#pragma unroll
                    for (int w = 0; w < kConvWaves; ++w) s_wlo[w] = lo[w];
                    s_wlo[kConvWaves] = base;
                }
            }
            __syncthreads();
            const int r_lo = __builtin_amdgcn_readfirstlane(s_wlo[wave]);
            const int my_rounds = __builtin_amdgcn_readfirstlane(s_wlo[wave + 1]) - r_lo;
            if (odd && my_rounds > 0) {
                // values that the parts do not hold: fp32 instructions on rows and weights as they are (not pipelined)
#pragma unroll 1
                for (int j = 0; j < my_rounds; ++j) {
                    const unsigned meta = __builtin_amdgcn_readfirstlane(s_rmeta[r_lo + j]);
                    const int first = (int)(meta & 0xffu), nb = (int)((meta >> 8) & 0xffu), t = (int)((meta >> 16) & 0xffu);
#pragma unroll 1
                    for (int k = 0; k < nb; ++k) {
                        unsigned in = s_flat[16 * (first + k) + jj] & kPairInMask;
                        asm volatile("" : "+v"(in));  // (as in rows_of)
                        const uint4 out = *(const uint4*)(s_flat + 16 * (first + k) + 4 * gq);
                        const unsigned o[4] = {out.x, out.y, out.z, out.w};
#pragma unroll 1
                        for (int kc = 0; kc < KC; ++kc) {
                            const int ch = kc * 32 + gq * 8;
                            const float* row = feats + (size_t)in * C_IN + ch;
                            f32x4 d[NB];
#pragma unroll
                            for (int cb = 0; cb < NB; ++cb) d[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                            for (int i = 0; i < 8; ++i) {
                                const float x = row[i];
#pragma unroll
                                for (int cb = 0; cb < NB; ++cb) {
                                    const float wv = w[((size_t)t * C_IN + ch + i) * C_OUT + cb * 16 + jj];
                                    d[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, wv, d[cb], 0, 0, 0);
                                }
                            }
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                const unsigned at = (o[v] >> kPairRowShift) * (unsigned)(CS * sizeof(double)) + lane_off;
#pragma unroll
                                for (int cb = 0; cb < NB; ++cb)
                                    __hip_atomic_fetch_add((__attribute__((address_space(3))) double*)(size_t)at + cb * 16,
                                                           (double)d[cb][v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                            }
                        }
                    }
                }
            } else if (my_rounds > 0) {
                // The wave's pipeline, per round: list entry (LDS) -> pair entries of its blocks (LDS) -> operands
                // (global, one 32-channel chunk at a time) -> compute.  Each step is issued a round (operands: a
                // chunk) before its result is needed, so that no LDS or memory round trip sits between two chunks'
                // matrix instructions.  All reads are unconditional: a round past the end repeats the wave's last
                // one (never computed), a block past a round's end repeats list entries and is never computed.
                struct Entries {
                    unsigned in[RB];  // pair jj of each block (its input row)
                    uint4 out[RB];    // pairs 4*gq .. 4*gq + 3 of each block (their result rows)
                };
                auto meta_at = [&](int j) { return s_rmeta[r_lo + (j < my_rounds ? j : my_rounds - 1)]; };
                auto read_entries = [&](unsigned meta, Entries& E) {
                    const int first = (int)(meta & 0xffu);
#pragma unroll
                    for (int k = 0; k < RB; ++k) {
                        const int blk = (first + k) < kStageBlocks ? (first + k) : kStageBlocks - 1;
                        E.in[k] = s_flat[16 * blk + jj];
                        E.out[k] = *(const uint4*)(s_flat + 16 * blk + 4 * gq);
                    }
                };
                // Rows are a multiple of 64 bytes apart, mostly of 256: sixteen lanes that read the same 16 bytes of
                // sixteen such rows take 58 clocks a load; with every other row's halves swapped, 35.
                const unsigned half0 = (unsigned)(jj & 1) * 16u;
                auto load_chunk = [&](unsigned meta, const unsigned (&in)[RB], int kc, ChunkRegs<NB, RB>& R) {
                    int tt = (int)((meta >> 16) & 0xffu);
                    tt = tt < taps ? tt : taps - 1;
                    const u32x4* wt = ws + (size_t)(tt * KC + kc) * (3 * NBP * 64);
#pragma unroll
                    for (int q = 0; q < 3; ++q)
#pragma unroll
                        for (int cb = 0; cb < NB; ++cb) R.b[q][cb] = (wt + (q * NBP + cb) * 64)[lane];
#pragma unroll
                    for (int k = 0; k < RB; ++k) {
                        const char* src = (const char*)feats + (size_t)in[k] * (C_IN * 4) + (kc * 4 + gq) * 32;
                        R.a[k][0] = *(const u32x4*)(src + half0);
                        R.a[k][1] = *(const u32x4*)(src + (16u - half0));
                    }
                };
                // A block = six bf16 products per 32 input and 16 output channels (split_products).  The results of two
                // chunks are added in fp64, and these 16 x 16 sums (rows = pairs 4*gq + v, column = channel 16*cb + jj) to
                // the fp64 accumulators: half the LDS atomics of one addition per chunk (256^3, 64 -> 64 channels, 125
                // taps: call 2.51 against 2.57 ms), and no rounding that one would not make (adding the two in fp32:
                // 2.41 ms, but on rows with few entries further from 64 bits than fp32 products).  Padding pairs land in
                // the dummy row.  Blocks are guarded one by one (uniform branches).
                float held[RB][NB][4];
                auto compute_chunk = [&](unsigned meta, const ChunkRegs<NB, RB>& R, const Entries& E, bool first, bool hold) {
                    const int nb = (int)((meta >> 8) & 0xffu);  // 1 .. RB
#pragma unroll
                    for (int k = 0; k < RB; ++k) {
                        if (k == 0 || k < nb) {  // (a round has at least one block)
                            u32x4 x[2], part[3];
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                x[0][e] = half0 ? R.a[k][1][e] : R.a[k][0][e];
                                x[1][e] = half0 ? R.a[k][0][e] : R.a[k][1][e];
                            }
                            split8(x, part);
                            const unsigned o[4] = {E.out[k].x, E.out[k].y, E.out[k].z, E.out[k].w};
                            unsigned at[4];
#pragma unroll
                            for (int v = 0; v < 4; ++v) at[v] = (o[v] >> kPairRowShift) * (unsigned)(CS * sizeof(double)) + lane_off;
#pragma unroll
                            for (int cb = 0; cb < NB; ++cb) {
                                f32x4 large, small;
                                split_products(part, R.b[0][cb], R.b[1][cb], R.b[2][cb], large, small);
#pragma unroll
                                for (int v = 0; v < 4; ++v) {
                                    const float d = large[v] + small[v];
                                    if (hold)
                                        held[k][cb][v] = d;
                                    else
                                        __hip_atomic_fetch_add((__attribute__((address_space(3))) double*)(size_t)at[v] + cb * 16,
                                                               first ? (double)d : (double)held[k][cb][v] + (double)d,
                                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                                }
                            }
                        }
                    }
                };
                auto rows_of = [&](const Entries& E, unsigned (&in)[RB]) {
                    // (a stale entry past the end of the list may name any row, but such a block is not computed)
#pragma unroll
                    for (int k = 0; k < RB; ++k) {
                        in[k] = E.in[k] & kPairInMask;
                        // opaque: seen through, the compiler takes the product with the row size for a 24-bit one, drops
                        // the mask as superfluous, and then multiplies all 32 bits of the entry
                        asm volatile("" : "+v"(in[k]));
                    }
                };
                constexpr int U = KC % 2 ? 2 : 1;  // rounds per turn of the loop: the two operand sets swap roles
                ChunkRegs<NB, RB> r[2];
                Entries e0, e1;   // of round j and of round j + 1
                unsigned in0[RB], in1[RB];
                unsigned m0 = __builtin_amdgcn_readfirstlane(meta_at(0));
                unsigned m1 = __builtin_amdgcn_readfirstlane(meta_at(1));
                unsigned m_ahead = meta_at(2);
                read_entries(m0, e0);
                read_entries(m1, e1);
                rows_of(e0, in0);
                load_chunk(m0, in0, 0, r[0]);
                for (int j0 = 0; j0 < my_rounds; j0 += U) {
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int j = j0 + u;
                        if (j < my_rounds) {
                            rows_of(e1, in1);
                            const unsigned m2 = __builtin_amdgcn_readfirstlane(m_ahead);
                            m_ahead = meta_at(j + 3);
                            Entries e2;
                            read_entries(m2, e2);
#pragma unroll
                            for (int kc = 0; kc < KC; ++kc) {
                                ChunkRegs<NB, RB>& now = r[(u * KC + kc) & 1];
                                ChunkRegs<NB, RB>& next = r[(u * KC + kc + 1) & 1];
                                if (kc + 1 < KC)
                                    load_chunk(m0, in0, kc + 1, next);
                                else
                                    load_chunk(m1, in1, 0, next);
                                compute_chunk(m0, now, e0, kc % 2 == 0, kc % 2 == 0 && kc + 1 < KC);
                            }
                            e0 = e1;
                            e1 = e2;
#pragma unroll
                            for (int k = 0; k < RB; ++k) in0[k] = in1[k];
                            m0 = m1;
                            m1 = m2;
                        }
                    }
                }
            }
        }
        // Draw the next tile: from the own span, and once that is used up from the other spans, so that no XCD ends
        // before the others.  The last wave does it when its share of the tile is done: it has the smallest share
        // on average and would otherwise only wait at the barrier, which hides the atomic's round trip.
        if (threadIdx.x == NT - 64) {
            int t = -1;
            for (int d = 0; d < kXcds && t < 0; ++d) {
                const int x = (xcd + d) % kXcds;
                const int end_x = (x + 1) * span < n_tiles ? (x + 1) * span : n_tiles;
                if (x * span + per_xcd >= end_x) continue;  // (a span with no tiles to draw)
                const int cand = x * span + per_xcd + (int)atomicAdd(&ctr->conv_ticket[x * kTicketStride], 1u);
                if (cand < end_x) t = cand;
            }
            s_next[parity] = t;
        }
        __syncthreads();
        const int next_tile = s_next[parity];
        // ---- epilogue: one rounding to fp32, bias on the non-zero entries, planar store; the accumulators are
        //      reset on the way.  A lane takes one row, a wave one channel at a time: consecutive rows lie
        //      CS doubles apart, i.e. 2 banks (mod 64), so the 64 reads of a wave spread over all LDS banks, and
        //      the wave's stores form one contiguous 256-byte run of the planar tile.
        {
            constexpr int OCW = (C_OUT + kConvWaves - 1) / kConvWaves, H = kTileRows / 64;
            double acc[OCW][H];
#pragma unroll
            for (int j = 0; j < OCW; ++j) {  // all reads first: one LDS latency for the lot
                const int oc = (wave + j * kConvWaves) < C_OUT ? (wave + j * kConvWaves) : C_OUT - 1;
#pragma unroll
                for (int h = 0; h < H; ++h) acc[j][h] = s_c[(h * 64 + lane) * CS + oc];
            }
#pragma unroll
            for (int j = 0; j < OCW; ++j) {
                const int oc = wave + j * kConvWaves;
                if (C_OUT % kConvWaves == 0 || oc < C_OUT) {
                    // (the weights stand in as a readable address when there is no bias)
                    const float bl = (bias ? bias : (const float*)ws)[oc];
                    const float bv = bias ? bl : 0.0f;
#pragma unroll
                    for (int h = 0; h < H; ++h) {
                        const int r = h * 64 + lane;
                        s_c[r * CS + oc] = 0.0;
                        float x = (float)acc[j][h];
                        if (x != 0.0f) x += bv;
                        resp[((size_t)tile * C_OUT + oc) * kTileRows + r] = x;
                    }
                }
            }
        }
        tile = next_tile;
    }
}

template <int KC, int NB, int LEAVE_ODD>
static hipError_t launch_conv_mfma_split_t(int taps, long long nnz_in, const float* feats, const u32x4* ws,
                                           const float* w, const float* bias,
                                           const unsigned* pairs, const unsigned short* block_tap, const uint2* tile_hdr,
                                           Counters* ctr, float* resp, hipStream_t s) {
    const size_t lds = conv_mfma_lds_bytes(NB * 16);
    // (set on every launch: the attribute belongs to the current device's copy of the kernel, and a flag remembering
    // that it was set would have to be kept per device and guarded between threads for the sake of a microsecond)
    hipError_t e = hipFuncSetAttribute((const void*)k_conv_mfma_split<KC, NB, LEAVE_ODD>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    int per_cu = (int)((160 * 1024) / lds);
    if (per_cu < 1) per_cu = 1;
    if (per_cu > 4) per_cu = 4;    // 16 waves per CU
    const int grid = (device_cu_count() * per_cu + kXcds - 1) / kXcds * kXcds;  // one span of tiles per XCD
    hipLaunchKernelGGL((k_conv_mfma_split<KC, NB, LEAVE_ODD>), dim3(grid), dim3(kConvWaves * 64), lds, s, taps, nnz_in, feats, ws,
                       w, bias, pairs, block_tap, tile_hdr, ctr, resp);
    return hipGetLastError();
}

bool conv_mfma_supported(const Geom& g, int c_in, int c_out, long long nnz_in) {
    if (g.T > 255) return false;  // block_tap holds the tap in one byte
    return ((c_in % 32 == 0 && c_in <= 128) || c_in == 16) && c_out % 16 == 0 && c_out <= 64 && nnz_in > 0 &&
           nnz_in < (1ll << kPairRowShift);
}

hipError_t launch_conv_mfma(const Geom& g, long long nnz_in, int only_odd, const float* feats, int c_in, const float* wb, int c_out,
                            const float* bias, const unsigned* pairs, const unsigned short* block_tap,
                            const uint2* tile_hdr, Counters* ctr, float* resp, hipStream_t s) {
#define SCNN_MFMA_CASE(KC_, NB_)                                                                                  \
    if (c_in == KC_ * 32 && c_out == NB_ * 16)                                                                    \
        return launch_conv_mfma_t<KC_, NB_>(g.T, nnz_in, only_odd, feats, wb, bias, pairs, block_tap, tile_hdr, ctr, resp, s);
    SCNN_MFMA_CASE(1, 1) SCNN_MFMA_CASE(1, 2) SCNN_MFMA_CASE(1, 3) SCNN_MFMA_CASE(1, 4)
    SCNN_MFMA_CASE(2, 1) SCNN_MFMA_CASE(2, 2) SCNN_MFMA_CASE(2, 3) SCNN_MFMA_CASE(2, 4)
    SCNN_MFMA_CASE(3, 1) SCNN_MFMA_CASE(3, 2) SCNN_MFMA_CASE(3, 3) SCNN_MFMA_CASE(3, 4)
    SCNN_MFMA_CASE(4, 1) SCNN_MFMA_CASE(4, 2) SCNN_MFMA_CASE(4, 3) SCNN_MFMA_CASE(4, 4)
#undef SCNN_MFMA_CASE
#define SCNN_MFMA_HALF(NB_)                                                                                       \
    if (c_in == 16 && c_out == NB_ * 16)                                                                          \
        return launch_conv_mfma_t<1, NB_, 1>(g.T, nnz_in, only_odd, feats, wb, bias, pairs, block_tap, tile_hdr, ctr, resp, s);
    SCNN_MFMA_HALF(1) SCNN_MFMA_HALF(2) SCNN_MFMA_HALF(3) SCNN_MFMA_HALF(4)
#undef SCNN_MFMA_HALF
    return hipErrorInvalidValue;
}

hipError_t launch_conv_mfma_split(const Geom& g, long long nnz_in, const float* feats, int c_in, const unsigned short* ws,
                                  const float* w, int leave_odd, int c_out, const float* bias, const unsigned* pairs,
                                  const unsigned short* block_tap, const uint2* tile_hdr, Counters* ctr, float* resp,
                                  hipStream_t s) {
#define SCNN_MFMA_ARGS g.T, nnz_in, feats, (const u32x4*)ws, w, bias, pairs, block_tap, tile_hdr, ctr, resp, s
#define SCNN_MFMA_CASE(KC_, NB_)                                                                                  \
    if (c_in == KC_ * 32 && c_out == NB_ * 16)                                                                    \
        return leave_odd ? launch_conv_mfma_split_t<KC_, NB_, 1>(SCNN_MFMA_ARGS) : launch_conv_mfma_split_t<KC_, NB_, 0>(SCNN_MFMA_ARGS);
#define SCNN_MFMA_FORWARD(KC_, NB_) /* (the adjoint takes these on fp32 products) */                              \
    if (c_in == KC_ * 32 && c_out == NB_ * 16 && !leave_odd) return launch_conv_mfma_split_t<KC_, NB_, 0>(SCNN_MFMA_ARGS);
    SCNN_MFMA_FORWARD(1, 1) SCNN_MFMA_FORWARD(1, 2) SCNN_MFMA_CASE(1, 3) SCNN_MFMA_CASE(1, 4)
    SCNN_MFMA_CASE(2, 1) SCNN_MFMA_CASE(2, 2) SCNN_MFMA_CASE(2, 3) SCNN_MFMA_CASE(2, 4)
    SCNN_MFMA_CASE(3, 1) SCNN_MFMA_CASE(3, 2) SCNN_MFMA_CASE(3, 3) SCNN_MFMA_CASE(3, 4)
    SCNN_MFMA_CASE(4, 1) SCNN_MFMA_CASE(4, 2) SCNN_MFMA_CASE(4, 3) SCNN_MFMA_CASE(4, 4)
#undef SCNN_MFMA_FORWARD
#undef SCNN_MFMA_CASE
#undef SCNN_MFMA_ARGS
    return hipErrorInvalidValue;
}

}  // namespace scnn
