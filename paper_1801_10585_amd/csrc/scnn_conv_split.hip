// Matrix-core convolution on split operands: fp32 inputs and weights as exact sums of three bf16 numbers.
//
// The bf16 matrix instructions of gfx950 do sixteen times the multiply-adds of the fp32 ones.  An fp32 number is the
// exact sum of three bf16 numbers, h + m + l, each the rounding of what the ones before it leave (8 significant bits
// each; split_exact says for which numbers), so a product of two fp32 numbers is the sum of nine bf16 products, every one
// of them exact in fp32.  Six are multiplied (split_products); the three left out are below 2^-23 of the product
// together.  A (tap, 32-channel chunk) of a group of sites is then six instructions per 16 output channels at 2.7 times
// the fp32 instructions' rate, and the result is no further from the exact sum than theirs, on full rows and on rows with
// few entries.
//
// The rest follows k_conv_quad: a wave owns consecutive candidate sites, sorts them by neighbour pattern, and
// multiplies groups of similar sites against the taps that any site of the group has; here a group is the sixteen
// rows of v_mfma_f32_16x16x32_bf16.  All sums of a site stay in the registers of one wave, in an order fixed by the
// data alone: bit-reproducible, no atomics.
#include <type_traits>

#include "scnn_internal.h"

namespace scnn {

constexpr int kSplitSites = 256;             // candidate sites per unit of work (a workgroup of four waves)
constexpr int kSplitMaxTaps = 32;            // per filter (one bit each in a site's neighbour pattern)
constexpr int kSplitSteal = 2;               // XCDs after its own that a workgroup helps once its own has nothing left
constexpr int kSplitChunkMin = 32;           // shortest chunk (units) of the tile order
constexpr int kSplitChunks = 8;              // chunks per XCD
constexpr unsigned kSplitAbsent = 0x80000000u;  // buffer offset of an absent neighbour: out of range, reads as 0

// LDS of a workgroup: the neighbour table (after the walk: 16 columns for the transposition), patterns and positions,
// group unions, the weights of a pass (before the walk: two sets of sort keys), and the lists of the four waves.
__host__ __device__ constexpr int split_tab_words(int taps) { return (taps > 17 ? taps : 17) * kSplitSites; }
__host__ __device__ constexpr int split_list_words(int taps, int nch) { return taps * nch + 1 + taps * nch * 4 + 3; }
__host__ __device__ constexpr int split_lds_words(int taps, int nch, int nb) {
    return split_tab_words(taps) + kSplitSites + 16 + 3 * nb * 256 + 4 * split_list_words(taps, nch);
}
// Waves per SIMD the kernel is built for: its registers are the sums (64 sites x 16 NB channels, 4 or 8 bytes each), the
// weights of a pass and two sets of gathered rows.
__host__ __device__ constexpr int split_waves_per_simd(int nb, int acc64) { return nb == 4 && acc64 ? 2 : 3; }

// A unit of work is a workgroup's 256 consecutive candidate sites (two response tiles).  Each of the four waves looks up
// the neighbours of 64 of them; all 256 are sorted together (the larger the window, the more alike the sixteen sites of
// a group: on shell surfaces 0.37-0.49 of the multiplied rows are neighbours within 64 sites, 0.41-0.55 within 128,
// 0.45-0.61 within 256); then wave i walks the taps for the groups i, i + 4, i + 8, i + 12 with their sums in registers.
//
// What bounds it is what a compute unit's vector memory returns: a row load (sixteen rows 192 bytes apart) takes about 33
// clocks of it, absent neighbours included, so a step's three take 99 for the 384 clocks (NB = 4) that its 24 matrix
// instructions hold one of the four SIMDs; the 12 KB of weights of a (tap, chunk) would take 180 per wave.  So the four
// waves walk the taps together and get the weights through LDS: a wave fetches a quarter of the next ones while it
// multiplies the current ones.  Matrix pipes busy 47 % of the time.  Against k_conv_quad, 32 -> 64 channels, 27 taps:
// 407 -> 220 us at 731 k candidates, 142 -> 78 at 146 k (HIP events); one-wave units of 64 / 128 sites took 295 / 243 at
// 731 k where this took 218.
// NCH = 32-channel chunks of the input; NB = blocks of 16 output channels (2 or 4);
// ACC64: sums over taps and chunks in fp64, else fp32; K3 = 3x3x3 filter (its loops are straight code).
// ODD: values that the parts do not hold (split_exact) are multiplied on fp32 instructions.
template <int NCH, int NB, int ACC64, int K3, int ODD>
__device__ __forceinline__ void split_units(
    Geom g, const unsigned long long* __restrict__ occ, const unsigned* __restrict__ occ_prefix, long long nnz_in,
    const float* __restrict__ feats, const unsigned short* __restrict__ xs, int c_in, const float* __restrict__ w,
    const u32x4* __restrict__ ws, const float* __restrict__ bias, int c_out, int col0, int c_out_all,
    const unsigned* __restrict__ cand_lin, const int* __restrict__ cand_start, const int* __restrict__ tile_start,
    Counters* __restrict__ ctr, float* __restrict__ resp, int n_tiles, unsigned act_mask) {
    constexpr int NS = 4;                                // groups per wave: wave, wave + 4, ..
    constexpr unsigned ROWB = 192;                       // bytes of a row's chunk, split
    typedef typename std::conditional<ACC64 != 0, double, float>::type acc_t;
    extern __shared__ __align__(16) unsigned smem_u[];
    const int T = K3 ? 27 : g.T, K0 = K3 ? 3 : g.K[0], K1 = K3 ? 3 : g.K[1], K2 = K3 ? 3 : g.K[2];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    unsigned* s_tab = smem_u;                                        // [taps][256] buffer offsets, sorted site order
    float* s_tr = (float*)smem_u;                                    // [256][17] after the walk
    unsigned* s_site = smem_u + split_tab_words(T);                  // [256] patterns, keys, positions
    unsigned* s_union = s_site + kSplitSites;                        // [16] taps of each group, then the next unit
    u32x4* s_b = (u32x4*)(s_union + 16);                             // [h | m | l][NB][64] weights of the current pass
    unsigned* s_pass = (unsigned*)(s_b + 3 * NB * 64) + wave * split_list_words(T, NCH);  // [passes + 1] tap | chunk << 8 | groups << 16
    unsigned* s_step = s_pass + (T * NCH + 1);                       // [steps + 3] (tap * 256 + group * 16) * 4 | chunk << 20

    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc((void*)xs, 0, (int)(nnz_in * (long long)(NCH * ROWB)), 0x00020000);
    const unsigned plane = (unsigned)nnz_in * ROWB;      // of one chunk

    // order of the units: as in k_conv_quad (workgroup i runs on XCD i % kXcds; an XCD owns chunks of consecutive units)
    const int n_un = (n_tiles + 1) / 2;
    const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds, per_xcd = gridDim.x / kXcds;
    const int n_chunks = n_un >= kXcds * kSplitChunks * kSplitChunkMin ? kSplitChunks : 1;
    const int chunk = n_un > 0 ? (n_un + kXcds * n_chunks - 1) / (kXcds * n_chunks) : 1;
    auto unit_of = [&](int x, int u) {
        const int c = u / chunk;
        const int un = (c * kXcds + x) * chunk + (u - c * chunk);
        return c < n_chunks && un < n_un ? un : -1;
    };
    unsigned* tickets = ctr->conv_ticket + (col0 >> 6) * kXcds * kTicketStride;

    for (int un = unit_of(xcd, slot); un >= 0;) {
        // ---- the thread's site
        const int tile = un * 2 + (tid >> 7);
        int my_pos = tid;  // sorted position of site `tid`
        int c0 = 0, c1 = 0, c2 = 0, b = 0;
        bool live = false;
        if (tile < n_tiles) {
            b = sample_of_tile(tile_start, g.batch, tile);
            const int c = cand_start[b] + (tile - tile_start[b]) * kTileRows + (tid & 127);
            live = c < cand_start[b + 1];
            if (live) site_of(g, cand_lin[c], c0, c1, c2);
        }
        // ---- its neighbours: buffer offsets and pattern bits
        unsigned m = 0;
        unsigned off[K3 ? 27 : 1];
        const unsigned w_last = (unsigned)g.batch * (unsigned)g.Wps - 1u;
        const int q2s = c2 - g.H[2];          // site of tap k of a line is q2s + k
        int k_lo, k_hi;                       // taps on the line, k_lo <= k < k_hi
        taps_on_line(g.E[2], c2, -g.H[2], K2, k_lo, k_hi);
        const unsigned on_line = (k_hi >= 32 ? ~0u : ((1u << (k_hi > 0 ? k_hi : 0)) - 1u)) & ~((1u << k_lo) - 1u);
        const int n_lines = K0 * K1;
        constexpr int LB = 9;  // lines whose bitmap words are fetched together
        for (int line0 = 0; line0 < n_lines; line0 += LB) {
            unsigned long long word_a[LB], word_b[LB];
            unsigned pre_a[LB], pre_b[LB], p[LB];
            bool ok[LB];
#pragma unroll
            for (int i = 0; i < LB; ++i) {
                const int line = line0 + i < n_lines ? line0 + i : n_lines - 1;
                const int t0 = line / K1, t1 = line - t0 * K1;
                const int q0 = c0 + t0 - g.H[0], q1 = c1 + t1 - g.H[1];
                ok[i] = live && line0 + i < n_lines && (unsigned)q0 < (unsigned)g.E[0] && (unsigned)q1 < (unsigned)g.E[1];
                const unsigned bit = ok[i] ? (unsigned)((q0 * g.E[1] + q1) * g.E[2] + q2s + k_lo) : 0u;
                p[i] = bit & 63u;  // position of the line's first site in word_a
                const unsigned w0 = (unsigned)b * (unsigned)g.Wps + (bit >> 6);
                const unsigned wa = w0 < w_last ? w0 : w_last, wb = wa < w_last ? wa + 1u : wa;
                word_a[i] = occ[wa];
                word_b[i] = occ[wb];
                pre_a[i] = occ_prefix[wa];
                pre_b[i] = occ_prefix[wb];
            }
#pragma unroll
            for (int i = 0; i < LB; ++i) {
                if (!K3 && line0 + i >= n_lines) break;
                const int tap0 = (line0 + i) * K2;
                unsigned long long both = word_a[i] >> p[i];
                if (p[i]) both |= word_b[i] << (64u - p[i]);
                const unsigned raw = (unsigned)both << k_lo;  // occupancy of the sites the taps look at
                const unsigned win = ok[i] ? raw & on_line & (act_mask >> tap0) : 0u;
                m |= win << tap0;
                // Rows are numbered in site order, so the line's occupied sites have consecutive rows, counted from
                // those of word_a below the line's first site, or, if word_a is empty (its row prefix then means
                // nothing), from the first of word_b.
                const unsigned base = word_a[i] ? pre_a[i] + (unsigned)__popcll(word_a[i] & ((1ull << p[i]) - 1ull)) : pre_b[i];
#pragma unroll
                for (int k = 0; k < (K3 ? 3 : 32); ++k) {
                    if (!K3 && k >= K2) break;
                    const unsigned row = base + (unsigned)__popc(raw & ((1u << k) - 1u));
                    const unsigned o = ((win >> k) & 1u) ? row * ROWB : kSplitAbsent;
                    if constexpr (K3)
                        off[3 * i + k] = o;
                    else
                        s_tab[(tap0 + k) * kSplitSites + tid] = o;
                }
            }
        }
        s_site[tid] = m;
        // ---- sort the sites by pattern (bitonic network; ties by site, so the order is a function of the data alone).
        //      The key keeps the pattern's upper 24 bits: which of two sites that differ in the lowest taps only comes
        //      first does not matter.
        unsigned key = (T > 24 ? m >> (T - 24) : m) << 8 | (unsigned)tid;
        unsigned* s_key = (unsigned*)s_b;  // (the weights come later) two sets in turn
        int key_set = 0;
        unsigned place = (unsigned)tid;  // opaque, so that the network's 36 lane masks are not kept for the next unit
        asm volatile("" : "+v"(place));
#pragma unroll
        for (int k = 2; k <= kSplitSites; k <<= 1)
#pragma unroll
            for (int j = k >> 1; j > 0; j >>= 1) {
                unsigned o;
                if (j >= 64) {
                    s_key[key_set * kSplitSites + tid] = key;
                    __syncthreads();
                    o = s_key[key_set * kSplitSites + (tid ^ j)];
                    key_set ^= 1;
                } else {
                    o = __shfl_xor(key, j, 64);
                }
                const unsigned mn = o < key ? o : key, mx = o < key ? key : o;
                key = ((place / k ^ place / j) & 1u) ? mx : mn;
            }
        // patterns of the sorted sites, their union over each group of sixteen
        unsigned u = s_site[key & 255u];
        u |= __shfl_xor(u, 1, 64);
        u |= __shfl_xor(u, 2, 64);
        u |= __shfl_xor(u, 4, 64);
        u |= __shfl_xor(u, 8, 64);
        __syncthreads();
        if ((lane & 15) == 0) s_union[tid >> 4] = u;
        s_site[key & 255u] = (unsigned)tid;
        __syncthreads();
        my_pos = (int)s_site[tid];
        if constexpr (K3) {
#pragma unroll
            for (int t = 0; t < 27; ++t) s_tab[t * kSplitSites + my_pos] = off[t];
        } else {
            for (int t = 0; t < T; ++t) {  // a tap's row into sorted order, in place
                const unsigned o = s_tab[t * kSplitSites + tid];
                __syncthreads();
                s_tab[t * kSplitSites + my_pos] = o;
            }
        }
        // ---- the wave's lists of passes (tap, chunk) and steps (pass, group): lane t writes tap t's
        unsigned sets = 0;
#pragma unroll
        for (int s = 0; s < NS; ++s) sets |= ((s_union[s * 4 + wave] >> (lane & 31)) & 1u) << s;
        if (lane >= T) sets = 0;
        const int cnt = __popc(sets);
        int incl = cnt;
#pragma unroll
        for (int d = 1; d < 32; d <<= 1) {
            const int o = __shfl_up(incl, d, 64);
            if (lane >= d) incl += o;
        }
        unsigned all = 0;
#pragma unroll
        for (int q = 0; q < 16; ++q) all |= s_union[q];
        const unsigned has = __builtin_amdgcn_readfirstlane(all);   // taps of any of the workgroup's groups
        const int n_pass = NCH * (int)__popc(has);
        const int n_step = NCH * (int)__builtin_amdgcn_readlane((unsigned)incl, 31);
        if (lane < T && ((has >> lane) & 1u)) {
            // (all taps of a chunk, then the next chunk: taps next to each other read nearly the same rows, and half of
            // a row's bytes at a time stay in the cache until then)
            const int p0 = (int)__popc(has & ((1u << lane) - 1u)), e0 = incl - cnt;
#pragma unroll
            for (int c = 0; c < NCH; ++c) s_pass[c * (n_pass / NCH) + p0] = (unsigned)lane | (unsigned)c << 8 | sets << 16;
            int at = 0;
#pragma unroll
            for (int s = 0; s < NS; ++s)
                if (sets & (1u << s)) {
#pragma unroll
                    for (int c = 0; c < NCH; ++c)
                        s_step[c * (n_step / NCH) + e0 + at] = (unsigned)((lane * kSplitSites + (s * 4 + wave) * 16) * 4) | (unsigned)c << 20;
                    ++at;
                }
        }
        // read ahead by the pipeline, never multiplied
        if (lane < 3) s_step[n_step + lane] = 0u;
        if (lane == 3) s_pass[n_pass] = 0u;
        __syncthreads();  // the table is complete

        acc_t acc[NS][NB][4];
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[s][nb][v] = (acc_t)0;

        if constexpr (ODD) {
            // ---- the same walk on fp32 instructions, rows and weights as they are, and only the sums of (site, tap) pairs
            //      that exist added, so that infinities and NaN reach what they belong to.  Not pipelined: 32 -> 64
            //      channels on 128^3 x 4, whole call 830 us against 442.
#pragma unroll 1
            for (int p = 0; p < n_pass; ++p) {
                const unsigned info = __builtin_amdgcn_readfirstlane(s_pass[p]);
                const int t = (int)(info & 0xffu), ch = (int)((info >> 8) & 0xffu) * 32 + (lane >> 4) * 8;
                float wv[NB][8];
#pragma unroll
                for (int i = 0; i < 8; ++i)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        const int oc = nb * 16 + (lane & 15);
                        wv[nb][i] = ch < c_in && oc < c_out ? w[((size_t)t * c_in + ch + i) * c_out_all + col0 + oc] : 0.0f;
                    }
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    if (!(info & (0x10000u << s))) continue;
                    const unsigned* at = s_tab + t * kSplitSites + (s * 4 + wave) * 16;
                    const unsigned o = at[lane & 15];
                    float4 x[2] = {make_float4(0.f, 0.f, 0.f, 0.f), make_float4(0.f, 0.f, 0.f, 0.f)};
                    if (o < plane && ch < c_in) {
                        const float4* row = (const float4*)(feats + (size_t)(o / ROWB) * c_in + ch);
                        x[0] = row[0];
                        x[1] = row[1];
                    }
                    const float xv[8] = {x[0].x, x[0].y, x[0].z, x[0].w, x[1].x, x[1].y, x[1].z, x[1].w};
                    f32x4 d[NB];
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) d[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int i = 0; i < 8; ++i)
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb)
                            d[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[i], wv[nb][i], d[nb], 0, 0, 0);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const bool pair = at[4 * (lane >> 4) + v] < plane;
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb) acc[s][nb][v] += pair ? (acc_t)d[nb][v] : (acc_t)0;
                    }
                }
            }
        } else if (n_pass > 0) {
            // ---- the walk.  Pipeline per step: list entry two steps ahead (LDS), the group's neighbour offsets one
            //      step ahead (LDS), the gathered rows one step ahead (buffer loads); per pass: the wave's share of the
            //      weights one pass ahead.
            constexpr int NSH = (3 * NB + 3) / 4;  // 1 KB pieces of the weights per wave (the last wave may have fewer)
            u32x4 a_next[3], bw[3][NB];
            const unsigned tab_lane = (unsigned)(size_t)s_tab + (unsigned)(lane & 15) * 4u;
            const unsigned kg_off = (unsigned)(lane >> 4) * 16u;
            auto tab_at = [&](unsigned e) {
                return *(const __attribute__((address_space(3))) unsigned*)(size_t)(tab_lane + (e & 0xffffu));
            };
            auto load_a = [&](unsigned o, unsigned e) {
                const unsigned vo = o + kg_off, so = NCH > 1 ? ((e >> 20) & 7u) * plane : 0u;
                a_next[0] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, vo, so, 0);
                a_next[1] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, vo + 64u, so, 0);
                a_next[2] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, vo + 128u, so, 0);
            };
            auto fetch_b = [&](unsigned info) {
                const u32x4* q = ws + (size_t)((info & 0xffu) * NCH + ((info >> 8) & 0xffu)) * (3 * NB * 64);
#pragma unroll
                for (int j = 0; j < NSH; ++j)
                    if (3 * NB % 4 == 0 || j * 4 + wave < 3 * NB)
                        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)((q + (j * 4 + wave) * 64) + lane),
                                                         (__attribute__((address_space(3))) void*)(s_b + (j * 4 + wave) * 64), 16, 0, 0);
            };
            unsigned info = __builtin_amdgcn_readfirstlane(s_pass[0]), next_raw = s_pass[1];
            fetch_b(info);
            const unsigned e_first = __builtin_amdgcn_readfirstlane(s_step[0]);
            unsigned e_1 = __builtin_amdgcn_readfirstlane(s_step[1]);
            load_a(tab_at(e_first), e_first);
            unsigned off_1 = tab_at(e_1);
            unsigned e_raw = s_step[2];
            int step = 0;
            // One step = one group against one pass: six products per 16 output channels (split_products), and their sum
            // added to the group's.
            auto run_step = [&](acc_t (&ac)[NB][4]) {
                // (the copies and the barrier keep the loads in front of the products: left alone, the compiler loads
                // straight into the operands, the last of them only after its last product)
                u32x4 a[3];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    a[k] = a_next[k];
                    asm volatile("" : "+v"(a[k]));
                }
                load_a(off_1, e_1);
                e_1 = __builtin_amdgcn_readfirstlane(e_raw);
                off_1 = tab_at(e_1);
                e_raw = s_step[step + 3];
                ++step;
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    f32x4 large, small;
                    split_products(a, bw[0][nb], bw[1][nb], bw[2][nb], large, small);
#pragma unroll
                    for (int v = 0; v < 4; ++v) ac[nb][v] += (acc_t)(large[v] + small[v]);
                }
            };
            for (int p = 0;;) {
                __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's share of them has arrived
                __syncthreads();                     // the weights of pass p are in LDS
#pragma unroll
                for (int k = 0; k < 3; ++k)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) bw[k][nb] = s_b[(k * NB + nb) * 64 + lane];
                __syncthreads();  // .. and in every wave's registers
                const unsigned groups = info >> 16;
                info = __builtin_amdgcn_readfirstlane(next_raw);
                const bool more = ++p < n_pass;
                if (more) fetch_b(info);
                next_raw = s_pass[more ? p + 1 : p];
#pragma unroll
                for (int s = 0; s < NS; ++s)
                    if (groups & (1u << s)) run_step(acc[s]);
                if (!more) break;
                }
        }

        // ---- next unit: ask the own span's counter now, look at the answer after the epilogue
        unsigned ticket = 0;
        if (tid == 0) ticket = atomicAdd(&tickets[xcd * kTicketStride], 1u);
        __syncthreads();  // every wave is done with the table

        // ---- epilogue: bias on the non-zero entries, 16 channels at a time through LDS into candidate order (thread =
        //      site), 256-byte stores to the planar tile.  Sites past the sample's end store 0.
        {
            float* tr_w = s_tr + (wave * 16 + 4 * (lane >> 4)) * 17 + (lane & 15);
            const float* tr_r = s_tr + my_pos * 17;
            float* dst = resp + ((size_t)(un * 2 + (wave >> 1)) * c_out_all + col0) * kTileRows + (wave & 1) * 64;  // (the same for the wave)
            const bool mine = un * 2 + (wave >> 1) < n_tiles;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const int c_n = c_out - nb * 16;
                if (c_n <= 0) break;
                if (nb) __syncthreads();
                if (bias) {
                    const float bv = (lane & 15) < c_n ? bias[nb * 16 + (lane & 15)] : 0.0f;
#pragma unroll
                    for (int s = 0; s < NS; ++s)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const float x = (float)acc[s][nb][v];
                            tr_w[(s * 64 + v) * 17] = x != 0.0f ? x + bv : x;
                        }
                } else {
#pragma unroll
                    for (int s = 0; s < NS; ++s)
#pragma unroll
                        for (int v = 0; v < 4; ++v) tr_w[(s * 64 + v) * 17] = (float)acc[s][nb][v];
                }
                __syncthreads();
                if (mine) {
                    if (c_n >= 16) {
                        float v[16];
#pragma unroll
                        for (int c = 0; c < 16; ++c) v[c] = tr_r[c];
#pragma unroll
                        for (int c = 0; c < 16; ++c) (dst + (size_t)(nb * 16 + c) * kTileRows)[lane] = v[c];
                    } else {
#pragma unroll 1
                        for (int c = 0; c < c_n; ++c) (dst + (size_t)(nb * 16 + c) * kTileRows)[lane] = tr_r[c];
                    }
                }
            }
        }
        if (tid == 0) {
            // the own units are used up: help the next XCDs, so that none ends long before the others
            int next = unit_of(xcd, per_xcd + (int)ticket);
            for (int d = 1; d <= kSplitSteal && next < 0; ++d) {
                const int x = (xcd + d) % kXcds;
                if (unit_of(x, per_xcd) < 0) continue;  // (an XCD with nothing to draw)
                next = unit_of(x, per_xcd + (int)atomicAdd(&tickets[x * kTicketStride], 1u));
            }
            s_union[0] = (unsigned)next;
        }
        __syncthreads();
        un = __builtin_amdgcn_readfirstlane((int)s_union[0]);
        __syncthreads();
    }
}

// (two copies of the loop: with the fp32 walk as a branch inside one, its operands' registers cost the other 3-5 %)
template <int NCH, int NB, int ACC64, int K3>
__global__ __launch_bounds__(256, split_waves_per_simd(NB, ACC64)) void k_conv_quad_split(
    Geom g, const unsigned long long* __restrict__ occ, const unsigned* __restrict__ occ_prefix, long long nnz_in,
    const float* __restrict__ feats, const unsigned short* __restrict__ xs, int c_in, const float* __restrict__ w,
    const u32x4* __restrict__ ws, const float* __restrict__ bias, int c_out, int col0, int c_out_all,
    const int* __restrict__ tap_active, const unsigned* __restrict__ cand_lin, const int* __restrict__ cand_start,
    const int* __restrict__ tile_start,
    Counters* __restrict__ ctr, float* __restrict__ resp) {
    // (with the flag: one wait for all three)
    const int n_tiles = (int)ctr->n_tiles, T = K3 ? 27 : g.T, lane = threadIdx.x & 63;
    const unsigned act_mask = (unsigned)__ballot(lane < T && tap_active[lane < T ? lane : 0] != 0);
    if (__builtin_amdgcn_readfirstlane(ctr->odd))
        split_units<NCH, NB, ACC64, K3, 1>(g, occ, occ_prefix, nnz_in, feats, xs, c_in, w, ws, bias, c_out, col0, c_out_all,
                                           cand_lin, cand_start, tile_start, ctr, resp, n_tiles, act_mask);
    else
        split_units<NCH, NB, ACC64, K3, 0>(g, occ, occ_prefix, nnz_in, feats, xs, c_in, w, ws, bias, c_out, col0, c_out_all,
                                           cand_lin, cand_start, tile_start, ctr, resp, n_tiles, act_mask);
}

// (The channel counts that conv_kernel_for's rule was measured at; the kernel would take any multiple of eight up to 128.)
bool conv_split_supported(const Geom& g, int c_in, int c_out, long long nnz_in) {
    const bool shape = (c_in == 16 || c_in == 24 || c_in == 32 || c_in == 40 || c_in == 48 || c_in == 64 || c_in == 96 ||
                        c_in == 128) &&
                       c_out >= 1 && c_out <= kQuadMaxCout;
    return g.T <= kSplitMaxTaps && shape && nnz_in > 0 && nnz_in * round_up(c_in, 32) * 6 < (1ll << 31);
}

template <int NCH, int NB, int ACC64, int K3>
static hipError_t launch_conv_split_t(const Geom& g, const unsigned long long* occ, const unsigned* occ_prefix,
                                      long long nnz_in, const float* feats, const unsigned short* xs, int c_in,
                                      const float* w, const unsigned short* ws, const float* bias, int c_out, int col0,
                                      int c_out_all, const int* tap_active, const unsigned* cand_lin,
                                      const int* cand_start, const int* tile_start, Counters* ctr, float* resp, int cus,
                                      hipStream_t s) {
    const size_t lds = (size_t)split_lds_words(g.T, NCH, NB) * 4;
    // (the same for every filter: another thread's launch may lie between this and ours)
    hipError_t e = hipFuncSetAttribute((const void*)k_conv_quad_split<NCH, NB, ACC64, K3>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, split_lds_words(kSplitMaxTaps, NCH, NB) * 4);
    if (e != hipSuccess) return e;
    // as many workgroups as run at once (they are persistent); a multiple of kXcds: one span of units per XCD
    int per_cu = split_waves_per_simd(NB, ACC64);
    while (per_cu > 1 && (size_t)per_cu * lds > 160 * 1024) --per_cu;
    const int grid = (cus * per_cu + kXcds - 1) / kXcds * kXcds;
    hipLaunchKernelGGL((k_conv_quad_split<NCH, NB, ACC64, K3>), dim3(grid), dim3(256), lds, s, g, occ, occ_prefix,
                       nnz_in, feats, xs, c_in, w, (const u32x4*)ws, bias, c_out, col0, c_out_all, tap_active, cand_lin,
                       cand_start, tile_start, ctr, resp);
    return hipGetLastError();
}

hipError_t launch_conv_split(const Geom& g, const unsigned long long* occ, const unsigned* occ_prefix, long long nnz_in,
                             const float* feats, const unsigned short* xs, int c_in, const float* w,
                             const unsigned short* ws, int c_out, const float* bias, const int* tap_active,
                             const unsigned* cand_lin, const int* cand_start, const int* tile_start, Counters* ctr,
                             float* resp, int cus, hipStream_t s) {
    const int nch = (c_in + 31) / 32;
    const bool k3 = g.K[0] == 3 && g.K[1] == 3 && g.K[2] == 3;
    for (int col0 = 0; col0 < c_out; col0 += 64) {
        const int cg = c_out - col0 < 64 ? c_out - col0 : 64;
        const unsigned short* ws_g = ws + (size_t)(col0 >> 6) * split_filter_elems(g.T, c_in);
        const float* bias_g = bias ? bias + col0 : nullptr;
        hipError_t e = hipErrorInvalidValue;
#define SCNN_SPLIT_ARGS g, occ, occ_prefix, nnz_in, feats, xs, c_in, w, ws_g, bias_g, cg, col0, c_out, tap_active, cand_lin, cand_start, tile_start, ctr, resp, cus, s
#define SCNN_SPLIT_CASE(CH, ACC)                                                                                      \
    if (nch == CH) {                                                                                                  \
        if (cg > 32)                                                                                                  \
            e = k3 ? launch_conv_split_t<CH, 4, ACC, 1>(SCNN_SPLIT_ARGS) : launch_conv_split_t<CH, 4, ACC, 0>(SCNN_SPLIT_ARGS); \
        else                                                                                                          \
            e = k3 ? launch_conv_split_t<CH, 2, ACC, 1>(SCNN_SPLIT_ARGS) : launch_conv_split_t<CH, 2, ACC, 0>(SCNN_SPLIT_ARGS); \
    }
        SCNN_SPLIT_CASE(1, 0) SCNN_SPLIT_CASE(2, 1) SCNN_SPLIT_CASE(3, 1) SCNN_SPLIT_CASE(4, 1)
#undef SCNN_SPLIT_CASE
#undef SCNN_SPLIT_ARGS
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace scnn
