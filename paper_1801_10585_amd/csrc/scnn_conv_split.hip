// Matrix-core convolution on split operands: fp32 inputs and weights as exact sums of three bf16 numbers.
//
// The bf16 matrix instructions of gfx950 do sixteen times the multiply-adds of the fp32 ones.  An fp32 number is the
// exact sum of three bf16 numbers, h + m + l, each the rounding of what the ones before it leave (8 significant bits
// each), so a product of two fp32 numbers is the sum of nine bf16 products, every one of them exact in fp32.  Six are
// multiplied, smallest first: x_l w_h + x_h w_l + x_m w_m + x_m w_h + x_h w_m + x_h w_h; the three left out are below
// 2^-24 of the product together.  A (tap, 32-channel chunk) of a group of sites is then six instructions per 16 output
// channels, each of which rounds its fp32 sum once, where the fp32 instructions round after every channel: the
// result is closer to the exact sum than theirs, at 2.7 times their rate.
//
// The rest follows k_conv_quad: a wave owns consecutive candidate sites, sorts them by neighbour pattern, and
// multiplies groups of similar sites against the taps that any site of the group has; here a group is the sixteen
// rows of v_mfma_f32_16x16x32_bf16.  All sums of a site stay in the registers of one wave, in an order fixed by the
// data alone: bit-reproducible, no atomics.
#include <type_traits>

#include "scnn_internal.h"

#ifndef SCNN_RPL
#define SCNN_RPL 2
#endif

namespace scnn {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kSplitWaves = 4;               // waves per workgroup
constexpr int kSplitSteal = 2;               // XCDs after its own that a wave helps once its own has nothing left
constexpr int kSplitChunkMin = 64;           // shortest chunk (units) of the tile order
constexpr int kSplitChunks = 8;              // chunks per XCD
constexpr unsigned kSplitAbsent = 0x80000000u;  // buffer offset of an absent neighbour: out of range, reads as 0

template <int RPL>
__host__ __device__ constexpr int split_lds_words(int taps, int nch) {
    constexpr int sites = 64 * RPL;
    const int walk = taps * sites + taps * nch + taps * nch * (sites / 16) + 4 + sites;
    return walk > sites * 17 ? walk : sites * 17;
}

// Input rows as the kernel reads them: [row][32-channel chunk][h | m | l][32] bf16 (192 bytes per row and chunk), so
// that a lane's eight channels of a part are one 16-byte load.  Bound by memory: 4 bytes read, 6 written per value.
__global__ __launch_bounds__(256) void k_split_rows(const float* __restrict__ feats, long long n_imm,
                                                    const long long* __restrict__ n_dev, long long n_cap, int c_in,
                                                    int nch, unsigned short* __restrict__ xs) {
    long long n = n_dev ? *n_dev : n_imm;
    if (n > n_cap) n = n_cap;
    if (n < 0) n = 0;
    const int per_row = nch * 4;  // pieces of eight channels
    const long long total = n * per_row;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (long long)gridDim.x * blockDim.x) {
        const long long row = i / per_row;
        const int p = (int)(i - row * per_row), chunk = p >> 2, piece = p & 3, c0 = chunk * 32 + piece * 8;
        float v[8];
        const float4* src = (const float4*)(feats + row * c_in + c0);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            float4 f = make_float4(0.f, 0.f, 0.f, 0.f);
            if (c0 + 4 * q < c_in) f = src[q];
            v[4 * q] = f.x; v[4 * q + 1] = f.y; v[4 * q + 2] = f.z; v[4 * q + 3] = f.w;
        }
        unsigned short part[3][8];
#pragma unroll
        for (int e = 0; e < 8; ++e) split3(v[e], part[0][e], part[1][e], part[2][e]);
        uint4* dst = (uint4*)(xs + (row * nch + chunk) * 96 + piece * 8);
#pragma unroll
        for (int k = 0; k < 3; ++k)
            dst[k * 4] = make_uint4(part[k][0] | (unsigned)part[k][1] << 16, part[k][2] | (unsigned)part[k][3] << 16,
                                    part[k][4] | (unsigned)part[k][5] << 16, part[k][6] | (unsigned)part[k][7] << 16);
    }
}

// NCH = 32-channel chunks of the input; NB = blocks of 16 output channels (2 or 4); RPL = sites per lane (a wave owns
// 64 * RPL); ACC64: sums over taps and chunks in fp64, else fp32; K3 = 3x3x3 filter (its loops are straight code).
template <int NCH, int NB, int RPL, int ACC64, int K3>
__global__ __launch_bounds__(kSplitWaves * 64, 2) void k_conv_quad_split(
    Geom g, const unsigned long long* __restrict__ occ, const unsigned* __restrict__ occ_prefix, long long nnz_in,
    const unsigned short* __restrict__ xs, const u32x4* __restrict__ ws, const float* __restrict__ bias, int c_out,
    int col0, int c_out_all, const int* __restrict__ tap_active, const unsigned* __restrict__ cand_lin,
    const int* __restrict__ cand_start, const int* __restrict__ tile_start, Counters* __restrict__ ctr,
    float* __restrict__ resp) {
    constexpr int SITES = 64 * RPL, NS = SITES / 16;     // sites and groups of sixteen per unit
    constexpr unsigned ROWB = NCH * 192;                 // bytes of a split row
    constexpr int UPT = kTileRows / SITES;               // units per response tile
    typedef typename std::conditional<ACC64 != 0, double, float>::type acc_t;
    extern __shared__ __align__(16) unsigned smem_u[];
    const int T = K3 ? 27 : g.T, K0 = K3 ? 3 : g.K[0], K1 = K3 ? 3 : g.K[1], K2 = K3 ? 3 : g.K[2];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    unsigned* s_tab = smem_u + wave * split_lds_words<RPL>(T, NCH);  // [taps][SITES] buffer offsets, sorted site order
    unsigned* s_pass = s_tab + T * SITES;                            // [passes] tap | chunk << 8 | groups << 16
    unsigned* s_step = s_pass + T * NCH;                             // [steps + 3] (tap * SITES + group * 16) * 4 | chunk << 20
    unsigned* s_site = s_step + (T * NCH * NS + 4);                  // [SITES] patterns, then sorted positions
    float* s_tr = (float*)s_tab;                                     // [SITES][17] after the walk

    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc((void*)xs, 0, (int)(nnz_in * (long long)ROWB), 0x00020000);
    const unsigned act_mask = (unsigned)__ballot(lane < T && tap_active[lane < T ? lane : 0] != 0);

    // order and units of work: as in k_conv_quad
    const int n_un = UPT * (int)ctr->n_tiles;
    const int xcd = blockIdx.x % kXcds, slot = (blockIdx.x / kXcds) * kSplitWaves + wave, per_xcd = (gridDim.x / kXcds) * kSplitWaves;
    const int n_chunks = n_un >= kXcds * kSplitChunks * kSplitChunkMin ? kSplitChunks : 1;
    const int chunk = n_un > 0 ? (n_un + kXcds * n_chunks - 1) / (kXcds * n_chunks) : 1;
    auto unit_of = [&](int x, int u, int& lo, int& hi) {
        int vspan = 0;  // units of XCD x
        for (int c = 0; c < n_chunks; ++c) {
            const int left = n_un - (c * kXcds + x) * chunk;
            vspan += left <= 0 ? 0 : (left < chunk ? left : chunk);
        }
        lo = 0;
        hi = SITES;
        const int whole = (vspan / per_xcd) * per_xcd, rest = vspan - whole;
        const int sl = rest * 4 <= per_xcd ? 2 : (rest * 2 <= per_xcd ? 1 : 0);
        int v = u;
        if (u >= whole) {
            const int r = u - whole;
            v = whole + (r >> sl);
            lo = (r & ((1 << sl) - 1)) * (SITES >> sl);
            hi = lo + (SITES >> sl);
        }
        if (v >= vspan) return -1;
        const int c = v / chunk;
        return (c * kXcds + x) * chunk + (v - c * chunk);
    };
    unsigned* tickets = ctr->conv_ticket + (col0 >> 6) * kXcds * kTicketStride;

    int row_lo = 0, row_hi = SITES, lo_next = 0, hi_next = 0;
    bool own_done = unit_of(xcd, per_xcd, lo_next, hi_next) < 0;
    for (int un = unit_of(xcd, slot, row_lo, row_hi); un >= 0;) {
        const int tile = un / UPT, part = un % UPT;
        const int b = sample_of_tile(tile_start, g.batch, tile);
        const int first = cand_start[b] + (tile - tile_start[b]) * kTileRows + part * SITES;
        int nrows = cand_start[b + 1] - first;
        nrows = nrows > SITES ? SITES : nrows;

        int my_pos[RPL];  // sorted position of site r * 64 + lane
#pragma unroll
        for (int r = 0; r < RPL; ++r) my_pos[r] = r * 64 + lane;
        int n_pass = 0, n_step = 0;

        if (nrows > row_lo) {
            // ---- neighbours of the sites: buffer offsets into s_tab[tap][site], pattern bits into `mask`
            unsigned mask[RPL];
            const int n_lines = K0 * K1;
            const unsigned w_last = (unsigned)g.batch * (unsigned)g.Wps - 1u;
#pragma unroll
            for (int r = 0; r < RPL; ++r) {
                const int site = r * 64 + lane;
                int c0 = 0, c1 = 0, c2 = 0;
                const bool live = site < nrows && site >= row_lo && site < row_hi;
                if (live) site_of(g, cand_lin[first + site], c0, c1, c2);
                unsigned tab_w = (unsigned)(size_t)s_tab + (unsigned)site * 4u;
                asm volatile("" : "+v"(tab_w));
                const int q2s = c2 - g.H[2];          // site of tap k of a line is q2s + k
                const int k_lo = q2s < 0 ? -q2s : 0;  // first tap whose site is on the line
                const int k_hi = g.E[2] - q2s < K2 ? g.E[2] - q2s : K2;
                const unsigned on_line = (k_hi >= 32 ? ~0u : ((1u << (k_hi > 0 ? k_hi : 0)) - 1u)) & ~((1u << k_lo) - 1u);
                unsigned m = 0;
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
                        // Rows are numbered in site order, so the line's occupied sites have consecutive rows, counted
                        // from those of word_a below the line's first site, or, if word_a is empty (its row prefix then
                        // means nothing), from the first of word_b.
                        const unsigned base = word_a[i] ? pre_a[i] + (unsigned)__popcll(word_a[i] & ((1ull << p[i]) - 1ull)) : pre_b[i];
                        for (int k = 0; k < K2; ++k) {
                            const unsigned row = base + (unsigned)__popc(raw & ((1u << k) - 1u));
                            const unsigned off = ((win >> k) & 1u) ? row * ROWB : kSplitAbsent;
                            *(__attribute__((address_space(3))) unsigned*)(size_t)(tab_w + (unsigned)(tap0 + k) * (SITES * 4u)) = off;
                        }
                    }
                }
                mask[r] = m;
                s_site[site] = m;
            }
            // ---- sort the sites by pattern (bitonic network; ties by site, so the order is a function of the data
            //      alone).  The key keeps the pattern's upper 25 bits: which of two sites that differ in the first
            //      two taps only comes first does not matter.
            unsigned key[RPL];
            const int drop = T > 25 ? T - 25 : 0;
#pragma unroll
            for (int r = 0; r < RPL; ++r) key[r] = (mask[r] >> drop) << 7 | (unsigned)(r * 64 + lane);
#pragma unroll
            for (int k = 2; k <= SITES; k <<= 1)
#pragma unroll
                for (int j = k >> 1; j > 0; j >>= 1) {
                    if (RPL == 2 && j == 64) {
                        const unsigned a = key[0], c = key[RPL - 1];
                        key[0] = a < c ? a : c;
                        key[RPL - 1] = a < c ? c : a;
                    } else {
#pragma unroll
                        for (int r = 0; r < RPL; ++r) {
                            const unsigned o = __shfl_xor(key[r], j, 64);
                            const unsigned mn = o < key[r] ? o : key[r], mx = o < key[r] ? key[r] : o;
                            const bool want_min = (((r * 64 + lane) & k) == 0) == ((lane & j) == 0);
                            key[r] = want_min ? mn : mx;
                        }
                    }
                }
            // patterns of the sorted sites, their union over each group of sixteen
            unsigned us[NS];
#pragma unroll
            for (int r = 0; r < RPL; ++r) {
                unsigned u = s_site[key[r] & 127u];
                u |= __shfl_xor(u, 1, 64);
                u |= __shfl_xor(u, 2, 64);
                u |= __shfl_xor(u, 4, 64);
                u |= __shfl_xor(u, 8, 64);
#pragma unroll
                for (int q = 0; q < 4; ++q) us[r * 4 + q] = __builtin_amdgcn_readlane(u, 16 * q);
            }
#pragma unroll
            for (int r = 0; r < RPL; ++r) s_site[key[r] & 127u] = (unsigned)(r * 64 + lane);
#pragma unroll
            for (int r = 0; r < RPL; ++r) my_pos[r] = (int)s_site[r * 64 + lane];
            // rows of the table into sorted order, in place (a wave's LDS reads finish before its next writes)
#pragma unroll 9
            for (int t = 0; t < T; ++t) {
                unsigned v[RPL];
#pragma unroll
                for (int r = 0; r < RPL; ++r) v[r] = s_tab[t * SITES + r * 64 + lane];
#pragma unroll
                for (int r = 0; r < RPL; ++r) s_tab[t * SITES + my_pos[r]] = v[r];
            }
            // ---- lists of passes (tap, chunk) and steps (pass, group): lane t writes tap t's
            unsigned sets = 0;
#pragma unroll
            for (int s = 0; s < NS; ++s) sets |= ((us[s] >> (lane & 31)) & 1u) << s;
            if (lane >= T) sets = 0;
            const int cnt = __popc(sets);
            int incl = cnt;
#pragma unroll
            for (int d = 1; d < 32; d <<= 1) {
                const int o = __shfl_up(incl, d, 64);
                if (lane >= d) incl += o;
            }
            const unsigned long long has = __ballot(cnt > 0);
            n_pass = NCH * (int)__popcll(has);
            n_step = NCH * (int)__builtin_amdgcn_readlane((unsigned)incl, 31);
            if (cnt > 0) {
                const int p0 = NCH * (int)__popcll(has & ((1ull << lane) - 1ull)), e0 = NCH * (incl - cnt);
#pragma unroll
                for (int c = 0; c < NCH; ++c) s_pass[p0 + c] = (unsigned)lane | (unsigned)c << 8 | sets << 16;
                int at = 0;
#pragma unroll
                for (int s = 0; s < NS; ++s)
                    if (sets & (1u << s)) {
#pragma unroll
                        for (int c = 0; c < NCH; ++c)
                            s_step[e0 + c * cnt + at] = (unsigned)((lane * SITES + s * 16) * 4) | (unsigned)c << 20;
                        ++at;
                    }
            }
            if (lane < 3) s_step[n_step + lane] = 0u;  // read ahead by the pipeline, never multiplied
        }

        acc_t acc[NS][NB][4];
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[s][nb][v] = (acc_t)0;

        if (n_step > 0) {
            // ---- the walk.  Pipeline per step: list entry two steps ahead (LDS), the group's neighbour offsets one
            //      step ahead (LDS), the gathered rows one step ahead (buffer loads).
            u32x4 a_next[3], bw[3][NB];
            const unsigned tab_lane = (unsigned)(size_t)s_tab + (unsigned)(lane & 15) * 4u;
            const unsigned kg_off = (unsigned)(lane >> 4) * 16u;
            auto tab_at = [&](unsigned e) {
                return *(const __attribute__((address_space(3))) unsigned*)(size_t)(tab_lane + (e & 0xffffu));
            };
            auto load_a = [&](unsigned off, unsigned e) {
                const unsigned vo = off + (kg_off + (NCH > 1 ? ((e >> 20) & 7u) * 192u : 0u));
                a_next[0] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, vo, 0, 0);
                a_next[1] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, vo + 64u, 0, 0);
                a_next[2] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, vo + 128u, 0, 0);
            };
            auto load_b = [&](unsigned info) {
                const u32x4* p = ws + ((size_t)((info & 0xffu) * NCH + ((info >> 8) & 0xffu)) * (3 * NB * 64) + lane);
#pragma unroll
                for (int k = 0; k < 3; ++k)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) bw[k][nb] = p[(k * NB + nb) * 64];
            };
            const unsigned e_first = __builtin_amdgcn_readfirstlane(s_step[0]);
            unsigned e_1 = __builtin_amdgcn_readfirstlane(s_step[1]);
            unsigned p_info = __builtin_amdgcn_readfirstlane(s_pass[0]);
            load_b(p_info);
            load_a(tab_at(e_first), e_first);
            unsigned off_1 = tab_at(e_1);
            unsigned e_raw = s_step[2];
            int step = 0;
            auto run_step = [&](acc_t (&ac)[NB][4]) {
                bf16x8 a[3];
#pragma unroll
                for (int k = 0; k < 3; ++k) a[k] = __builtin_bit_cast(bf16x8, a_next[k]);
                load_a(off_1, e_1);
                e_1 = __builtin_amdgcn_readfirstlane(e_raw);
                off_1 = tab_at(e_1);
                e_raw = s_step[step + 3];
                ++step;
                f32x4 d[NB];
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) d[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
                // smallest products first: (l,h) (h,l) (m,m) (m,h) (h,m) (h,h)
                constexpr int PX[6] = {2, 0, 1, 1, 0, 0}, PW[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
                for (int q = 0; q < 6; ++q)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
                        d[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[PX[q]], __builtin_bit_cast(bf16x8, bw[PW[q]][nb]), d[nb], 0, 0, 0);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                    for (int v = 0; v < 4; ++v) ac[nb][v] += (acc_t)d[nb][v];
            };
            for (int p = 0; p < n_pass; ++p) {
                const unsigned sets = p_info >> 16;
#pragma unroll
                for (int s = 0; s < NS; ++s)
                    if (sets & (1u << s)) run_step(acc[s]);
                if (p + 1 < n_pass) {
                    p_info = __builtin_amdgcn_readfirstlane(s_pass[p + 1]);
                    load_b(p_info);
                }
            }
        }

        // ---- next unit: ask the own span's counter now and look at the answer after the epilogue
        unsigned ticket = 0;
        if (!own_done && lane == 0) ticket = atomicAdd(&tickets[xcd * kTicketStride], 1u);

        // ---- epilogue: bias on the non-zero entries, sixteen channels at a time through LDS into candidate order
        //      (lane = site), 256-byte stores to the planar tile.  Sites past the sample's end store 0.
        {
            const int col = lane & 15;
            float* tr_w = s_tr + 4 * (lane >> 4) * 17 + col;
            float* dst = resp + ((size_t)tile * c_out_all + col0) * kTileRows + part * SITES + lane;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const int c_end = c_out - nb * 16 < 16 ? c_out - nb * 16 : 16;
                if (c_end <= 0) break;
                const float bv = (bias && col < c_end) ? bias[nb * 16 + col] : 0.0f;
#pragma unroll
                for (int s = 0; s < NS; ++s)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        float x = (float)acc[s][nb][v];
                        if (bias && x != 0.0f) x += bv;
                        tr_w[(s * 16 + v) * 17] = x;
                    }
#pragma unroll
                for (int r = 0; r < RPL; ++r) {
                    const float* tr_r = s_tr + my_pos[r] * 17;
                    const bool mine = r * 64 + lane >= row_lo && r * 64 + lane < row_hi;
                    float* out = dst + (size_t)nb * 16 * kTileRows + r * 64;
                    float v[16];
#pragma unroll
                    for (int c = 0; c < 16; ++c) v[c] = tr_r[c];
                    if (mine) {
                        if (c_end == 16) {
#pragma unroll
                            for (int c = 0; c < 16; ++c) out[(size_t)c * kTileRows] = v[c];
                        } else {
#pragma unroll
                            for (int c = 0; c < 16; ++c)
                                if (c < c_end) out[(size_t)c * kTileRows] = v[c];
                        }
                    }
                }
            }
        }
        int next_un = -1;
        if (!own_done) {
            next_un = unit_of(xcd, per_xcd + (int)__builtin_amdgcn_readfirstlane(ticket), lo_next, hi_next);
            own_done = next_un < 0;
        }
        if (own_done) {
            int got = -1;
            if (lane == 0) {
                for (int d = 1; d <= kSplitSteal && got < 0; ++d) {
                    const int x = (xcd + d) % kXcds;
                    if (unit_of(x, per_xcd, lo_next, hi_next) < 0) continue;
                    got = unit_of(x, per_xcd + (int)atomicAdd(&tickets[x * kTicketStride], 1u), lo_next, hi_next);
                }
            }
            next_un = __builtin_amdgcn_readfirstlane(got);
            lo_next = __builtin_amdgcn_readfirstlane(lo_next);
            hi_next = __builtin_amdgcn_readfirstlane(hi_next);
        }
        row_lo = lo_next;
        row_hi = hi_next;
        un = next_un;
    }
}

bool conv_split_supported(const Geom& g, int c_in, int c_out, long long nnz_in) {
    return g.T <= 32 && (c_in == 32 || c_in == 64) && c_out >= 1 && c_out <= kQuadMaxCout && nnz_in > 0 &&
           nnz_in * (long long)c_in * 6 < (1ll << 31);
}

hipError_t launch_split_rows(const float* feats, long long n_imm, const long long* n_dev, long long n_cap, int c_in,
                             unsigned short* xs, hipStream_t s) {
    const int nch = (c_in + 31) / 32;
    long long blocks = (n_cap * nch * 4 + 255) / 256;
    if (blocks < 1) blocks = 1;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_split_rows, dim3((unsigned)blocks), dim3(256), 0, s, feats, n_imm, n_dev, n_cap, c_in, nch, xs);
    return hipGetLastError();
}

template <int NCH, int NB, int RPL, int ACC64, int K3>
static hipError_t launch_conv_split_t(const Geom& g, const unsigned long long* occ, const unsigned* occ_prefix,
                                      long long nnz_in, const unsigned short* xs, const unsigned short* ws,
                                      const float* bias, int c_out, int col0, int c_out_all, const int* tap_active,
                                      const unsigned* cand_lin, const int* cand_start, const int* tile_start,
                                      Counters* ctr, float* resp, int cus, hipStream_t s) {
    const size_t lds = (size_t)split_lds_words<RPL>(g.T, NCH) * 4 * kSplitWaves;
    hipError_t e = hipFuncSetAttribute((const void*)k_conv_quad_split<NCH, NB, RPL, ACC64, K3>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    int per_cu = 2;
    if ((size_t)per_cu * lds > 160 * 1024) per_cu = 1;
    const int grid = (cus * per_cu + kXcds - 1) / kXcds * kXcds;
    hipLaunchKernelGGL((k_conv_quad_split<NCH, NB, RPL, ACC64, K3>), dim3(grid), dim3(kSplitWaves * 64), lds, s, g, occ,
                       occ_prefix, nnz_in, xs, (const u32x4*)ws, bias, c_out, col0, c_out_all, tap_active, cand_lin,
                       cand_start, tile_start, ctr, resp);
    return hipGetLastError();
}

hipError_t launch_conv_split(const Geom& g, const unsigned long long* occ, const unsigned* occ_prefix, long long nnz_in,
                             const unsigned short* xs, int c_in, const unsigned short* ws, int c_out, const float* bias,
                             const int* tap_active, const unsigned* cand_lin, const int* cand_start,
                             const int* tile_start, Counters* ctr, float* resp, int cus, hipStream_t s) {
    const int nch = (c_in + 31) / 32;
    const bool k3 = g.K[0] == 3 && g.K[1] == 3 && g.K[2] == 3;
    for (int col0 = 0; col0 < c_out; col0 += 64) {
        const int cg = c_out - col0 < 64 ? c_out - col0 : 64;
        const unsigned short* ws_g = ws + (size_t)(col0 >> 6) * split_filter_elems(g.T, c_in);
        const float* bias_g = bias ? bias + col0 : nullptr;
        hipError_t e = hipErrorInvalidValue;
#define SCNN_SPLIT_ARGS g, occ, occ_prefix, nnz_in, xs, ws_g, bias_g, cg, col0, c_out, tap_active, cand_lin, cand_start, tile_start, ctr, resp, cus, s
#define SCNN_SPLIT_CASE(CH, RPL, ACC)                                                              \
    if (nch == CH) {                                                                               \
        if (cg > 32)                                                                               \
            e = k3 ? launch_conv_split_t<CH, 4, RPL, ACC, 1>(SCNN_SPLIT_ARGS)                      \
                   : launch_conv_split_t<CH, 4, RPL, ACC, 0>(SCNN_SPLIT_ARGS);                     \
        else                                                                                       \
            e = k3 ? launch_conv_split_t<CH, 2, 2, ACC, 1>(SCNN_SPLIT_ARGS)                        \
                   : launch_conv_split_t<CH, 2, 2, ACC, 0>(SCNN_SPLIT_ARGS);                       \
    }
        SCNN_SPLIT_CASE(1, SCNN_RPL, 0) SCNN_SPLIT_CASE(2, 1, 1)
#undef SCNN_SPLIT_CASE
#undef SCNN_SPLIT_ARGS
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace scnn
