// Whole layers of small samples: one workgroup computes one sample, from its rows to its output rows, in LDS.
//
// A layer on a 28 x 28 image is ten dependent launches of 3 to 7 us each on the general path, and a thousand such images
// are the same ten launches of 3 to 15 us: occupancy bits, candidates, responses, thresholds and pooled rows all go
// through memory between them.  A sample of up to two thousand sites fits the 160 KB of a compute unit, so here the steps
// are separated by barriers only: rows -> values per site and the taps that every site has (which also says what the
// candidate sites are) -> responses of the compacted candidates -> k-th strongest per channel, a wave each -> surviving
// rows -> pooled rows.  One sample's rows are the call's output; several samples leave theirs in a staging area with their
// counts, and a second launch (k_tiny_emit) adds up the counts before a sample and moves its rows.  Bound by latency: a
// workgroup of 1024 threads takes a 28 x 28 image in 13 us (no phase above 3), a thousand workgroups of 256, four to a
// compute unit, 32, and the second launch takes 6.  Calls, 1 -> 8 channels, pooled: one image 46.4 -> 13.7 us, 1024 images
// 101.0 -> 38.3.
// The sums are k_conv_valu_one's: fp64, taps in ascending order, channels in ascending order, one rounding.
#include "scnn_internal.h"

namespace scnn {

constexpr int kTinyTaps = 32;
constexpr int kTinyCin = 8, kTinyCout = 16;
constexpr long long kTinyMaxSites = 2048;  // 32 words of 64 sites; a wave holds a column in 32 registers
constexpr size_t kTinyLds = 152 * 1024;

// The workgroup's LDS.
struct TinyLayout {
    int np;        // sites, rounded up to whole words
    int nw;        // words
    int ws;        // doubles of a tap's weights (+ 2: lanes at different taps read different banks)
    size_t w, cand, keep, pos, raw, x, resp, lin, total;
};
__host__ __device__ inline TinyLayout tiny_layout(const Geom& g, int c_in, int c_out) {
    TinyLayout l;
    l.np = (int)g.Npad;
    l.nw = g.Wps;
    const int ocb = c_out <= 8 ? 8 : 16;
    l.ws = c_in * ocb + 2;
    size_t at = 0;
    l.w = at;    at += (size_t)g.T * l.ws * 8;
    l.cand = at; at += (size_t)l.nw * 8;
    l.keep = at; at += (size_t)l.nw * 8;   // by site: rows that survive the selection; then by pooled site
    l.pos = at;  at += (size_t)l.nw * 8;   // by position in the candidate list
    l.raw = at;  at += (size_t)l.np * 4;
    l.x = at;    at += (size_t)l.np * c_in * 4;
    l.resp = at; at += (size_t)l.np * c_out * 4;
    l.lin = at;  at += (size_t)l.np * 2;
    l.total = (at + 15) & ~(size_t)15;
    return l;
}

// Which layers.  One workgroup does all of a sample's work, so there is a line where the general path, whose launches use
// the whole chip, wins: in the products of a sample (rows x taps x channels, of which each costs 8 bytes of weights out of
// LDS) and in the entries that are selected from.  The launch lasts as long as its richest sample, and all that the host knows
// of that one is that it has no more rows than the call and the grid, so the line is drawn for the richest that the call can
// hold.  Calls, us, general path against this:
//   one sample: 28 x 28, 1 -> 8, a tenth occupied 32 / 14; 8 -> 16, half (452 k products) 39 / 38; 20 x 20, 8 -> 16, all (461 k)
//     35 / 33; 45 x 45, 4 -> 8, half (291 k) 34 / 36, all (583 k) 33 / 44; 1 -> 12, all (292 k) 36 / 41; 12^3, 8 -> 8, all (3 M) 37 / 113
//   eight, one occupied and the others empty: 28 x 28, 8 -> 8 (452 k) 37 / 36; 12^3, 8 -> 8 (3 M) 37 / 117; 45 x 45, 1 -> 8 (146 k)
//     34 / 36; 1 -> 12 (292 k) 36 / 47, a fifth of the one (58 k) 35 / 39 (the second launch is 6 us)
//   64, one occupied: 28 x 28, 8 -> 8 39 / 36; 45 x 45, 1 -> 8 37 / 36, 1 -> 12 41 / 47; 12^3, 8 -> 8 41 / 118
//   300, one occupied: 12^3, 4 -> 8 (1.5 M) 63 / 69, half of it (746 k) 60 / 51; 8^3, 8 -> 8 (885 k) 44 / 45; all half occupied,
//     28 x 28, 8 -> 8 (226 k on average) 68 / 57, 6^3, 8 -> 16, 1000 of them (373 k) 121 / 139
// Still on the slower side: layers of 16 k entries and more with some 100 k products and more, where the general path is up to
// 1.3 times as fast, for one sample and where one of 64 and more is rich.  Many samples are many rounds of workgroups, of which one without a row still loads
// the weights and passes the barriers.  Workgroups of 1024 threads (kTinyWide), 45 x 45, 1 -> 8, ten rows a sample, 1024 / 1536 /
// 4096 / 262144 samples 55 / 61 / 125 / 5046 against 44 / 63 / 160 / 11761; of 256 threads, 28 x 28, 1 -> 8, one row a sample,
// 4096 / 131072 / 262144 105 / 6988 / 3898 against 55 / 1565 / 3179, a row in one sample of fifty 80 / 6022 / 1506 against 46 /
// 1095 / 2244; 8 x 8, 8 -> 16 (1152 weights), 4096 / 16384 / 65536 69 / 171 / 575 against 58 / 186 / 667, one row a sample
// 117 / 408 / 1660 against 79 / 290 / 1111.
constexpr long long kTinyProducts = 400000, kTinyEntries = 24576;
constexpr size_t kTinyWide = 40 * 1024;  // LDS from which on four workgroups do not share a CU: all the threads it takes, then
bool layer_tiny_shape(const Geom& g, int c_in, int c_out) {
    return c_in <= kTinyCin && c_out <= kTinyCout && g.T <= kTinyTaps && g.N <= kTinyMaxSites &&
           g.N * c_out <= kTinyEntries && tiny_layout(g, c_in, c_out).total <= kTinyLds;
}
bool layer_tiny_pays(const Geom& g, int c_in, int c_out, long long rows) {
    const long long row = (long long)g.T * c_in * (c_out <= 8 ? 8 : 16);  // products
    const long long richest = (rows < g.N ? rows : g.N) * row;
    if (g.batch < 256)
        return richest <= kTinyProducts && (g.batch == 1 || g.batch >= 64 || richest + 15 * g.N * c_out <= 470000);
    if (richest > 750000 || rows * row > 300000ll * g.batch) return false;
    if (g.batch > 4096 && row > 1000 && rows < g.batch / 4) return false;
    return tiny_layout(g, c_in, c_out).total > kTinyWide ? g.batch <= 1024 : (long long)g.batch * g.Wps <= 1ll << 21;
}

// Exclusive sums of the popcounts of up to 64 words (lane i: the words before i); total: all of them.  (whole wave)
__device__ __forceinline__ unsigned word_sums(const unsigned long long* words, int n, unsigned& total) {
    const int lane = threadIdx.x & 63;
    const unsigned own = lane < n ? (unsigned)__popcll(words[lane]) : 0u;
    const unsigned inc = wave_inclusive_add(own);
    total = (unsigned)__builtin_amdgcn_readlane((int)inc, 63);
    return inc - own;
}

// A row's coordinates; is it on the grid?  Flags as the index build sets them (the row before it is looked at, too).
__device__ __forceinline__ bool tiny_row(const Geom& g, const int32_t* __restrict__ coords, long long r, int& b, int& c0, int& c1,
                                         int& c2, unsigned& flags) {
    const int stride = 1 + g.ndim;
    load_site(g, coords + r * stride, b, c0, c1, c2);
    int pb = -1, p0 = 0, p1 = 0, p2 = 0;
    if (r > 0) load_site(g, coords + (r - 1) * stride, pb, p0, p1, p2);
    if (!site_in_grid(g, b, c0, c1, c2)) {
        flags |= SCNN_FLAG_BAD_COORD;
        return false;
    }
    if (site_in_grid(g, pb, p0, p1, p2) && (pb > b || (pb == b && lin_of(g, p0, p1, p2) >= lin_of(g, c0, c1, c2))))
        flags |= SCNN_FLAG_UNSORTED;
    return true;
}

// (n <= 64 NU, column[0 .. last] are there)
template <int NU>
__device__ __forceinline__ void tiny_column(const float* column, int n, int last, int mode, long long k, unsigned& tau,
                                            unsigned& cut) {
    const int lane = threadIdx.x & 63;
    unsigned key[NU];
    constexpr int G = NU < 16 ? NU : 8;  // loads in flight together
#pragma unroll
    for (int u0 = 0; u0 < NU; u0 += G) {
        float x[G];
#pragma unroll
        for (int u = 0; u < G; ++u) x[u] = column[min((u0 + u) * 64 + lane, last)];
#pragma unroll
        for (int u = 0; u < G; ++u) key[u0 + u] = (u0 + u) * 64 + lane < n ? score_key(x[u], mode) : 0u;
        __builtin_amdgcn_sched_barrier(0);
    }
    unsigned n_nz;
    wave_threshold<NU>(key, k, n_nz, tau, cut);
}

template <int NT /* threads */, int CI /* input channels: 1, or 0 for any number */, int OCB /* output channels at most */>
__global__ __launch_bounds__(NT) void k_layer_tiny(Geom g, Geom gp, const int32_t* __restrict__ coords,
                                                   const float* __restrict__ feats, long long n_imm,
                                                   const long long* __restrict__ n_dev, int c_in_any,
                                                   const float* __restrict__ w, const float* __restrict__ bias, int c_out,
                                                   long long k, int mode, int relu, int pool, long long cand_cap,
                                                   unsigned* __restrict__ stage_lin, float* __restrict__ stage_feats,
                                                   long long stage_cap, TinySample* __restrict__ info,
                                                   int32_t* __restrict__ out_coords, float* __restrict__ out_feats,
                                                   long long out_capacity, long long* __restrict__ nnz_out) {
    extern __shared__ __align__(16) char s_mem[];
    __shared__ long long s_range[2];
    __shared__ unsigned s_act, s_flags;
    __shared__ unsigned s_tau[kTinyCout], s_cut[kTinyCout];
    __shared__ int s_off[kTinyTaps];
    constexpr int kWaves = NT / 64;
    __shared__ unsigned s_pre[64];  // candidates in the words before
    const int c_in = CI ? CI : c_in_any;
    const TinyLayout l = tiny_layout(g, c_in, c_out);
    double* s_w = (double*)(s_mem + l.w);
    unsigned long long* s_cand = (unsigned long long*)(s_mem + l.cand);
    unsigned long long* s_keep = (unsigned long long*)(s_mem + l.keep);
    unsigned long long* s_pos = (unsigned long long*)(s_mem + l.pos);
    unsigned* s_raw = (unsigned*)(s_mem + l.raw);
    float* s_x = (float*)(s_mem + l.x);
    float* s_resp = (float*)(s_mem + l.resp);
    unsigned short* s_lin = (unsigned short*)(s_mem + l.lin);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int np = l.np, nw = l.nw, T = g.T, K1 = g.K[1], K2 = g.K[2], b = (int)blockIdx.x;
    long long n = n_dev ? *n_dev : n_imm;
    n = n > n_imm ? n_imm : (n < 0 ? 0 : n);

    if (tid == 0) s_act = s_flags = 0u;
    if (tid < kTinyTaps) {
        const int t0 = tid / (K1 * K2), t1 = tid / K2 % K1, t2 = tid % K2;
        s_off[tid] = ((t0 - g.H[0]) * g.E[1] + (t1 - g.H[1])) * g.E[2] + (t2 - g.H[2]);
    }
    for (int i = tid; i < nw; i += NT) s_keep[i] = 0ull;
    for (int i = tid; i < np; i += NT) s_raw[i] = 0u;
    // the sample's rows (the caller's rows are sorted), a boundary per wave
    if (g.batch == 1) {
        if (tid == 0) s_range[0] = 0, s_range[1] = n;
    } else if (wave < 2) {
        const long long r = wave_first_row(coords, 1 + g.ndim, n, b + wave);
        if (lane == 0) s_range[wave] = r;
    }
    __syncthreads();
    unsigned act = 0;
    for (int i = NT - 1 - tid; i < T * c_in * OCB; i += NT) {  // (from the last thread down: the first have the rows)
        const int o = i % OCB, ti = i / OCB, t = ti / c_in;
        const float v = o < c_out ? w[(size_t)ti * c_out + o] : 0.0f;
        s_w[t * l.ws + (ti - t * c_in) * OCB + o] = (double)v;
        if (v != 0.0f) act |= 1u << t;
    }
    if (act) atomicOr(&s_act, act);
    // ---- values per site, and which of its taps every site has (bit t): a row tells the sites that look at it
    unsigned flags = 0;
    for (long long r = s_range[0] + tid; r < s_range[1]; r += NT) {
        int rb, c0, c1, c2;
        unsigned f = 0;
        const bool ok = tiny_row(g, coords, r, rb, c0, c1, c2, f);
        if (g.batch == 1) flags |= f;
        if (!ok || rb != b) continue;
        const int lin = (int)lin_of(g, c0, c1, c2);
        for (int c = 0; c < c_in; ++c) s_x[lin * c_in + c] = feats[(size_t)r * c_in + c];
        int t = 0;
        for (int t0 = 0; t0 < g.K[0]; ++t0)
            for (int t1 = 0; t1 < K1; ++t1) {
                const int q0 = c0 - (t0 - g.H[0]), q1 = c1 - (t1 - g.H[1]);
                const bool line = (unsigned)q0 < (unsigned)g.E[0] && (unsigned)q1 < (unsigned)g.E[1];
                const int site = (q0 * g.E[1] + q1) * g.E[2];
                for (int t2 = 0; t2 < K2; ++t2, ++t) {
                    const int q2 = c2 - (t2 - g.H[2]);
                    if (line && (unsigned)q2 < (unsigned)g.E[2]) atomicOr(&s_raw[site + q2], 1u << t);
                }
            }
    }
    // several samples: where the rows are not sorted the samples' ranges need not cover them, so they are checked by share
    if (g.batch > 1)
        for (long long r = n * b / g.batch + tid, end = n * (b + 1) / g.batch; r < end; r += NT) {
            int rb, c0, c1, c2;
            (void)tiny_row(g, coords, r, rb, c0, c1, c2, flags);
        }
    if (flags) atomicOr(&s_flags, flags);
    __syncthreads();

    // ---- the candidate sites: those with an active tap
    act = s_act;
    for (int s = tid; s < np; s += NT) {
        const unsigned raw = s_raw[s] & act;
        s_raw[s] = raw;
        const unsigned long long m = __ballot(raw != 0u);
        if (lane == 0) s_cand[s >> 6] = m;
    }
    __syncthreads();
    unsigned n_cand;
    const unsigned pre = word_sums(s_cand, nw, n_cand);
    if (wave == 0) s_pre[lane] = pre;
    const bool overflow = (long long)n_cand > cand_cap;  // (of this sample alone: of several, k_tiny_emit adds them up)
    for (int s = tid; s < np; s += NT) {  // (whole waves: np is a multiple of 64)
        const unsigned long long m = s_cand[s >> 6];
        const unsigned base = (unsigned)__builtin_amdgcn_readlane((int)pre, s >> 6);
        if ((m >> lane) & 1ull) s_lin[base + (unsigned)__popcll(m & ((1ull << lane) - 1ull))] = (unsigned short)s;
    }
    __syncthreads();

    // ---- responses: a thread per candidate walks the neighbours that it has
    for (int p = tid; p < (int)n_cand; p += NT) {
        const int lin = s_lin[p];
        double acc[OCB];
#pragma unroll
        for (int o = 0; o < OCB; ++o) acc[o] = 0.0;
        for (unsigned m = s_raw[lin]; m != 0u; m &= m - 1u) {
            const int t = __builtin_ctz(m);
            const float* x = s_x + (lin + s_off[t]) * c_in;
            const double2* wr = (const double2*)(s_w + t * l.ws);
            for (int ic = 0; ic < c_in; ++ic) {
                const double xd = (double)x[ic];
#pragma unroll
                for (int o = 0; o < OCB / 2; ++o) {
                    const double2 v = wr[ic * (OCB / 2) + o];
                    acc[2 * o] = fma(xd, v.x, acc[2 * o]);
                    acc[2 * o + 1] = fma(xd, v.y, acc[2 * o + 1]);
                }
            }
        }
#pragma unroll
        for (int o = 0; o < OCB; ++o) {
            if (o >= c_out) break;
            float v = (float)acc[o];
            if (bias && v != 0.0f) v += bias[o];
            s_resp[o * np + p] = v;
        }
    }
    __syncthreads();

    // ---- the k-th strongest response of every channel
    for (int c = wave; c < c_out; c += kWaves) {
        const float* column = s_resp + c * np;
        const int regs = ((int)n_cand + 63) >> 6;
        unsigned tau, cut;
        if (regs <= 4) tiny_column<4>(column, (int)n_cand, np - 1, mode, k, tau, cut);
        else if (regs <= 6) tiny_column<6>(column, (int)n_cand, np - 1, mode, k, tau, cut);
        else if (regs <= 10) tiny_column<10>(column, (int)n_cand, np - 1, mode, k, tau, cut);
        else if (regs <= 16) tiny_column<16>(column, (int)n_cand, np - 1, mode, k, tau, cut);
        else tiny_column<32>(column, (int)n_cand, np - 1, mode, k, tau, cut);
        if (lane == 0) {
            s_tau[c] = tau;
            s_cut[c] = cut;
        }
    }
    __syncthreads();

    // ---- what survives: zeros in the place of what does not, the rows that keep an entry by position and by site
    const int ncp = ((int)n_cand + 63) & ~63;
    for (int p = tid; p < ncp; p += NT) {
        bool any = false;
        if (p < (int)n_cand) {
            float x[OCB];
#pragma unroll
            for (int c = 0; c < OCB; ++c) x[c] = c < c_out ? s_resp[c * np + p] : 0.0f;
#pragma unroll
            for (int c = 0; c < OCB; ++c) {
                if (c >= c_out) break;
                const unsigned tau = s_tau[c];
                bool kept = score_key(x[c], mode) > ((unsigned)p <= s_cut[c] ? tau - (tau != 0u ? 1u : 0u) : tau);
                if (relu) kept = kept && x[c] > 0.0f;
                if (!kept) s_resp[c * np + p] = 0.0f;
                any |= kept;
            }
        }
        const unsigned long long m = __ballot(any);
        if (lane == 0) s_pos[p >> 6] = m;
        if (pool && any) {
            const int lin = s_lin[p];
            atomicOr(&s_keep[lin >> 6], 1ull << (lin & 63));
        }
    }
    __syncthreads();

    // ---- output rows
    // Several samples: a sample has at most as many rows as its input rows reach sites and as there are sites, so the samples
    // before it take at most min(their rows * taps, their sites) of the staging area.  (Rows that are not sorted can make the
    // ranges overlap: the room keeps the writes inside.)
    const long long at_rows = s_range[0] * T, at_sites = (long long)b * g.N;
    const long long first = g.batch == 1 ? 0 : (at_rows < at_sites ? at_rows : at_sites);
    const long long room = g.batch == 1 ? (overflow ? 0 : out_capacity) : stage_cap - first;
    float* const dst = g.batch == 1 ? out_feats : stage_feats + first * c_out;
    const bool vec = (c_out & 3) == 0 && ((size_t)dst & 15) == 0;
    // row o of the sample: site lin of the output grid go, v its channels
    auto write = [&](const Geom& go, unsigned lin, unsigned o, const float (&v)[OCB]) __attribute__((always_inline)) {
        if ((long long)o >= room) return;
        if (g.batch == 1) {
            int c0, c1, c2;
            site_of(go, lin, c0, c1, c2);
            store_site(go, out_coords + (size_t)o * (1 + go.ndim), b, c0, c1, c2);
        } else {
            stage_lin[first + o] = lin;
        }
        float* row = dst + (size_t)o * c_out;
        if (vec) {
#pragma unroll
            for (int c = 0; c < OCB; c += 4)
                if (c < c_out) *(float4*)(row + c) = make_float4(v[c], v[c + 1], v[c + 2], v[c + 3]);
        } else {
#pragma unroll
            for (int c = 0; c < OCB; ++c)
                if (c < c_out) row[c] = v[c];
        }
    };
    unsigned rows;
    if (!pool) {
        const unsigned before = word_sums(s_pos, ncp >> 6, rows);
        for (int p = tid; p < ncp; p += NT) {
            const unsigned long long m = s_pos[p >> 6];
            const unsigned base = (unsigned)__builtin_amdgcn_readlane((int)before, p >> 6);
            if (!((m >> lane) & 1ull)) continue;
            float v[OCB];
#pragma unroll
            for (int c = 0; c < OCB; ++c) v[c] = c < c_out ? s_resp[c * np + p] : 0.0f;
            write(g, s_lin[p], base + (unsigned)__popcll(m & ((1ull << lane) - 1ull)), v);
        }
    } else {
        // a pooled site takes, per channel, the largest of the entries that its up to eight sites keep
        const int npp = (int)gp.Npad;
        // its sites on the grid that keep a row: at(site, keeps a row); the first axis has one layer in 2-D
        const int layers = g.E[0] > 1 ? 8 : 4;
        auto children = [&](int s, auto at) __attribute__((always_inline)) {
            int p0, p1, p2;
            site_of(gp, (unsigned)s, p0, p1, p2);
            const int lin0 = (2 * p0 * g.E[1] + 2 * p1) * g.E[2] + 2 * p2;
            const bool two0 = 2 * p0 + 1 < g.E[0], two1 = 2 * p1 + 1 < g.E[1], two2 = 2 * p2 + 1 < g.E[2];
#pragma unroll
            for (int d = 0; d < 8; ++d) {
                if (d >= layers) break;
                const bool on = (!(d & 4) || two0) && (!(d & 2) || two1) && (!(d & 1) || two2);
                const int lin = on ? lin0 + ((d >> 2) * g.E[1] + ((d >> 1) & 1)) * g.E[2] + (d & 1) : lin0;
                at(lin, on && ((s_keep[lin >> 6] >> (lin & 63)) & 1ull));
            }
        };
        for (int s = tid; s < npp; s += NT) {
            bool any = false;
            if (s < (int)gp.N) children(s, [&](int, bool has) { any |= has; });
            const unsigned long long m = __ballot(any);
            if (lane == 0) s_pos[s >> 6] = m;
        }
        __syncthreads();
        const unsigned before = word_sums(s_pos, npp >> 6, rows);
        for (int s = tid; s < npp; s += NT) {
            const unsigned long long m = s_pos[s >> 6];
            const unsigned base = (unsigned)__builtin_amdgcn_readlane((int)before, s >> 6);
            if (!((m >> lane) & 1ull)) continue;
            float best[OCB];  // (0: none yet; an entry is not 0)
#pragma unroll
            for (int c = 0; c < OCB; ++c) best[c] = 0.0f;
            children(s, [&](int lin, bool has) {
                const int pos = (int)(s_pre[lin >> 6] + (unsigned)__popcll(s_cand[lin >> 6] & ((1ull << (lin & 63)) - 1ull)));
#pragma unroll
                for (int c = 0; c < OCB; ++c) {
                    const float v = has && c < c_out ? s_resp[c * np + pos] : 0.0f;
                    if (v != 0.0f) best[c] = best[c] != 0.0f ? fmaxf(best[c], v) : v;
                }
                if constexpr (OCB > 8) __builtin_amdgcn_sched_barrier(0);  // (eight children's would not fit the registers)
            });
            write(gp, (unsigned)s, base + (unsigned)__popcll(m & ((1ull << lane) - 1ull)), best);
        }
    }
    if (tid != 0) return;
    if (g.batch > 1) {
        info[b] = TinySample{(long long)rows < room ? (int)rows : (int)room, (int)n_cand, s_flags, (unsigned)first};
        return;
    }
    unsigned f = s_flags;
    if (overflow) {
        f |= SCNN_FLAG_CAND_OVERFLOW;
        rows = 0;
    }
    if ((long long)rows > out_capacity) f |= SCNN_FLAG_OUT_OVERFLOW;
    nnz_out[0] = rows;
    nnz_out[1] = n_cand;
    nnz_out[2] = f;
    nnz_out[3] = 0;
}

// Second launch, several samples: a workgroup owns consecutive samples, adds up the rows of those before them and moves its
// own from the staging area to their place; the last one writes the result counters.
constexpr int kTinyEmitBlocks = 2048;
__global__ __launch_bounds__(256) void k_tiny_emit(Geom go, int channels, const TinySample* __restrict__ info,
                                                   const unsigned* __restrict__ stage_lin,
                                                   const float* __restrict__ stage_feats, long long cand_cap,
                                                   int32_t* __restrict__ out_coords, float* __restrict__ out_feats,
                                                   long long out_capacity, long long* __restrict__ nnz_out) {
    __shared__ unsigned long long s_rows[4], s_cands[4];
    __shared__ unsigned s_flags[4];
    const int per = (go.batch + (int)gridDim.x - 1) / (int)gridDim.x;
    const int first = (int)blockIdx.x * per, last = first + per < go.batch ? first + per : go.batch;
    const bool counters = blockIdx.x == 0;
    if (first >= last) return;
    unsigned long long before = 0, cands = 0, all = 0;
    unsigned flags = 0;
    for (int i = threadIdx.x; i < go.batch; i += 256) {
        const TinySample t = info[i];
        cands += (unsigned)t.cands;
        all += (unsigned)t.rows;
        flags |= t.flags;
        if (i < first) before += (unsigned)t.rows;
    }
    if (counters) before = all;  // (the first workgroup has no rows before its own: it adds up all of them)
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        before += __shfl_xor(before, d, 64);
        cands += __shfl_xor(cands, d, 64);
        flags |= (unsigned)__shfl_xor((int)flags, d, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        s_rows[threadIdx.x >> 6] = before;
        s_cands[threadIdx.x >> 6] = cands;
        s_flags[threadIdx.x >> 6] = flags;
    }
    __syncthreads();
    long long base = (long long)(s_rows[0] + s_rows[1] + s_rows[2] + s_rows[3]);
    const long long n_cand = (long long)(s_cands[0] + s_cands[1] + s_cands[2] + s_cands[3]);
    const bool overflow = n_cand > cand_cap;
    if (counters) {
        if (threadIdx.x == 0) {
            unsigned f = s_flags[0] | s_flags[1] | s_flags[2] | s_flags[3];
            const long long rows = overflow ? 0 : base;
            if (overflow) f |= SCNN_FLAG_CAND_OVERFLOW;
            if (rows > out_capacity) f |= SCNN_FLAG_OUT_OVERFLOW;
            nnz_out[0] = rows;
            nnz_out[1] = n_cand;
            nnz_out[2] = f;
            nnz_out[3] = 0;
        }
        base = 0;
    }
    if (overflow) return;
    const bool vec = (channels & 3) == 0 && ((size_t)out_feats & 15) == 0;
    for (int b = first; b < last; ++b) {
        const int rows = info[b].rows;
        const size_t at = info[b].first;
        const int room = base + rows <= out_capacity ? rows : (base < out_capacity ? (int)(out_capacity - base) : 0);
        for (int r = threadIdx.x; r < room; r += 256) {
            int c0, c1, c2;
            site_of(go, stage_lin[at + r], c0, c1, c2);
            store_site(go, out_coords + (base + r) * (1 + go.ndim), b, c0, c1, c2);
        }
        const float* src = stage_feats + at * channels;
        float* dst = out_feats + base * channels;
        if (vec) {
            for (int i = threadIdx.x; i < room * channels / 4; i += 256) ((float4*)dst)[i] = ((const float4*)src)[i];
        } else {
            for (int i = threadIdx.x; i < room * channels; i += 256) dst[i] = src[i];
        }
        base += rows;
    }
}

template <int NT, int CI, int OCB, typename... Args>
static hipError_t launch_tiny_t(const Geom& g, size_t lds, hipStream_t s, Args... args) {
    if (lds > 64 * 1024) {  // (the same for every layer: another thread's launch may lie between this and ours)
        hipError_t e = hipFuncSetAttribute((const void*)k_layer_tiny<NT, CI, OCB>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)kTinyLds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_layer_tiny<NT, CI, OCB>), dim3((unsigned)g.batch), dim3(NT), lds, s, g, args...);
    return hipGetLastError();
}

hipError_t launch_layer_tiny(const Geom& g, const Geom& gp, const int32_t* coords, const float* feats, long long n_imm,
                             const long long* n_dev, int c_in, const float* w, const float* bias, int c_out, long long k,
                             int mode, int relu, int pool, long long cand_cap, long long stage_cap, unsigned* stage_lin,
                             float* stage_feats, TinySample* info, int32_t* out_coords, float* out_feats, long long out_capacity,
                             long long* nnz_out, hipStream_t s) {
    const int ocb = c_out <= 8 ? 8 : 16;
    const size_t lds = tiny_layout(g, c_in, c_out).total;
    // Few samples leave most of the chip idle and are done when their one workgroup is: all the waves a unit takes.
    const bool wide = g.batch <= device_cu_count() || lds > kTinyWide;
    hipError_t e;
#define SCNN_TINY(NT_, CI_, OCB_)                                                                                        \
    e = launch_tiny_t<NT_, CI_, OCB_>(g, lds, s, gp, coords, feats, n_imm, n_dev, c_in, w, bias, c_out, k, mode, relu, pool, \
                                      cand_cap, stage_lin, stage_feats, stage_cap, info, out_coords, out_feats,          \
                                      out_capacity, nnz_out)
#define SCNN_TINY_OCB(NT_, CI_)                   \
    do {                                          \
        if (ocb == 8) SCNN_TINY(NT_, CI_, 8);     \
        else SCNN_TINY(NT_, CI_, 16);             \
    } while (0)
    if (wide) {
        if (c_in == 1) SCNN_TINY_OCB(1024, 1);
        else SCNN_TINY_OCB(1024, 0);
    } else {
        if (c_in == 1) SCNN_TINY_OCB(256, 1);
        else SCNN_TINY_OCB(256, 0);
    }
#undef SCNN_TINY_OCB
#undef SCNN_TINY
    if (e != hipSuccess || g.batch == 1) return e;
    const Geom& go = pool ? gp : g;
    const unsigned blocks = (unsigned)(g.batch < kTinyEmitBlocks ? g.batch : kTinyEmitBlocks);
    hipLaunchKernelGGL(k_tiny_emit, dim3(blocks), dim3(256), 0, s, go, c_out, info, stage_lin, stage_feats, cand_cap,
                       out_coords, out_feats, out_capacity, nnz_out);
    return hipGetLastError();
}

}  // namespace scnn
