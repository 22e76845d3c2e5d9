// The attention step (Sec. 3.2; Algorithm 1 steps 13, 15-17): per (sample,
// output channel) keep the k strongest non-zero responses, then compact the
// surviving sites into sorted output rows.
//
// Selection = radix select on an order-preserving 32-bit key of the score, on a
// small part of each column.  A workgroup per column first reads a sample of
// the column (every S-th tile) and brackets the k-th strongest key between two
// of the sample's order statistics.  One pass over the response matrix then
// counts, per column, the entries above the bracket, copies the few percent
// inside it (value and position in the column) to a side buffer, and notes
// which rows hold an entry above the bracket.  A workgroup per column settles
// the rest on the side buffer: the exact k-th largest key tau and how many of
// the entries equal to it, q, still fit.  An entry survives iff  key > tau, or
// key == tau and it is among the q equal entries of lowest lin; candidate sites
// are stored in ascending lin, so "lowest lin" is "smallest position", and the
// q-th smallest position among the equal entries is the cut.  Both come from
// digit passes until at most 64 entries are left, which one wave ranks by
// (key, position).
// A bracket that turns out not to hold the k-th entry costs time, never
// exactness: the column is then settled from the response matrix itself.
// The response matrix is read twice in full (the classifying pass, and the
// final mask + compaction + write) and once in a sample of 1/S.  Columns short
// enough for one workgroup's registers are selected in a single launch.
//
// Compaction: where the selection has noted the rows (layers of 17 to 64
// channels with columns of more than one workgroup's), the rows that survive in
// every tile are known before the last pass, a scan gives each tile its first
// output row, and the write pass streams with no ordering between tiles.  Other
// layers of at most 32 channels count and write in two launches from some size
// on (narrow_pair_tiles), and so do wider ones from kCountedTiles on, from
// kCountedPlainTiles on where nothing is selected.  Elsewhere tiles are taken
// in order and a tile learns its first output row by looking back at its
// predecessors.
#include <type_traits>

#include "scnn_internal.h"

namespace scnn {

// ------------------------------------------------------------------ layout conversion (standalone entry)
// Sample ranges of a sorted row list: cand_start[b] = first row of sample b.
constexpr int kBoundsByWave = 16;
__global__ __launch_bounds__(256) void k_rows_sample_bounds(Geom g, const int32_t* __restrict__ coords,
                                                            long long rows, int* __restrict__ cand_start,
                                                            int* __restrict__ tile_start, Counters* ctr) {
    const int stride = 1 + g.ndim;
    if (g.batch <= kBoundsByWave) {
        // few samples: a wave per boundary, 64 probes at a time (a thread's binary search is 18 dependent loads for
        // 154 k rows: 10.2 us a launch, this 5.0); the four waves take the boundaries in turn, three loads each, so that
        // the threads are faster again from some twenty samples on (32 samples of 128 k rows: call 51 against 55)
        const int lane = threadIdx.x & 63;
        for (int b = threadIdx.x >> 6; b <= g.batch; b += 4) {
            const long long lo = wave_first_row(coords, stride, rows, b);
            if (lane == 0) cand_start[b] = (int)lo;
        }
    } else
    for (int b = threadIdx.x; b <= g.batch; b += blockDim.x) {
        long long lo = 0, hi = rows;  // first row with sample index >= b
        while (lo < hi) {
            long long mid = (lo + hi) >> 1;
            if (coords[mid * stride] < b) lo = mid + 1; else hi = mid;
        }
        cand_start[b] = (int)lo;
    }
    __syncthreads();
    __shared__ unsigned s_wave[4];
    const int n_tiles = sample_ranges_256(g.batch, cand_start, tile_start, nullptr, s_wave);
    if (threadIdx.x == 0) {
        ctr->n_tiles = n_tiles;
        ctr->n_cand = rows;
    }
}

hipError_t launch_rows_sample_bounds(const Geom& g, const int32_t* coords, long long rows, int* cand_start,
                                     int* tile_start, Counters* ctr, hipStream_t s) {
    hipLaunchKernelGGL(k_rows_sample_bounds, dim3(1), dim3(256), 0, s, g, coords, rows, cand_start, tile_start,
                       ctr);
    return hipGetLastError();
}

// Site-major rows -> planar tiles, through LDS so that both sides coalesce.
__global__ __launch_bounds__(256) void k_rows_to_planar(Geom g, const int32_t* __restrict__ coords,
                                                        const float* __restrict__ feats, int channels,
                                                        const int* __restrict__ cand_start,
                                                        const int* __restrict__ tile_start,
                                                        const Counters* __restrict__ ctr,
                                                        unsigned* __restrict__ cand_lin, float* __restrict__ resp) {
    __shared__ float s_t[kTileRows][65];
    const int n_tiles = (int)ctr->n_tiles;
    const int stride = 1 + g.ndim;
    const bool vec = channels % 4 == 0 && ((uintptr_t)feats & 15) == 0;
    for (int tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const int b = sample_of_tile(tile_start, g.batch, tile);
        const int first = cand_start[b] + (tile - tile_start[b]) * kTileRows;
        int nrows = cand_start[b + 1] - first;
        if (nrows > kTileRows) nrows = kTileRows;
        if (threadIdx.x < nrows) {
            int bb, c0, c1, c2;
            load_site(g, coords + (size_t)(first + threadIdx.x) * stride, bb, c0, c1, c2);
            unsigned lin = 0;
            if (site_in_grid(g, bb, c0, c1, c2)) lin = (unsigned)lin_of(g, c0, c1, c2);
            cand_lin[first + threadIdx.x] = lin;
        }
        for (int cc = 0; cc < channels; cc += 64) {
            const int cw = (channels - cc) < 64 ? (channels - cc) : 64;
            __syncthreads();
            // (all of a thread's loads in flight together: one after the other, they were the kernel's whole time)
            if (vec) {
                float4 v[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const int r = (k * 256 + (int)threadIdx.x) >> 4, c = (threadIdx.x & 15) * 4;
                    v[k] = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (r < nrows && c < cw) v[k] = *(const float4*)(feats + (size_t)(first + r) * channels + cc + c);
                }
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    float* t = &s_t[(k * 256 + (int)threadIdx.x) >> 4][(threadIdx.x & 15) * 4];
                    t[0] = v[k].x; t[1] = v[k].y; t[2] = v[k].z; t[3] = v[k].w;
                }
            } else {
                float v[32];
#pragma unroll
                for (int k = 0; k < 32; ++k) {
                    const int r = k * 4 + (threadIdx.x >> 6), c = threadIdx.x & 63;
                    v[k] = r < nrows && c < cw ? feats[(size_t)(first + r) * channels + cc + c] : 0.0f;
                }
#pragma unroll
                for (int k = 0; k < 32; ++k) s_t[k * 4 + (threadIdx.x >> 6)][threadIdx.x & 63] = v[k];
            }
            __syncthreads();
            float* out = resp + ((size_t)tile * channels + cc) * kTileRows;
#pragma unroll 8
            for (int k = 0; k < 32; ++k) {
                const int c = k * 2 + (threadIdx.x >> 7), r = threadIdx.x & 127;
                if (c < cw) out[c * kTileRows + r] = s_t[r][c];
            }
        }
    }
}

hipError_t launch_rows_to_planar(const Geom& g, const int32_t* coords, const float* feats, int channels,
                                 const int* cand_start, const int* tile_start, const Counters* ctr,
                                 long long tiles_cap, unsigned* cand_lin, float* resp, hipStream_t s) {
    long long blocks = tiles_cap < 1 ? 1 : (tiles_cap > 4096 ? 4096 : tiles_cap);
    hipLaunchKernelGGL(k_rows_to_planar, dim3((unsigned)blocks), dim3(256), 0, s, g, coords, feats, channels,
                       cand_start, tile_start, ctr, cand_lin, resp);
    return hipGetLastError();
}

// ------------------------------------------------------------------ radix select

// Rank search in a 2048-bin histogram held in LDS.  descending: find the bin holding the kk-th entry counted from
// the top bin; else from the bottom bin.  Returns the bin and the number of entries strictly before it in that
// order.  1 <= kk <= total must hold.  Contains two __syncthreads(); s_res is two shared words that the next call
// must not share (callers alternate between two pairs): the result is read after the last barrier.
constexpr int kPickThreads = 1024, kPickWaves = kPickThreads / 64;  // a thread owns two bins
template <int RANKS /* searched for together: s_res is two words for each */>
__device__ inline void block_pick(const unsigned* s_h /* 8-byte aligned */, const long long (&ranks)[RANKS], bool descending,
                                  unsigned* s_wave /* [kPickWaves], 16-byte aligned */, int* s_res, int (&bin_out)[RANKS],
                                  unsigned (&before_out)[RANKS]) {
    static_assert(kHistBins == 2 * kPickThreads, "two bins a thread");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint2 c = ((const uint2*)s_h)[threadIdx.x];
    const unsigned local = c.x + c.y, inc = wave_inclusive_add(local);
    if (lane == 63) s_wave[wave] = inc;
    __syncthreads();
    unsigned base = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kPickWaves; ++w) {
        const unsigned x = s_wave[w];
        base += w < wave ? x : 0u;
        total += x;
    }
    const unsigned excl = base + inc - local;
    const unsigned before = descending ? total - excl - local : excl;
#pragma unroll
    for (int i = 0; i < RANKS; ++i) {
        const long long kk = ranks[i];
        if ((long long)before < kk && kk <= (long long)before + (long long)local) {
            const unsigned first = descending ? c.y : c.x;
            const bool second = kk > (long long)before + (long long)first;
            s_res[2 * i] = 2 * (int)threadIdx.x + (descending != second ? 1 : 0);
            s_res[2 * i + 1] = (int)(before + (second ? first : 0u));
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RANKS; ++i) {
        bin_out[i] = s_res[2 * i];
        before_out[i] = (unsigned)s_res[2 * i + 1];
    }
}
__device__ inline void block_pick(const unsigned* s_h, long long kk, bool descending, unsigned* s_wave, int* s_res, int& bin_out,
                                  unsigned& before_out) {
    const long long ranks[1] = {kk};
    int bin[1];
    unsigned before[1];
    block_pick<1>(s_h, ranks, descending, s_wave, s_res, bin, before);
    bin_out = bin[0];
    before_out = before[0];
}

// First launch: a bracket [tau_lo, tau_hi] around the k-th strongest key of every column, from a sample of the
// column.  One workgroup per column reads every S-th tile of it (at most kBracketTiles tiles, whole tiles: 512
// contiguous bytes per channel), keeps the keys in registers and looks up, by two radix digits (22 key bits), the
// sample's keys at the ranks  r -+ delta,  r = k * (sample slots / column slots)  being where the k-th strongest
// entry of the column is expected in the sample (empty slots rank last, as key 0).  delta = 8 standard deviations
// of a uniformly drawn sample's rank plus half a percent of the sample: tiles are pieces of space, not independent
// draws, hence the margin (6 deviations plus a quarter percent missed on three layers of the 128^3 network and on
// the r = 128 layer).  Nothing depends on the bracket being right: the second launch counts what lies above it and
// the third one checks that the k-th entry fell inside, and settles the column from the response matrix itself when
// it did not.
constexpr int kBracketThreads = 1024;
constexpr int kBracketBin = 16;
constexpr int kBracketPerThread = 16;
constexpr int kBracketTiles = kBracketThreads * kBracketPerThread / kTileRows;  // 128

__global__ __launch_bounds__(kBracketThreads) void k_bracket(int mode, int channels,
                                                             const int* __restrict__ tile_start,
                                                             const float* __restrict__ resp, long long k,
                                                             ColState* __restrict__ cols) {
    __shared__ __align__(16) unsigned s_h[kHistBins], s_h2[kHistBins];
    __shared__ __align__(16) unsigned s_wave[kPickWaves];
    __shared__ int s_res[4];
    __shared__ unsigned s_total;
    __shared__ unsigned s_range[2];
    auto clamp_add = [](unsigned a, unsigned c) { return a + c < a ? 0xffffffffu : a + c; };
    const int col = blockIdx.x;
    const int b = col / channels, oc = col - b * channels;
    const int t0 = tile_start[b], t1 = tile_start[b + 1];
    const int T = t1 - t0;
    ColState st;
    st.tau = 0; st.cut = 0xffffffffu; st.tau_lo = 1u; st.tau_hi = 0u; st.n_nz = 0; st.n_above = 0;
    st.side_fill = 0; st.done = 0;
    st.side_off = ((unsigned long long)t0 * channels + (unsigned long long)oc * T) * kTileRows;
    if (k <= 0 || T == 0) {
        st.done = 1;
        if (k <= 0) st.tau = 0xffffffffu;  // no key is stronger: nothing survives
        if (threadIdx.x == 0) cols[col] = st;
        return;
    }
    const int S = (T + kBracketTiles - 1) / kBracketTiles;  // every S-th tile
    const int ns_tiles = (T + S - 1) / S;
    const unsigned m_s = (unsigned)ns_tiles * kTileRows;
    if (threadIdx.x == 0) {
        s_total = 0;
        s_range[0] = 0xffffffffu;
        s_range[1] = 0u;
    }
    // entry u of the thread is row threadIdx.x % 128 of sampled tile 8 u + threadIdx.x / 128, the same in all of a wave; past
    // the sample the last tile is read again and dropped, so that all loads are in flight together
    unsigned key[kBracketPerThread];
    unsigned mine = 0;
    {
        const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        float x[kBracketPerThread];
#pragma unroll
        for (int u = 0; u < kBracketPerThread; ++u) {
            const int at = u * (kBracketThreads / kTileRows) + (wave >> 1);
            const float* tile = resp + ((size_t)(t0 + (at < ns_tiles ? at : ns_tiles - 1) * S) * channels + oc) * kTileRows;
            x[u] = tile[threadIdx.x & (kTileRows - 1)];
        }
#pragma unroll
        for (int u = 0; u < kBracketPerThread; ++u) {
            key[u] = u * (kBracketThreads / kTileRows) + (wave >> 1) < ns_tiles ? score_key(x[u], mode) : 0u;
            mine += key[u] != 0u ? 1u : 0u;
        }
    }
    // the sample's entries, and the range of their keys
    unsigned kmin = 0xffffffffu, kmax = 0u;
#pragma unroll
    for (int u = 0; u < kBracketPerThread; ++u) {
        if (key[u] != 0u) {
            kmin = key[u] < kmin ? key[u] : kmin;
            kmax = key[u] > kmax ? key[u] : kmax;
        }
    }
    for (int i = threadIdx.x; i < kHistBins; i += kBracketThreads) s_h[i] = 0;
    __syncthreads();  // (s_total and the range words are set up)
    mine = wave_add(mine);
    kmin = wave_min(kmin);
    kmax = wave_max(kmax);
    if ((threadIdx.x & 63) == 0 && mine) {
        atomicAdd(&s_total, mine);
        atomicMin(&s_range[0], kmin);
        atomicMax(&s_range[1], kmax);
    }
    __syncthreads();
    const long long nz = (long long)s_total;
    kmin = s_range[0];
    kmax = s_range[1];
    const double r = (double)k * (double)m_s / ((double)T * kTileRows);
    const double frac = r / (double)m_s;
    double delta = 0.0;  // (a sample of every tile is the column: the ranks are exact)
    if (S > 1) delta = 8.0 * sqrt(r * (frac < 1.0 ? 1.0 - frac : 0.0)) + 0.005 * (double)m_s + 16.0;
    const double r_up = floor(r - delta), r_dn = ceil(r + delta);
    // The sample's keys at ranks r_up and r_dn (1 = strongest), cut down to two digits of 11 bits.  The digits are
    // taken from key - kmin: the leading bits of the keys themselves are the same for most of a column (sign, high
    // exponent bits), and a histogram whose entries fall into a dozen bins is a queue at those LDS words.  Past the
    // sample's entries on the strong side nothing is above the bracket; past them on the weak side every entry is in
    // it or above it.
    const bool want_up = r_up >= 1.0 && (long long)r_up <= nz, want_dn = r_dn >= 1.0 && r_dn <= (double)nz;  // (uniform)
    const long long rank_up = want_up ? (long long)r_up : 1, rank_dn = want_dn ? (long long)r_dn : 1;
    const unsigned span = nz > 0 ? kmax - kmin : 0u;
    const int nb = span ? 32 - __clz(span) : 1;  // bits of key - kmin
    const int sh1 = nb > 11 ? nb - 11 : 0;       // first digit: bits [sh1, nb)
    const int sh2 = sh1 > 11 ? sh1 - 11 : 0;     // second digit: bits [sh2, sh1)
    const unsigned mask2 = (1u << (sh1 - sh2)) - 1u;
#pragma unroll
    for (int u = 0; u < kBracketPerThread; ++u)
        if (key[u] != 0u) atomicAdd(&s_h[(key[u] - kmin) >> sh1], 1u);
    __syncthreads();
    int bin[2] = {0, 0}, sub[2] = {0, 0};  // of the upper end and of the lower
    unsigned before[2] = {0, 0};
    long long rank[2] = {rank_up, rank_dn};
    int sh = sh1;  // bits that the digits taken leave open
    if (nz > 0) block_pick<2>(s_h, rank, true, s_wave, s_res, bin, before);
    // a second digit where an end's bin holds more entries than widen the bracket by an eighth (it is 2.9 us of this kernel)
    const unsigned few = (unsigned)kBracketBin + (unsigned)(delta * 0.25);
    if (sh1 > 0 && (s_h[bin[0]] > few || s_h[bin[1]] > few)) {  // (uniform)
        rank[0] -= (long long)before[0];
        rank[1] -= (long long)before[1];
        __syncthreads();  // (the bins' counts have been read)
        for (int i = threadIdx.x; i < kHistBins; i += kBracketThreads) {
            s_h[i] = 0;
            s_h2[i] = 0;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kBracketPerThread; ++u) {
            if (key[u] == 0u) continue;
            const unsigned d = key[u] - kmin;
            if ((int)(d >> sh1) == bin[0]) atomicAdd(&s_h[(d >> sh2) & mask2], 1u);
            if ((int)(d >> sh1) == bin[1]) atomicAdd(&s_h2[(d >> sh2) & mask2], 1u);
        }
        __syncthreads();
        block_pick(s_h, rank[0], true, s_wave, s_res, sub[0], before[0]);
        block_pick(s_h2, rank[1], true, s_wave, s_res + 2, sub[1], before[1]);
        sh = sh2;
    }
    st.tau_hi = 0xffffffffu;  // rank < 1: nothing is above
    if (r_up >= 1.0)  // (the upper end of the bin)
        st.tau_hi =
            want_up ? clamp_add(kmin, ((unsigned)bin[0] << sh1) | ((unsigned)sub[0] << sh2) | ((1u << sh) - 1u)) : 0u;
    if (want_dn) {
        const unsigned lo = kmin + (((unsigned)bin[1] << sh1) | ((unsigned)sub[1] << sh2));
        st.tau_lo = lo ? lo : 1u;
    }
    if (threadIdx.x == 0) cols[col] = st;
}

// Second launch, grid = (sample x group of kClassifyWaves channels, slices); a wave per channel, the waves of a
// workgroup on the same tiles (adjacent channels of a tile are adjacent in memory).  Counts the column's entries and
// those above the bracket, copies the entries inside it (value and position in the column) to the side buffer, and,
// when row_plane is given, records which rows hold an entry above the bracket -- those survive whatever the exact
// threshold turns out to be -- in the channel's own plane of row marks, two 64-bit words per tile, which
// k_combine_marks merges.  Waves share nothing but the cursor of their column's side-buffer entries and never wait
// for one another.  (Marks kept in one shared plane cost 40 us of device-scope atomics on the r = 128 layer, whose
// every tile half would be updated by every channel.)  The loop is bound by
// instruction issue, hence the float compares on ballots, the counts in scalar registers and the marks gathered
// with v_writelane.
// With the score s(x) = |x| or x: the value t such that, for an entry x (non-zero, not a NaN),
// score_key(x) > key  <=>  s(x) > t  and  score_key(x) >= key  <=>  s(x) >= t:  the float whose key `key` is, or, for the
// keys below every float's (signed order: 0 .. 0x007fffff), minus infinity.  Key 0xffffffff gives a NaN: no score
// compares above it.
__device__ inline float score_bound(unsigned key, int mode) {
    if (mode == SCNN_TOPK_ABS) return __uint_as_float(key);  // (keys are the bit patterns of |x|; key 0 is 0.0)
    if (key >= 0x80000000u) return __uint_as_float(key & 0x7fffffffu);
    return key <= 0x007fffffu ? -INFINITY : __uint_as_float(~key);
}

// lo and hi with lane `lane` (a constant once the loops are unrolled) replaced by the halves of the lane mask m.  The
// mask is copied by scalar moves first: it may come straight from a vector compare, and a lane write that reads a
// scalar register too soon after a vector instruction wrote it gets the old contents; the compiler, which keeps
// that distance for its own instructions, does not look inside an asm statement (and has no builtin for the lane
// write here).  A scalar move waits for the vector instruction by itself.
__device__ inline void write_lanes(unsigned& lo, unsigned& hi, unsigned long long m, int lane) {
    unsigned t0, t1;
    asm("s_mov_b32 %2, %4\n\ts_mov_b32 %3, %5\n\tv_writelane_b32 %0, %2, %6\n\tv_writelane_b32 %1, %3, %6"
        : "+v"(lo), "+v"(hi), "=&s"(t0), "=&s"(t1)
        : "s"((unsigned)m), "s"((unsigned)(m >> 32)), "i"(lane));
}

constexpr int kClassifyWaves = 8;
constexpr int kClassifyTiles = 4;
constexpr int kClassifyStage = 768;  // entries staged per wave (640, four workgroups per CU, measured the same)
constexpr int kClassifySlicesMax = 256;  // (the third launch scans a column's slices with its first 256 threads)

// Tiles per slice when a column of T tiles is cut into `slices` runs of whole iterations.
__host__ __device__ inline int classify_slice_tiles(int T, int slices) {
    const int per = (T + slices - 1) / slices;
    return (per + kClassifyTiles - 1) / kClassifyTiles * kClassifyTiles;
}

template <int MODE, bool MARKS /* row_plane given: the rows of sure survivors are recorded */>
__global__ __launch_bounds__(kClassifyWaves * 64) void k_classify(int relu, int channels,
                                                                  const int* __restrict__ tile_start,
                                                                  const float* __restrict__ resp,
                                                                  ColState* __restrict__ cols,
                                                                  uint2* __restrict__ side, uint2* __restrict__ part,
                                                                  unsigned long long* __restrict__ row_plane,
                                                                  long long plane_words) {
    constexpr int U = kClassifyTiles;  // tiles per iteration
    constexpr int WCAP = kClassifyStage;  // staged entries per wave (a flush leaves room for an iteration's worth)
    __shared__ uint2 s_buf[kClassifyWaves * WCAP];
    const int groups = (channels + kClassifyWaves - 1) / kClassifyWaves;
    const int b = blockIdx.x / groups;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // (uniform, and known to be)
    const int oc = (blockIdx.x - b * groups) * kClassifyWaves + wave;
    if (oc >= channels) return;  // (the last group may be short)
    const int col = b * channels + oc;
    const ColState st = cols[col];
    if (st.done) return;
    const int t0 = tile_start[b], t1 = tile_start[b + 1];
    const float s_lo = score_bound(st.tau_lo, MODE), s_hi = score_bound(st.tau_hi, MODE);
    const unsigned long long relu_off = relu ? 0ull : ~0ull;
    // |x| as the score: a row survives for sure when y > sure_hi, y = x under ReLU (a negative value is dropped
    // later), |x| without; sure_hi = the bracket's upper end where that is a number not below zero (an entry above it
    // is then non-zero, and positive under ReLU), 0 where it is negative (every entry is above it), infinity where it
    // is no number (no entry compares above it)
    const unsigned sure_sign = relu ? 0xffffffffu : 0x7fffffffu;
    const float sure_hi = s_hi >= 0.0f ? s_hi : (s_hi < 0.0f ? 0.0f : INFINITY);
    uint2* wbuf = s_buf + wave * WCAP;
    int fill = 0;                    // wave-uniform
    unsigned n_nz = 0, n_above = 0;  // per lane
    // slice y of the column: tiles [first, last)
    const int L = classify_slice_tiles(t1 - t0, (int)gridDim.y);
    const int first = t0 + (int)blockIdx.y * L;
    const int last = first + L < t1 ? first + L : t1;
    // a flush reserves its piece of the column's side-buffer entries from the column's cursor: one returning atomic
    // per wave and flush, a few thousand a layer, which is what keeps the column's entries in one run
    uint2* run = side + st.side_off;
    auto flush = [&]() {
        unsigned base = 0;
        if (lane == 0) base = atomicAdd(&cols[col].side_fill, (unsigned)fill);
        base = __builtin_amdgcn_readfirstlane(base);
        for (int i = lane; i < fill; i += 64) run[base + i] = wbuf[i];
        fill = 0;
    };
    unsigned long long* plane = MARKS ? row_plane + (size_t)oc * plane_words : nullptr;
    // the values of tiles tile0 .. tile0 + U - 1 at rows lane and lane + 64 (a tile past the slice: the slice's first)
    auto load = [&](int tile0, float (&v)[U][2]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int tile = tile0 + u;
            const float* seg = resp + ((size_t)(tile < last ? tile : first) * channels + oc) * kTileRows;
            v[u][0] = seg[lane];
            v[u][1] = seg[64 + lane];
        }
    };
    // one iteration: the tiles tile0 .. tile0 + U - 1, whose values are in v; FULL: all of them are in the slice.
    // The loop is bound by scalar instructions (lane masks are combined, counted and turned into branch conditions
    // there), so whatever can be decided per lane is: the two counts are kept per lane and added up at the end,
    // the bracket test is one condition whose mask is also the staging order, and with |x| as the score the rows
    // that survive for sure are one compare (x, or |x| without ReLU, against the bracket's upper end).
    auto process = [&](int tile0, const float (&v)[U][2], auto full) {
        constexpr bool FULL = decltype(full)::value;
        unsigned mark_lo = 0, mark_hi = 0;  // lane j: the marks of tile j / 2, rows (j & 1) * 64 ..
        const unsigned pos0 = (unsigned)(tile0 - t0) * kTileRows + (unsigned)lane;
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float x = (FULL || tile0 + u < last) ? v[u][h] : 0.0f;
                const float sc = MODE == SCNN_TOPK_ABS ? fabsf(x) : x;
                const bool nz = x != 0.0f, above = nz && sc > s_hi;
                const bool hit = nz && sc >= s_lo && !(sc > s_hi);  // inside the bracket
                const unsigned long long m = __ballot(hit);
                n_nz += nz ? 1u : 0u;
                n_above += above ? 1u : 0u;
                if constexpr (MARKS) {
                    unsigned long long sure;
                    if constexpr (MODE == SCNN_TOPK_ABS)
                        sure = __ballot(__uint_as_float(__float_as_uint(x) & sure_sign) > sure_hi);
                    else
                        sure = __ballot(above) & (__ballot(x > 0.0f) | relu_off);
                    write_lanes(mark_lo, mark_hi, sure, u * 2 + h);
                }
                if (hit) {  // the value itself is staged; its key is taken when the entry is read
                    const unsigned rank =
                        __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
                    wbuf[fill + (int)rank] = make_uint2(__float_as_uint(x), pos0 + (unsigned)(u * kTileRows + h * 64));
                }
                fill += __popcll(m);
            }
        }
        if (MARKS && lane < 2 * U && (FULL || tile0 + (lane >> 1) < last))
            plane[2 * (size_t)tile0 + lane] = ((unsigned long long)mark_hi << 32) | mark_lo;
    };
    auto process_any = [&](int tile0, const float (&v)[U][2]) {
        if (tile0 + U <= last) process(tile0, v, std::true_type{});
        else process(tile0, v, std::false_type{});
    };
    // Two register sets in turn, so that an iteration's loads are in flight during the whole of the one before it.
    // The staging buffer is emptied, when an iteration could overfill it, before the next loads are issued, never
    // between an iteration's loads and their use, and the next loads are issued whether or not there is a next
    // iteration: the compiler counts outstanding loads along every path, and behind a loop of stores, or a branch
    // that may have skipped the loads, it waits for all of them.
    auto make_room = [&]() {
        if (fill > WCAP - U * kTileRows) flush();
    };
    float va[U][2], vb[U][2];
    if (first < last) load(first, va);
    for (int tile0 = first; tile0 < last; tile0 += 2 * U) {
        make_room();
        load(tile0 + U, vb);  // (always: past the slice it reads the slice's first tile again, and nobody looks)
        process_any(tile0, va);
        if (tile0 + U >= last) break;
        make_room();
        load(tile0 + 2 * U, va);
        process_any(tile0 + U, vb);
    }
    if (fill > 0) flush();
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        n_nz += __shfl_xor(n_nz, d, 64);
        n_above += __shfl_xor(n_above, d, 64);
    }
    if (lane == 0) part[(size_t)col * gridDim.y + blockIdx.y] = make_uint2(n_nz, n_above);
}

// Third launch, one workgroup per column: the exact k-th strongest key tau, the number of entries equal to it and,
// if those do not all fit, the position up to which they do -- by radix select over the column's side-buffer
// entries when the bracket held the k-th entry (the rule), over the column itself when it did not.
constexpr int kSideThreads = 1024;

struct SideEntries {  // entry i of a column's side-buffer entries: {key, position}; the buffer holds the value's bits
    const uint2* e;
    int mode;
    __device__ uint2 operator()(unsigned i) const {
        const uint2 x = e[i];
        return make_uint2(score_key(__uint_as_float(x.x), mode), x.y);
    }
};
struct ColumnEntries {  // slot i of a column of the response matrix (key 0: not an entry)
    const float* col;   // the column's values in its first tile
    size_t tile_pitch;  // floats from one tile to the next
    int mode;
    __device__ uint2 operator()(unsigned i) const {
        return make_uint2(score_key(col[(size_t)(i >> 7) * tile_pitch + (i & 127u)], mode), i);
    }
};

// The kk strongest of m entries {key, position} whose keys lie in [key_lo, key_hi] (key 0: not an entry), of equal keys those
// of lowest position, are the ones above tau and the ones equal to tau at positions <= cut.  1 <= kk <= number of
// entries.  The digits of the radix select, 11 bits at most, are taken from key - key_lo, most significant first, until at
// most 64 entries share them (a bracket of some ten thousand: the first) or all that share them survive.  Between the passes up to kSettleCached entries per thread are held
// in registers and kSettleLds more per workgroup in LDS (brackets that hold long runs of equal scores run to 30 000
// entries on the paper's first layers).  (whole workgroup)
// Two sizes: 20 per thread + 12288 (one workgroup per compute unit: its registers and LDS), the rule; 4 per thread +
// 2048 for layers of many columns, whose brackets are short and whose workgroups then fit two to a compute unit.
template <int kSettleCached> constexpr unsigned kSettleRegsOf = (unsigned)kSettleCached * 1024u;

// held: the entries threadIdx.x + 1024 * u of the column, more: the entries from kSettleRegs on, if cached
// (m <= kSettleRegs + kSettleLds); both loaded by the caller.
constexpr int kSettleFew = 64;
struct SettleFew {  // (LDS)
    uint2 entry[kSettleFew], found;
    unsigned fill;
};

template <int kSettleCached, class Entries>
__device__ __forceinline__ void settle_column(const Entries& entry, unsigned m, const uint2 (&held)[kSettleCached],
                                     const uint2* more, bool cached, unsigned key_lo, unsigned key_hi, long long kk,
                                     unsigned* s_h, unsigned* s_wave, int* s_res, SettleFew& few, unsigned& tau,
                                     unsigned& cut) {
    constexpr unsigned kSettleRegs = kSettleRegsOf<kSettleCached>;
    auto clear = [&]() {
        for (int i = threadIdx.x; i < kHistBins; i += kSideThreads) s_h[i] = 0;
        __syncthreads();
    };
    // Data with long runs of equal scores (unit input values) sends most lanes of a wave to one bin, and LDS serves
    // the atomics of a wave on one word one after the other: the lanes that share the first active lane's bin add
    // once, through that lane; the others add on their own.
    auto add = [&](bool valid, unsigned bin) {
        const unsigned long long act = __ballot(valid);
        if (act == 0ull) return;  // (uniform)
        const int first = __ffsll((long long)act) - 1;
        const unsigned b0 = __shfl(valid ? bin : 0u, first, 64);
        const unsigned long long same = __ballot(valid && bin == b0);
        if ((int)(threadIdx.x & 63) == first) atomicAdd(&s_h[b0], (unsigned)__popcll(same));
        else if (valid && bin != b0) atomicAdd(&s_h[bin], 1u);
    };
    // histogram of digit(entry) over the entries that pass(entry)
    auto histogram = [&](auto pass, auto digit) {
        clear();
        if (cached) {
#pragma unroll
            for (int u = 0; u < kSettleCached; ++u) {
                const bool valid = held[u].x != 0u && pass(held[u]);
                add(valid, valid ? digit(held[u]) : 0u);
            }
            if (m > kSettleRegs) {  // (uniform; whole waves take part in every round: add() uses ballots)
                const unsigned n_more = m - kSettleRegs;
                for (unsigned j0 = 0; j0 < n_more; j0 += kSideThreads) {
                    const unsigned j = j0 + threadIdx.x;
                    const uint2 x = j < n_more ? more[j] : make_uint2(0u, 0u);
                    const bool valid = x.x != 0u && pass(x);
                    add(valid, valid ? digit(x) : 0u);
                }
            }
        } else {
            for (unsigned i0 = threadIdx.x; i0 < m; i0 += kSideThreads * 8) {  // loads issued eight at a time
                uint2 x[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const unsigned i = i0 + (unsigned)kSideThreads * u;
                    x[u] = i < m ? entry(i) : make_uint2(0u, 0u);
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const bool valid = x[u].x != 0u && pass(x[u]);
                    add(valid, valid ? digit(x[u]) : 0u);
                }
            }
        }
        __syncthreads();
    };
    // f(entry) for all of them
    auto each = [&](auto f) {
        if (cached) {
#pragma unroll
            for (int u = 0; u < kSettleCached; ++u) f(held[u]);
            if (m > kSettleRegs)
                for (unsigned j = threadIdx.x; j < m - kSettleRegs; j += kSideThreads) f(more[j]);
        } else {
            for (unsigned i0 = threadIdx.x; i0 < m; i0 += kSideThreads * 8) {
                uint2 x[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const unsigned i = i0 + (unsigned)kSideThreads * u;
                    x[u] = i < m ? entry(i) : make_uint2(0u, 0u);
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) f(x[u]);
            }
        }
    };
    int bin = 0, picks = 0;
    unsigned before = 0, in_bin = 0;
    const unsigned span = key_hi - key_lo;
    int nb = span ? 32 - __clz(span) : 1;  // bits of key - key_lo still open
    unsigned prefix = 0;                   // the bits above them
    if (threadIdx.x == 0) few.fill = 0u;   // (the histogram's barriers lie between)
    do {  // (uniform)
        const int w = nb < 11 ? nb : 11, shift = nb - w;
        const int above = nb;  // (captured by value)
        if (picks > 0) __syncthreads();  // (the last histogram has been read)
        histogram([=](uint2 x) { return (unsigned)((unsigned long long)(x.x - key_lo) >> above) == prefix; },
                  [=](uint2 x) { return ((x.x - key_lo) >> shift) & ((1u << w) - 1u); });
        block_pick(s_h, kk, true, s_wave, s_res + 2 * (picks++ & 1), bin, before);
        kk -= (long long)before;
        in_bin = s_h[bin];
        prefix = (prefix << w) | (unsigned)bin;
        nb = shift;
    } while (nb > 0 && in_bin > (unsigned)kSettleFew && (long long)in_bin != kk);
    tau = key_lo + (prefix << nb);  // the least of the bin's keys
    cut = 0xffffffffu;
    if ((long long)in_bin == kk) {  // all of the bin survive
        __syncthreads();
        return;
    }
    if (in_bin <= (unsigned)kSettleFew) {
        // few share these bits: a wave ranks them by key and position
        const int low = nb;
        each([&](uint2 x) {
            if (x.x != 0u && (x.x - key_lo) >> low == prefix) few.entry[atomicAdd(&few.fill, 1u)] = x;
        });
        __syncthreads();
        if (threadIdx.x < in_bin) {
            const uint2 own = few.entry[threadIdx.x];
            int rank = 0;  // entries that go before it: stronger, or as strong at a lower position
            for (int i = 0; i < (int)in_bin; ++i) {
                const uint2 o = few.entry[i];
                rank += o.x > own.x || (o.x == own.x && o.y < own.y) ? 1 : 0;
            }
            if (rank == (int)kk - 1) few.found = own;
        }
        __syncthreads();
        tau = few.found.x;
        cut = few.found.y;
        return;
    }
    // a run of equal keys (no bit is open), not all of which fit: ascending radix select on the position
    const unsigned t = tau;
    unsigned pprefix = 0;
    long long rank = kk;
    for (int pass = 0; pass < 3; ++pass) {
        const int shift = pass == 0 ? 21 : (pass == 1 ? 10 : 0), bits = pass == 2 ? 10 : 11;
        __syncthreads();
        histogram([=](uint2 x) { return x.x == t && (pass == 0 || (x.y >> (shift + bits)) == pprefix); },
                  [=](uint2 x) { return (x.y >> shift) & ((1u << bits) - 1u); });
        block_pick(s_h, rank, false, s_wave, s_res + 2 * (picks++ & 1), bin, before);
        pprefix = (pprefix << bits) | (unsigned)bin;
        rank -= (long long)before;
    }
    cut = pprefix;
}

template <int kSettleCached, unsigned kSettleLds, bool MARKS /* row_keep and tile_base given */>
__global__ __launch_bounds__(kSideThreads) __attribute__((amdgpu_waves_per_eu(kSettleCached > 8 ? 4 : 8)))
void k_settle(int mode, int relu, int channels, long long k,
                                                         const int* __restrict__ tile_start,
                                                         const float* __restrict__ resp, ColState* __restrict__ cols,
                                                         const uint2* __restrict__ side,
                                                         const uint2* __restrict__ part, int slices,
                                                         unsigned long long* row_keep,
                                                         long long* __restrict__ tile_base, Counters* ctr) {
    __shared__ __align__(16) unsigned s_h[kHistBins];
    __shared__ __align__(16) unsigned s_wave[kPickWaves];
    __shared__ int s_res[4];
    __shared__ uint2 s_part[4];
    constexpr unsigned kSettleRegs = kSettleRegsOf<kSettleCached>;
    __shared__ uint2 s_more[kSettleLds];
    __shared__ unsigned s_cnt;
    __shared__ SettleFew s_few;
    const int col = blockIdx.x;
    const int b = col / channels, oc = col - b * channels;
    const int t0 = tile_start[b], t1 = tile_start[b + 1];
    ColState st = cols[col];
    // the slices' counts of entries and of entries above the bracket (read along with the column's state; unused, and
    // possibly stale, where the column is settled already)
    uint2 my_part = make_uint2(0u, 0u);
    if ((int)threadIdx.x < slices) my_part = part[(size_t)col * slices + threadIdx.x];
    if (!st.done) {
        const unsigned sum_nz = wave_add(my_part.x), sum_above = wave_add(my_part.y);
        if (threadIdx.x < 256 && (threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = make_uint2(sum_nz, sum_above);
        __syncthreads();
        st.n_nz = s_part[0].x + s_part[1].x + s_part[2].x + s_part[3].x;
        st.n_above = s_part[0].y + s_part[1].y + s_part[2].y + s_part[3].y;
        const unsigned m = st.side_fill;
        const float* col0 = resp + ((size_t)t0 * channels + oc) * kTileRows;
        const size_t pitch = (size_t)channels * kTileRows;
        const SideEntries e{side + st.side_off, mode};
        // the side buffer's entries of the column, in registers if they are few enough (the rule)
        const bool cached = m <= kSettleRegs + kSettleLds;  // (uniform)
        uint2 kept[kSettleCached];
        if (cached) {
#pragma unroll
            for (int u = 0; u < kSettleCached; ++u) {
                const unsigned i = threadIdx.x + (unsigned)kSideThreads * u;
                kept[u] = i < m ? e(i) : make_uint2(0u, 0u);
            }
            for (unsigned i = kSettleRegs + threadIdx.x; i < m; i += kSideThreads) s_more[i - kSettleRegs] = e(i);
            __syncthreads();
        }
        // the row of a surviving entry of the bracket is marked unless some channel has marked it already
        auto word_of = [&](uint2 x) { return row_keep + 2 * (size_t)(t0 + (int)(x.y >> 7)) + ((x.y >> 6) & 1u); };
        auto mark = [&](uint2 x, unsigned long long have) {
            const unsigned long long bit = 1ull << (x.y & 63u);
            if (have & bit) return;
            if (relu && !(col0[(size_t)(x.y >> 7) * pitch + (x.y & 127u)] > 0.0f)) return;
            atomicOr(word_of(x), bit);
        };
        unsigned m_eff = m;        // the entries the marking below runs over, and whether they are the cached ones
        bool cached_eff = cached;
        bool held;  // the side buffer decides the column
        if ((long long)st.n_nz <= k) {
            // fewer entries than k: all survive (tau = 0, every non-zero key is above it); the rows are all marked if
            // no entry lay below the bracket
            st.tau = 0;
            held = st.n_above + m == st.n_nz;
        } else {
            const long long k_rem = k - (long long)st.n_above;
            held = k_rem >= 1 && k_rem <= (long long)m;
            bool settled = false;
            if (held && !cached) {
                // A bracket too long to cache (few, very long columns): read it twice instead of once per digit.
                // First the histogram of the leading digit; then, with the k-th key's bin known, the entries of that
                // bin go to LDS and the entries above it, which survive whatever the rest of the key, mark their
                // rows; the remaining digits and the tie cut are settled on the cached bin.
                const unsigned span = st.tau_hi - st.tau_lo;
                const int nb = span ? 32 - __clz(span) : 1;
                const int w = nb < 11 ? nb : 11, shift = nb - w;
                const unsigned lo = st.tau_lo;
                auto digit = [=](uint2 x) { return ((x.x - lo) >> shift) & ((1u << w) - 1u); };
                for (int i = threadIdx.x; i < kHistBins; i += kSideThreads) s_h[i] = 0;
                if (threadIdx.x == 0) s_cnt = 0;
                __syncthreads();
                for (unsigned i0 = threadIdx.x; i0 < m; i0 += kSideThreads * 16) {  // sixteen values in flight per thread
                    unsigned x[16];
#pragma unroll
                    for (int u = 0; u < 16; ++u) {
                        const unsigned i = i0 + (unsigned)kSideThreads * u;
                        x[u] = i < m ? e.e[i].x : 0u;
                    }
#pragma unroll
                    for (int u = 0; u < 16; ++u) {
                        const unsigned key = score_key(__uint_as_float(x[u]), mode);
                        if (key != 0u) atomicAdd(&s_h[digit(make_uint2(key, 0u))], 1u);
                    }
                }
                __syncthreads();
                int bin;
                unsigned before;
                block_pick(s_h, k_rem, true, s_wave, s_res + 2, bin, before);
                const unsigned in_bin = s_h[bin];
                __syncthreads();  // (every thread has read the count before the histogram is cleared again)
                if (in_bin <= kSettleLds) {  // (uniform)
                    constexpr int F = MARKS ? 8 : 16;  // entries in flight per thread
                    for (unsigned i0 = threadIdx.x; i0 < m; i0 += kSideThreads * F) {
                        uint2 x[F];
                        unsigned long long have[MARKS ? F : 1];
#pragma unroll
                        for (int u = 0; u < F; ++u) {
                            const unsigned i = i0 + (unsigned)kSideThreads * u;
                            x[u] = i < m ? e(i) : make_uint2(0u, 0u);
                        }
#pragma unroll
                        for (int u = 0; u < (MARKS ? F : 0); ++u) {
                            have[u] = ~0ull;
                            if (x[u].x != 0u && (int)digit(x[u]) > bin)
                                have[u] = __hip_atomic_load(word_of(x[u]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        }
#pragma unroll
                        for (int u = 0; u < F; ++u) {
                            if (x[u].x == 0u) continue;
                            const int d = (int)digit(x[u]);
                            if (d == bin) s_more[atomicAdd(&s_cnt, 1u)] = x[u];
                            else if (MARKS && d > bin) mark(x[u], have[MARKS ? u : 0]);
                        }
                    }
                    uint2 none[kSettleCached];
#pragma unroll
                    for (int u = 0; u < kSettleCached; ++u) none[u] = make_uint2(0u, 0u);
                    if constexpr (MARKS) {
#pragma unroll
                        for (int u = 0; u < kSettleCached; ++u) kept[u] = none[u];
                    }
                    __syncthreads();
                    const unsigned long long lo2 = (unsigned long long)lo + ((unsigned long long)(unsigned)bin << shift);
                    unsigned long long hi2 = lo2 + ((1ull << shift) - 1ull);
                    if (hi2 > st.tau_hi) hi2 = st.tau_hi;
                    m_eff = kSettleRegs + in_bin;  // (the first kSettleRegs entries are the empty registers)
                    cached_eff = true;
                    settle_column<kSettleCached>(e, m_eff, none, s_more, true, (unsigned)lo2, (unsigned)hi2, k_rem - (long long)before, s_h,
                                  s_wave, s_res, s_few, st.tau, st.cut);
                    settled = true;
                }
            }
            if (settled) {
            } else if (held)
                settle_column<kSettleCached>(e, m, kept, s_more, cached, st.tau_lo, st.tau_hi, k_rem, s_h, s_wave, s_res, s_few, st.tau,
                              st.cut);
            else
                settle_column<kSettleCached>(ColumnEntries{col0, pitch, mode}, (unsigned)(t1 - t0) * kTileRows, kept, s_more, false, 0u,
                              0xffffffffu, k, s_h, s_wave, s_res, s_few, st.tau, st.cut);
        }
        if (threadIdx.x == 0) {
            st.done = 1;
            cols[col] = st;
            if (!held) atomicOr(&ctr->bracket_failed, 1u);  // the rows marked so far cannot be relied on
        }
        if (MARKS && held) {
            // the bracket's entries that survive keep their rows too
            auto survives = [&](uint2 x) { return x.x > st.tau || (x.x == st.tau && x.x != 0u && x.y <= st.cut); };
            if (cached_eff) {
#pragma unroll
                for (int u0 = 0; u0 < kSettleCached; u0 += 8) {  // eight words in flight per thread
                    unsigned long long have[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        have[u] = ~0ull;
                        if (u0 + u < kSettleCached && survives(kept[u0 + u]))
                            have[u] = __hip_atomic_load(word_of(kept[u0 + u]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        if (u0 + u < kSettleCached) mark(kept[u0 + u], have[u]);
                }
                for (unsigned i = kSettleRegs + threadIdx.x; i < m_eff; i += kSideThreads) {
                    const uint2 x = s_more[i - kSettleRegs];
                    if (survives(x)) mark(x, __hip_atomic_load(word_of(x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                }
            } else {
                for (unsigned i0 = threadIdx.x; i0 < m_eff; i0 += kSideThreads * 8) {  // eight entries in flight per thread
                    uint2 x[8];
                    unsigned long long have[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const unsigned i = i0 + (unsigned)kSideThreads * u;
                        x[u] = i < m_eff ? e(i) : make_uint2(0u, 0u);
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        have[u] = ~0ull;
                        if (survives(x[u]))
                            have[u] = __hip_atomic_load(word_of(x[u]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u) mark(x[u], have[u]);
                }
            }
        }
    }
    if constexpr (!MARKS) return;
    // The workgroup that ends last turns the marked rows into the output row at which every tile starts.  The marks
    // are only ever touched by device-scope atomics, which are performed at the point of coherence; the barrier waits
    // for this workgroup's to be acknowledged, so no cache write-back (a fence, tens of microseconds here) is needed
    // before the count.
    __syncthreads();
    if (threadIdx.x == 0) s_res[0] = (atomicAdd(&ctr->cols_done, 1u) == gridDim.x - 1) ? 1 : 0;
    __syncthreads();
    if (!s_res[0]) return;
    if (__hip_atomic_load(&ctr->bracket_failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
    const int n_tiles = (int)ctr->n_tiles;
    const int per = (n_tiles + kSideThreads - 1) / kSideThreads;  // consecutive tiles per thread
    const int first = threadIdx.x * per;
    auto rows_of = [&](int t) -> unsigned {
        return (unsigned)(__popcll(__hip_atomic_load(&row_keep[2 * (size_t)t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) +
                          __popcll(__hip_atomic_load(&row_keep[2 * (size_t)t + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)));
    };
    constexpr int kKept = 8;  // counts held in registers between the two sweeps
    unsigned cnt[kKept];
    unsigned local = 0;
#pragma unroll
    for (int j = 0; j < kKept; ++j) {
        const int t = first + j;
        cnt[j] = (j < per && t < n_tiles) ? rows_of(t) : 0u;
        local += cnt[j];
    }
    for (int t = first + kKept; t < first + per && t < n_tiles; ++t) local += rows_of(t);
    // exclusive scan over the 1024 threads (64-bit sums through s_h)
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned long long inc = local;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned long long t = __shfl_up(inc, d, 64);
        if (lane >= d) inc += t;
    }
    unsigned long long* s_tot = (unsigned long long*)s_h;
    __syncthreads();
    if (lane == 63) s_tot[wave] = inc;
    __syncthreads();
    unsigned long long base = 0, total = 0;
    for (int w = 0; w < kSideThreads / 64; ++w) {
        const unsigned long long x = s_tot[w];
        if (w < wave) base += x;
        total += x;
    }
    long long run = (long long)(base + inc - local);
#pragma unroll
    for (int j = 0; j < kKept; ++j) {
        const int t = first + j;
        if (j < per && t < n_tiles) tile_base[t] = run;
        run += cnt[j];
    }
    for (int t = first + kKept; t < first + per && t < n_tiles; ++t) {
        tile_base[t] = run;
        run += rows_of(t);
    }
    if (threadIdx.x == 0) ctr->n_rows = (long long)total;
}

// The whole selection of a column in one workgroup, for columns that fit its registers (grids of at most 32768
// sites per sample: the paper's networks from the second resolution level on), over keys read once; no global histogram, no
// side buffer and one launch instead of three (what such a layer costs is launches).  The digits, 11 bits at most, are taken
// from the distance to the smallest key, most significant first, until the bin of the k-th key holds at most 64 entries (columns of 4096
// positions: nearly always the first digit) or all of its entries survive; a wave then ranks these by key and position.  Runs
// of more equal keys end in a radix select on the position.  Bound by its barriers and the latency of the steps between them.
constexpr int kSmallThreads = 1024;
constexpr int kSmallPerThread = 32;
constexpr long long kSmallColumn = (long long)kSmallThreads * kSmallPerThread;  // entries of a column at most
constexpr int kSmallFew = 64;

template <int NU /* keys per thread: columns of at most 1024 NU positions */>
__global__ __launch_bounds__(kSmallThreads) void k_select_small(int mode, int channels,
                                                                const int* __restrict__ tile_start,
                                                                const float* __restrict__ resp, long long k,
                                                                ColState* __restrict__ cols) {
    __shared__ __align__(16) unsigned s_h[kHistBins];
    __shared__ __align__(16) unsigned s_wave[kPickWaves];
    __shared__ int s_res[4];
    __shared__ unsigned s_total, s_range[2], s_fill;
    __shared__ uint2 s_few[kSmallFew];
    const int col = blockIdx.x;
    const int b = col / channels, oc = col - b * channels;
    const int t0 = tile_start[b], t1 = tile_start[b + 1];
    const unsigned n = (unsigned)(t1 - t0) * kTileRows;  // positions of the column (<= 1024 NU, see the launcher)
    if (threadIdx.x == 0) {
        s_total = s_fill = 0u;
        s_range[0] = 0xffffffffu;
        s_range[1] = 0u;
    }
    auto clear = [&]() {
        for (int i = threadIdx.x; i < kHistBins; i += kSmallThreads) s_h[i] = 0;
    };
    clear();
    // entry u of the thread sits at position u * 1024 + thread: a wave reads 64 consecutive rows of one tile
    unsigned key[NU];
    unsigned mine = 0, kmin = 0xffffffffu, kmax = 0u;
    {
        const float* first = resp + ((size_t)(t0 + (int)(threadIdx.x >> 7)) * channels + oc) * kTileRows + (threadIdx.x & 127u);
        const size_t pitch = (size_t)(kSmallThreads / kTileRows) * channels * kTileRows;  // from a thread's entry to its next
        constexpr int G = NU < 8 ? NU : 8;                                                // loads in flight together
#pragma unroll
        for (int u0 = 0; u0 < NU; u0 += G) {
            float x[G];
#pragma unroll
            for (int u = 0; u < G; ++u) {
                const bool has = (unsigned)(u0 + u) * kSmallThreads + threadIdx.x < n;
                x[u] = has ? first[(size_t)(u0 + u) * pitch] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < G; ++u) {
                const unsigned v = score_key(x[u], mode);
                key[u0 + u] = v;
                mine += v != 0u ? 1u : 0u;
                kmin = v != 0u && v < kmin ? v : kmin;
                kmax = v > kmax ? v : kmax;
            }
        }
    }
    __syncthreads();
    mine = wave_add(mine);
    kmin = wave_min(kmin);
    kmax = wave_max(kmax);
    if ((threadIdx.x & 63) == 0 && mine) {
        atomicAdd(&s_total, mine);
        atomicMin(&s_range[0], kmin);
        atomicMax(&s_range[1], kmax);
    }
    __syncthreads();
    ColState st;
    st.tau = 0; st.cut = 0xffffffffu; st.tau_lo = 0; st.tau_hi = 0; st.n_nz = s_total;
    st.n_above = 0; st.side_fill = 0; st.done = 1; st.side_off = 0;
    if (k <= 0) st.tau = 0xffffffffu;  // no key is stronger: nothing survives
    if (k <= 0 || (long long)st.n_nz <= k) {  // or fewer entries than k: all survive (tau = 0)
        if (threadIdx.x == 0) cols[col] = st;
        return;
    }
    // keys from here on: key - smallest + 1, still 0 where there is no entry
    const unsigned base = s_range[0] - 1u, span = s_range[1] - base;
#pragma unroll
    for (int u = 0; u < NU; ++u) key[u] = key[u] != 0u ? key[u] - base : 0u;
    int open = 32 - __clz(span);  // low bits still open
    unsigned prefix = 0, in_bin = 0, before = 0;  // the bits above them
    long long k_rem = k;
    int bin = 0, picks = 0;
    // of the entries that pass(key, position), histogram of digit(key, position); s_h is clear
    auto histogram = [&](auto pass, auto digit) {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const unsigned i = (unsigned)u * kSmallThreads + threadIdx.x;
            if (key[u] != 0u && pass(key[u], i)) atomicAdd(&s_h[digit(key[u], i)], 1u);
        }
        __syncthreads();
    };
    auto pick = [&](bool descending) {
        block_pick(s_h, k_rem, descending, s_wave, s_res + 2 * (picks++ & 1), bin, before);
        k_rem -= (long long)before;
    };
    auto fresh = [&]() {  // (the last histogram has been read)
        __syncthreads();
        clear();
        __syncthreads();
    };
    {
        const int w = open < 11 ? open : 11;
        open -= w;
        histogram([](unsigned, unsigned) { return true; }, [=](unsigned x, unsigned) { return x >> open; });
        pick(true);
        in_bin = s_h[bin];
        prefix = (unsigned)bin;
    }
#pragma unroll 1
    while (open > 0 && in_bin > (unsigned)kSmallFew && (long long)in_bin != k_rem) {  // (uniform)
        const int w = open < 11 ? open : 11, shift = open - w, above = open;
        fresh();
        histogram([=](unsigned x, unsigned) { return (x >> above) == prefix; },
                  [=](unsigned x, unsigned) { return (x >> shift) & ((1u << w) - 1u); });
        pick(true);
        in_bin = s_h[bin];
        prefix = (prefix << w) | (unsigned)bin;
        open = shift;
    }
    if ((long long)in_bin == k_rem) {  // all of the bin survive
        if (threadIdx.x == 0) {
            const unsigned least = prefix << open;
            st.tau = base + (least ? least : 1u);
            cols[col] = st;
        }
        return;
    }
    if (in_bin <= (unsigned)kSmallFew) {
#pragma unroll
        for (int u = 0; u < NU; ++u)
            if (key[u] != 0u && key[u] >> open == prefix)
                s_few[atomicAdd(&s_fill, 1u)] = make_uint2(key[u], (unsigned)u * kSmallThreads + threadIdx.x);
        __syncthreads();
        if (threadIdx.x >= in_bin) return;
        const uint2 own = s_few[threadIdx.x];
        int rank = 0;  // entries that go before it: stronger, or as strong at a lower position
        for (int i = 0; i < (int)in_bin; ++i) {
            const uint2 o = s_few[i];
            rank += o.x > own.x || (o.x == own.x && o.y < own.y) ? 1 : 0;
        }
        if (rank == (int)k_rem - 1) {
            st.tau = base + own.x;
            st.cut = own.y;
            cols[col] = st;
        }
        return;
    }
    // a run of equal keys (no bit is open): the position of the k_rem-th (positions have 15 bits)
    const unsigned tau = prefix;
    fresh();
    histogram([tau](unsigned x, unsigned) { return x == tau; }, [](unsigned, unsigned i) { return i >> 4; });
    pick(false);
    const unsigned phi = (unsigned)bin;
    fresh();
    histogram([tau, phi](unsigned x, unsigned i) { return x == tau && (i >> 4) == phi; },
              [](unsigned, unsigned i) { return i & 15u; });
    pick(false);
    if (threadIdx.x == 0) {
        st.tau = base + tau;
        st.cut = (phi << 4) | (unsigned)bin;
        cols[col] = st;
    }
}

// The same for columns of at most 1024 positions (eight tiles: 2-D grids up to 32 x 32, 3-D up to 10^3), one WAVE per
// column and no shared memory: a workgroup of 1024 threads with five passes over a 2048-bin histogram costs a column about
// 10 us.  The k-th strongest key is found bit by bit, from the top: the largest value that at least k keys reach (a compare
// and a ballot's count per register and bit, which is what it is bound by; hence as few registers as the column's tiles
// need, a uniform choice); the tie cut is the position of the q-th equal key in position order.  28 x 28 x 1024, three
// tiles a column, 8192 columns: 28.6 -> 14.8 us (sixteen registers always, the keys' leading bits compared, before); one
// image, eight columns, 10.6 by a workgroup per column, 4.2 so.  kTinyPerLane = 64 takes columns of up to 4096 positions
// (16^3 grids) where there are a thousand of them or more; with 64 a wave's 32 steps over 64 registers take 43 us and a
// workgroup's histogram passes 11.
constexpr long long kTinyColumn = 64 * 16;   // positions of a column at most, 16 keys per lane
constexpr long long kTinyColumn64 = 64 * 64;  // ... 64 keys per lane
constexpr int kTinyManyColumns = 1024;

template <int NU /* keys per lane: n <= 64 NU */>
__device__ __forceinline__ void select_tiny(int mode, const float* __restrict__ column, size_t pitch, unsigned n, long long k,
                                            ColState* __restrict__ out) {
    const int lane = threadIdx.x & 63;
    // key u of the lane sits at position u * 64 + lane
    unsigned key[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const unsigned i = (unsigned)u * 64u + (unsigned)lane;
        key[u] = i < n ? score_key(column[(size_t)(i >> 7) * pitch + (i & 127u)], mode) : 0u;
    }
    ColState st;
    st.tau_lo = 0; st.tau_hi = 0; st.n_above = 0; st.side_fill = 0; st.done = 1; st.side_off = 0;
    wave_threshold<NU>(key, k, st.n_nz, st.tau, st.cut);
    if (lane == 0) *out = st;
}

template <int kTinyPerLane>
__global__ __launch_bounds__(256) void k_select_tiny(int mode, int channels, int ncols,
                                                     const int* __restrict__ tile_start,
                                                     const float* __restrict__ resp, long long k,
                                                     ColState* __restrict__ cols) {
    const int col = __builtin_amdgcn_readfirstlane((int)blockIdx.x * 4 + (int)(threadIdx.x >> 6));
    if (col >= ncols) return;  // (whole waves)
    const int b = col / channels, oc = col - b * channels;
    const int t0 = tile_start[b], tiles = tile_start[b + 1] - t0;
    const unsigned n = (unsigned)tiles * kTileRows;  // positions of the column (<= 64 kTinyPerLane, see the launcher)
    const float* column = resp + ((size_t)t0 * channels + oc) * kTileRows;
    const size_t pitch = (size_t)channels * kTileRows;
    if constexpr (kTinyPerLane == 16) {
        if (tiles <= 2) select_tiny<4>(mode, column, pitch, n, k, cols + col);
        else if (tiles == 3) select_tiny<6>(mode, column, pitch, n, k, cols + col);
        else if (tiles <= 5) select_tiny<10>(mode, column, pitch, n, k, cols + col);
        else select_tiny<16>(mode, column, pitch, n, k, cols + col);
    } else {
        if (tiles <= 16) select_tiny<32>(mode, column, pitch, n, k, cols + col);
        else select_tiny<64>(mode, column, pitch, n, k, cols + col);
    }
}

static long long column_positions(const Geom& g) { return (long long)((g.N + kTileRows - 1) / kTileRows) * kTileRows; }

bool topk_small_columns(const Geom& g) {
    return (long long)((g.N + kTileRows - 1) / kTileRows) * kTileRows <= kSmallColumn;
}

// row_keep[w] = the channels' marks for word w (two words per tile) taken together.  A wave takes 64 consecutive
// words; its loads of a plane are one 512-byte piece, eight planes in flight at a time.
__global__ __launch_bounds__(64) void k_combine_marks(int planes, const unsigned long long* __restrict__ row_plane,
                                                      long long plane_words, const Counters* __restrict__ ctr,
                                                      unsigned long long* __restrict__ row_keep) {
    const long long words = 2 * ctr->n_tiles;
    for (long long w = (long long)blockIdx.x * 64 + threadIdx.x; w < words; w += (long long)gridDim.x * 64) {
        unsigned long long m = 0;
        int p = 0;
        for (; p + 8 <= planes; p += 8) {
            unsigned long long x[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] = row_plane[(size_t)(p + j) * plane_words + w];
#pragma unroll
            for (int j = 0; j < 8; ++j) m |= x[j];
        }
        for (; p < planes; ++p) m |= row_plane[(size_t)p * plane_words + w];
        row_keep[w] = m;
    }
}

hipError_t launch_topk(const Geom& g, int channels, long long k, int mode, int relu, const int* tile_start,
                       const float* resp, ColState* cols, uint2* side, uint2* part, unsigned long long* row_keep,
                       unsigned long long* row_plane, long long* tile_base, long long tiles_cap, Counters* ctr,
                       hipStream_t s) {
    const int ncols = g.batch * channels;
    if (ncols <= 0) return hipSuccess;
    if (column_positions(g) <= kTinyColumn) {
        hipLaunchKernelGGL(k_select_tiny<16>, dim3((unsigned)((ncols + 3) / 4)), dim3(256), 0, s, mode, channels, ncols,
                           tile_start, resp, k, cols);
        return hipGetLastError();
    }
    if (column_positions(g) <= kTinyColumn64 && ncols >= kTinyManyColumns) {
        hipLaunchKernelGGL(k_select_tiny<64>, dim3((unsigned)((ncols + 3) / 4)), dim3(256), 0, s, mode, channels, ncols,
                           tile_start, resp, k, cols);
        return hipGetLastError();
    }
    if (topk_small_columns(g)) {
        const long long n = column_positions(g);
#define SCNN_SELECT_SMALL(NU)                                                                                              \
    hipLaunchKernelGGL(k_select_small<NU>, dim3(ncols), dim3(kSmallThreads), 0, s, mode, channels, tile_start, resp, k, cols)
        if (n <= 4 * kSmallThreads) SCNN_SELECT_SMALL(4);
        else if (n <= 16 * kSmallThreads) SCNN_SELECT_SMALL(16);
        else SCNN_SELECT_SMALL(kSmallPerThread);
#undef SCNN_SELECT_SMALL
        return hipGetLastError();
    }
    const int groups = g.batch * ((channels + kClassifyWaves - 1) / kClassifyWaves);
    int slices = 2048 / groups;  // (r = 128 layer: 1024 and 4096 workgroups in all measured 2 and 3 us slower)
    if (slices < 1) slices = 1;
    if (slices > kClassifySlicesMax) slices = kClassifySlicesMax;
    const bool marks = row_keep && row_plane && tile_base && k > 0;
    hipLaunchKernelGGL(k_bracket, dim3(ncols), dim3(kBracketThreads), 0, s, mode, channels, tile_start, resp, k, cols);
#define SCNN_CLASSIFY(MODE_, MARKS_)                                                                                 \
    hipLaunchKernelGGL((k_classify<MODE_, MARKS_>), dim3(groups, slices), dim3(kClassifyWaves * 64), 0, s, relu,    \
                       channels, tile_start, resp, cols, side, part, marks ? row_plane : nullptr, 2 * tiles_cap)
    if (mode == SCNN_TOPK_ABS) {
        if (marks) SCNN_CLASSIFY(SCNN_TOPK_ABS, true);
        else SCNN_CLASSIFY(SCNN_TOPK_ABS, false);
    } else {
        if (marks) SCNN_CLASSIFY(SCNN_TOPK_SIGNED, true);
        else SCNN_CLASSIFY(SCNN_TOPK_SIGNED, false);
    }
#undef SCNN_CLASSIFY
    if (marks) {
        long long cb = (2 * tiles_cap + 63) / 64;
        cb = cb < 1 ? 1 : (cb > 2048 ? 2048 : cb);
        hipLaunchKernelGGL(k_combine_marks, dim3((unsigned)cb), dim3(64), 0, s, channels, row_plane, 2 * tiles_cap, ctr,
                           row_keep);
    }
#define SCNN_SETTLE(CACHED, LDS, MARKS_)                                                                               \
    hipLaunchKernelGGL((k_settle<CACHED, LDS, MARKS_>), dim3(ncols), dim3(kSideThreads), 0, s, mode, relu, channels, k,  \
                       tile_start, resp, cols, side, part, slices, marks ? row_keep : nullptr,                           \
                       marks ? tile_base : nullptr, ctr)
    if (ncols > 256) {  // (more columns than compute units: two light workgroups per unit)
        if (marks) SCNN_SETTLE(4, 2048u, true);
        else SCNN_SETTLE(4, 2048u, false);
    } else {
        if (marks) SCNN_SETTLE(20, 12288u, true);
        else SCNN_SETTLE(20, 12288u, false);
    }
#undef SCNN_SETTLE
    return hipGetLastError();
}

// ------------------------------------------------------------------ keep mask, ReLU, compaction, write (one pass)
// Tiles are taken in ascending order through a ticket counter; the number of surviving rows before a tile comes
// from a decoupled look-back over per-tile status words {status, count}: a tile first publishes its own count,
// then walks back over its predecessors' words until it meets an inclusive prefix.  A predecessor always belongs
// to a workgroup that is already running (tickets are handed out in order), so the wait is short; it is bounded
// all the same, and a wait that runs out is reported in the status bits instead of hanging.
constexpr unsigned long long kStateAggregate = 1ull << 62, kStateInclusive = 2ull << 62, kStateValueMask = (1ull << 62) - 1;
constexpr int kLookbackSpinLimit = 1 << 22;

// Decoupled look-back, run by the first wave of the workgroup: publishes this tile's count, then inspects its
// predecessors, nearest first, kLookbackSlices * 64 of them per step.  The tiles in flight advance together, so the
// nearest tile whose inclusive sum is known usually lies about as far back as there are workgroups; reading that
// whole stretch with one batch of loads costs one memory round trip instead of one per 64 tiles.
// Returns the number of surviving rows before the tile (valid in every lane).
constexpr int kLookbackSlices = 6;
// (one thread) makes a tile's own count known to its successors
__device__ inline void publish_count(unsigned long long* tile_state, int tile, int count) {
    __hip_atomic_store(&tile_state[tile], (tile == 0 ? kStateInclusive : kStateAggregate) | (unsigned long long)count,
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// (first wave; the tile's count has been published) sums the counts of all predecessors
__device__ inline long long lookback_published(unsigned long long* tile_state, int tile, int count, Counters* ctr) {
    const int lane = threadIdx.x & 63;
    if (tile == 0) return 0;
    long long base = 0;
    int hi = tile - 1;  // nearest predecessor not yet accounted for
    int spins = 0;
    while (hi >= 0) {
        unsigned long long w[kLookbackSlices];
#pragma unroll
        for (int u = 0; u < kLookbackSlices; ++u) {
            const int j = hi - u * 64 - lane;
            w[u] = kStateAggregate;  // positions past tile 0 count as empty aggregates
            if (j >= 0) w[u] = __hip_atomic_load(&tile_state[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        long long v = 0;
        int consumed = 0;
        bool done = false;
#pragma unroll
        for (int u = 0; u < kLookbackSlices; ++u) {
            const unsigned status = (unsigned)(w[u] >> 62);
            const unsigned long long empty = __ballot(status == 0), incl = __ballot(status == 2);
            // the usable prefix of the slice ends at the first inclusive word, or before the first empty one
            const int first_incl = incl ? __ffsll((long long)incl) - 1 : 64;
            const int first_empty = empty ? __ffsll((long long)empty) - 1 : 64;
            const int usable = first_incl < first_empty ? first_incl + 1 : first_empty;  // lanes [0, usable)
            if (lane < usable) v += (long long)(w[u] & kStateValueMask);
            consumed += usable;
            if (first_incl < first_empty) {
                done = true;  // reached an inclusive prefix
                break;
            }
            if (usable < 64) break;  // an unpublished tile: look again from there
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
        base += v;
        if (done) break;
        hi -= consumed;
        if (consumed == 0) {
            if (++spins > kLookbackSpinLimit) {
                if (lane == 0) atomicOr(&ctr->flags, SCNN_FLAG_INTERNAL);
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
    }
    if (lane == 0)
        __hip_atomic_store(&tile_state[tile], kStateInclusive | (unsigned long long)(base + count), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    return base;
}
__device__ inline long long lookback_wave(unsigned long long* tile_state, int tile, int count, Counters* ctr) {
    if ((threadIdx.x & 63) == 0) publish_count(tile_state, tile, count);
    return lookback_published(tile_state, tile, count, ctr);
}

// (one thread) The next of the compaction pass's queue.  Read-modify-writes of one address are served one at a time, about
// 13 ns each on this chip (a plain load of the counter is no cheaper), so a pass over a few thousand tiles can be bound by
// its tickets alone, and a thousand workgroups asking at once wait 13 us for theirs.  Hence no ticket that is known to come
// back empty: a launch with at least as many workgroups as tickets takes one per workgroup (`once`), and a workgroup that
// has seen the queue empty does not ask again.
__device__ inline unsigned take_ticket(Counters* ctr) { return atomicAdd(&ctr->ticket, 1u); }

// (one thread) The result counters.  aux = second counter: the candidate count (aux_is_cand) or a host-side number.
// nnz_out may be null: a later kernel writes them.
__device__ inline void write_counters(Counters* ctr, long long rows, long long* nnz_out, long long aux_imm, int aux_is_cand,
                                      long long out_capacity) {
    if (!nnz_out) return;
    unsigned flags = __hip_atomic_load(&ctr->flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (rows > out_capacity) flags |= SCNN_FLAG_OUT_OVERFLOW;
    nnz_out[0] = rows;
    nnz_out[1] = aux_is_cand ? ctr->n_cand : aux_imm;
    nnz_out[2] = (long long)flags;
    nnz_out[3] = (long long)__hip_atomic_load(&ctr->bracket_failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// .. written by the last workgroup of the compaction pass to end.
__device__ inline void finish_if_last(Counters* ctr, long long* nnz_out, long long aux_imm, int aux_is_cand,
                                      long long out_capacity, unsigned workgroups) {
    if (!nnz_out) return;
    __syncthreads();  // (waits for the workgroup's counter updates, all device-scope atomics, to be acknowledged)
    if (threadIdx.x != 0) return;
    if (atomicAdd(&ctr->finished, 1u) != workgroups - 1) return;
    write_counters(ctr, __hip_atomic_load(&ctr->n_rows, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), nnz_out, aux_imm,
                   aux_is_cand, out_capacity);
}

__global__ __launch_bounds__(256) void k_select_write(Geom g, int channels, int mode, int relu,
                                                      const int* __restrict__ cand_start,
                                                      const int* __restrict__ tile_start,
                                                      const unsigned* __restrict__ cand_lin,
                                                      const float* __restrict__ resp,
                                                      const ColState* __restrict__ cols,
                                                      unsigned long long* tile_state, Counters* ctr,
                                                      int32_t* __restrict__ out_coords, float* __restrict__ out_feats,
                                                      long long out_capacity, long long* __restrict__ nnz_out,
                                                      long long aux_imm, int aux_is_cand) {
    __shared__ unsigned s_tau[1024];
    __shared__ unsigned s_cut[1024];
    __shared__ unsigned s_flag[kTileRows];
    __shared__ int s_rank[kTileRows];
    __shared__ int s_wcount[2];
    __shared__ float s_v[kTileRows][65];
    __shared__ int s_ticket;
    __shared__ long long s_base;

    const int n_tiles = (int)ctr->n_tiles;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned long long lt_mask = (1ull << lane) - 1ull;
    const int n_chunks = (channels + 63) / 64;
    int cur_b = -1;

    for (;;) {
        __syncthreads();  // s_ticket and the tile buffers of the previous round are no longer read
        if (threadIdx.x == 0) s_ticket = (int)take_ticket(ctr);
        __syncthreads();
        const int tile = s_ticket;
        if (tile >= n_tiles) break;
        const int b = sample_of_tile(tile_start, g.batch, tile);
        const int first = cand_start[b] + (tile - tile_start[b]) * kTileRows;
        const unsigned pos0 = (unsigned)(tile - tile_start[b]) * kTileRows;  // position of row 0 in its column
        if (b != cur_b) {
            for (int c = threadIdx.x; c < channels; c += 256) {
                const ColState* st = cols + (size_t)b * channels + c;
                s_tau[c] = st->tau;
                s_cut[c] = st->cut;
            }
            cur_b = b;
        }
        if (threadIdx.x < kTileRows) s_flag[threadIdx.x] = 0;
        __syncthreads();

        // A wave handles channels wave, wave + 4, ... over the tile's 128 rows, four channels per step so that
        // eight loads are in flight.
        auto process = [&](int oc_first, int oc_end, bool stage, int cc) {
            for (int ob = oc_first + wave; ob < oc_end; ob += 16) {
                float v[4][2];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int oc = ob + 4 * j;
                    const float* seg = resp + ((size_t)tile * channels + (oc < oc_end ? oc : ob)) * kTileRows;
                    v[j][0] = seg[lane];
                    v[j][1] = seg[64 + lane];
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int oc = ob + 4 * j;
                    if (oc < oc_end) {
                        const unsigned tau = s_tau[oc], cut = s_cut[oc];
#pragma unroll
                        for (int half = 0; half < 2; ++half) {
                            const int r = half * 64 + lane;
                            const float x = v[j][half];
                            const unsigned key = score_key(x, mode);
                            bool keep = key > tau || (key == tau && key != 0u && pos0 + (unsigned)r <= cut);
                            if (relu) keep = keep && (x > 0.0f);
                            if (keep) s_flag[r] = 1u;
                            if (stage) s_v[r][oc - cc] = keep ? x : 0.0f;
                        }
                    }
                }
            }
        };
        process(0, channels, n_chunks == 1, 0);  // with several chunks the row flags need every channel first
        __syncthreads();
        if (threadIdx.x < kTileRows) {
            const unsigned long long m = __ballot(s_flag[threadIdx.x] != 0u);
            s_rank[threadIdx.x] = __popcll(m & lt_mask);
            if (lane == 0) s_wcount[wave] = __popcll(m);
        }
        __syncthreads();
        const int count = s_wcount[0] + s_wcount[1];
        if (wave == 0) {
            const long long base = lookback_wave(tile_state, tile, count, ctr);
            if (lane == 0) {
                if (tile == n_tiles - 1)
                    __hip_atomic_store(&ctr->n_rows, base + count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                s_base = base;
            }
        }
        __syncthreads();
        const long long base = s_base;
        if (threadIdx.x < kTileRows && s_flag[threadIdx.x]) {
            const int rank = s_rank[threadIdx.x] + (wave ? s_wcount[0] : 0);
            s_rank[threadIdx.x] = rank;
            const long long orow = base + rank;
            if (orow < out_capacity) {
                int c0, c1, c2;
                site_of(g, cand_lin[first + threadIdx.x], c0, c1, c2);
                store_site(g, out_coords + orow * (1 + g.ndim), b, c0, c1, c2);
            }
        }
        __syncthreads();
        for (int cc = 0; cc < channels; cc += 64) {
            const int cw = (channels - cc) < 64 ? (channels - cc) : 64;
            if (n_chunks > 1) {
                process(cc, cc + cw, true, cc);
                __syncthreads();
            }
            for (int i = threadIdx.x; i < kTileRows * 64; i += 256) {
                const int r = i >> 6, c = i & 63;
                if (c < cw && s_flag[r]) {
                    const long long orow = base + s_rank[r];
                    if (orow < out_capacity) out_feats[orow * channels + cc + c] = s_v[r][c];
                }
            }
            __syncthreads();
        }
    }
    finish_if_last(ctr, nnz_out, aux_imm, aux_is_cand, out_capacity, gridDim.x);
}

// The same pass for up to 64 channels, software-pipelined over three tiles.  A workgroup holds tile X (being
// written), tile Y (loaded) and tile Z (its loads in flight).  Per step it decides which entries of Y survive and
// publishes Y's row count, takes the ticket for Z and issues Z's loads, and only then looks back for X and writes
// it.  A tile's count is therefore known to its successors a whole step before its own look-back, so that a
// look-back rarely finds a predecessor unpublished, and the reads of one tile overlap the writes of another.
// The rows of a tile that keep an entry are two 64-bit masks (rows 0..63, 64..127) in one of three rotating slots;
// a row's rank is a popcount.  Three barriers per step.
// STREAM: the output row at which every tile starts is known (tile_base, from the rows marked during the
// selection): tiles are dealt out by workgroup index, nothing is published or looked back at, and no tile waits for
// another.  The selection can find, late, that its marks are not to be relied on (ctr->bracket_failed): the kernel
// then works by look-back although it was given tile_base (the choice is uniform over the launch).
// RANGED: a workgroup owns consecutive tiles, and the rows of those before them are counted (k_select_count64).
template <bool RANGED>
__global__ __launch_bounds__(256, 4) void k_select_write64(Geom g, int channels, int mode, int relu,
                                                        const int* __restrict__ cand_start,
                                                        const int* __restrict__ tile_start,
                                                        const unsigned* __restrict__ cand_lin,
                                                        const float* __restrict__ resp,
                                                        const ColState* __restrict__ cols,
                                                        unsigned long long* tile_state, Counters* ctr,
                                                        int32_t* __restrict__ out_coords,
                                                        float* __restrict__ out_feats, long long out_capacity,
                                                        long long* __restrict__ nnz_out, long long aux_imm,
                                                        int aux_is_cand, const long long* __restrict__ tile_base,
                                                        const unsigned* __restrict__ counts) {
    const bool STREAM = !RANGED && tile_base != nullptr && ctr->bracket_failed == 0u;
    __shared__ uint4 s_thr[64];  // per channel: {threshold if the position passes the cut, threshold if not, cut, -}
    __shared__ unsigned long long s_mask[3][2];
    __shared__ int s_rank[kTileRows];  // output row of a kept row of the tile being written, relative; -1 = dropped
    __shared__ float s_v[kTileRows][65];
    __shared__ int s_ticket;
    __shared__ long long s_base;

    const int n_tiles = (int)ctr->n_tiles;
    // The result counters: STREAM knows them before it starts, and a thousand workgroups that count each other out on one
    // address take 7 us for it where they end together (53 x 75 x 94 x 3, 64 channels: 27.3 -> 21.0 us; on the largest
    // layers, 128^3 x 4: 77 either way).
    auto finish = [&]() {
        if (RANGED) return;  // (written by the workgroup of the last tiles)
        if (!STREAM)
            finish_if_last(ctr, nnz_out, aux_imm, aux_is_cand, out_capacity, gridDim.x);
        else if (blockIdx.x == 0 && threadIdx.x == 0)
            write_counters(ctr, ctr->n_rows, nnz_out, aux_imm, aux_is_cand, out_capacity);
    };
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const bool vec4 = (channels & 3) == 0 && ((size_t)out_feats & 15) == 0;  // rows are 16-byte aligned
    int cur_b = -1;

    // values of channel wave + 4*m at rows lane and lane + 64
    auto load_tile = [&](int tile, float (&v)[16][2]) {
        const float* seg = resp + ((size_t)tile * channels + wave) * kTileRows + lane;
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            if (wave + 4 * m < channels) {  // (uniform in the wave)
                v[m][0] = seg[m * 4 * kTileRows];
                v[m][1] = seg[m * 4 * kTileRows + 64];
            }
        }
    };
    // Zeroes, in the registers, the thread's values that do not survive; the rows that keep an entry are OR-ed into
    // the slot's masks (the slot is zero on entry).  An entry survives iff its key exceeds a threshold that depends
    // on its position only through the tie cut: key > tau, or key >= tau (tau > 0) where the position is within
    // the cut -- the same rule as "above tau, or equal to tau, non-zero and not past the cut".
    auto decide = [&](int tile, int slot, float (&v)[16][2]) {
        const int b = sample_of_tile(tile_start, g.batch, tile);
        const unsigned pos0 = (unsigned)(tile - tile_start[b]) * kTileRows;  // position of row 0 in its column
        if (b != cur_b) {  // (uniform: every thread sees the same tiles; the thresholds' readers are past a barrier)
            if (threadIdx.x < channels) {
                const ColState* st = cols + (size_t)b * channels + threadIdx.x;
                const unsigned tau = st->tau;
                s_thr[threadIdx.x] = make_uint4(tau - (tau != 0u ? 1u : 0u), tau, st->cut, 0u);
            }
            cur_b = b;
            __syncthreads();
        }
        bool row0 = false, row1 = false;
        const unsigned p0 = pos0 + (unsigned)lane, p1 = p0 + 64u;
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            const int oc = wave + 4 * m;
            if (oc < channels) {
                const uint4 t = s_thr[oc];
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const float x = v[m][half];
                    const unsigned key = score_key(x, mode);
                    bool keep = key > ((half ? p1 : p0) <= t.z ? t.x : t.y);
                    if (relu) keep = keep && (x > 0.0f);
                    v[m][half] = keep ? x : 0.0f;
                    if (half == 0) row0 |= keep; else row1 |= keep;
                }
            }
        }
        const unsigned long long b0 = __ballot(row0), b1 = __ballot(row1);
        if (lane == 0) {
            if (b0) atomicOr(&s_mask[slot][0], b0);
            if (b1) atomicOr(&s_mask[slot][1], b1);
        }
    };
    // the surviving values of a tile (the others are zero already), from registers to the transposition buffer
    auto stage_tile = [&](const float (&v)[16][2]) {
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            const int oc = wave + 4 * m;
            if (oc < channels) {
                s_v[lane][oc] = v[m][0];
                s_v[64 + lane][oc] = v[m][1];
            }
        }
    };
    // ranks of the rows of the tile about to be written (threads 0..127, between the step's last two barriers)
    auto rank_rows = [&](int slot) {
        if (threadIdx.x < kTileRows) {
            const unsigned long long m0 = s_mask[slot][0], m1 = s_mask[slot][1];
            const unsigned long long mine = wave ? m1 : m0, below = (1ull << lane) - 1ull;
            const int rank = (wave ? __popcll(m0) : 0) + __popcll(mine & below);
            s_rank[threadIdx.x] = ((mine >> lane) & 1ull) ? rank : -1;
        }
    };
    // write of the staged tile: rows before the tile in s_base, rows within it in s_rank
    auto write_tile = [&](int tile) {
        const int b = sample_of_tile(tile_start, g.batch, tile);
        const int first = cand_start[b] + (tile - tile_start[b]) * kTileRows;
        const long long base = s_base;
        if (threadIdx.x < kTileRows) {
            const int rank = s_rank[threadIdx.x];
            if (rank >= 0 && base + rank < out_capacity) {
                int c0, c1, c2;
                site_of(g, cand_lin[first + threadIdx.x], c0, c1, c2);
                store_site(g, out_coords + (base + rank) * (1 + g.ndim), b, c0, c1, c2);
            }
        }
        if (vec4) {  // 16 bytes per thread: 16 threads cover a row of 64 channels
            const int c = (threadIdx.x & 15) * 4;
            if (c < channels) {
#pragma unroll
                for (int it = 0; it < kTileRows / 16; ++it) {
                    const int r = (threadIdx.x >> 4) + 16 * it;
                    const int rank = s_rank[r];
                    if (rank >= 0 && base + rank < out_capacity) {
                        float4 q;
                        q.x = s_v[r][c];
                        q.y = s_v[r][c + 1];
                        q.z = s_v[r][c + 2];
                        q.w = s_v[r][c + 3];
                        *(float4*)(out_feats + (base + rank) * channels + c) = q;
                    }
                }
            }
        } else {
            for (int i = threadIdx.x; i < kTileRows * 64; i += 256) {
                const int r = i >> 6, c = i & 63;
                const int rank = s_rank[r];
                if (c < channels && rank >= 0 && base + rank < out_capacity)
                    out_feats[(base + rank) * channels + c] = s_v[r][c];
            }
        }
    };

    // (thread 0) the next tile of this workgroup; a launch with a workgroup per tile asks once
    const bool once = (long long)gridDim.x >= n_tiles;
    bool asked = false;
    int dealt = (int)blockIdx.x;  // (STREAM, RANGED) the next tile of this workgroup
    // (RANGED) consecutive tiles, the rows before them known from the counts of the launch before
    int last_own = 0;
    unsigned run = 0;  // (the first wave) the next tile's first output row (31 bits: at most as many as candidates)
    if constexpr (RANGED) {
        const int per = (n_tiles + (int)gridDim.x - 1) / (int)gridDim.x, first_own = (int)blockIdx.x * per;
        last_own = first_own + per < n_tiles ? first_own + per : n_tiles;
        if (first_own >= last_own && blockIdx.x != 0) return;
        dealt = first_own;
        __shared__ unsigned s_sum[4];
        unsigned before = 0;
        for (int i = threadIdx.x; i < (int)blockIdx.x; i += 256) before += counts[i];
        before = wave_add(before);
        if (lane == 0) s_sum[wave] = before;
        __syncthreads();
        run = (s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3]);
        if (last_own == n_tiles && threadIdx.x == 0) {
            const long long rows = (long long)run + (first_own < last_own ? counts[blockIdx.x] : 0u);
            ctr->n_rows = rows;
            write_counters(ctr, rows, nnz_out, aux_imm, aux_is_cand, out_capacity);
        }
    }
    auto next_tile = [&]() -> int {
        if (RANGED) return dealt < last_own ? dealt++ : n_tiles;
        if (STREAM) {
            const int t = dealt < n_tiles ? dealt : n_tiles;
            dealt = t + (int)gridDim.x;
            return t;
        }
        const int t = (once && asked) ? n_tiles : (int)take_ticket(ctr);
        asked = true;
        return t;  // (at or past n_tiles: no tile)
    };
    if (threadIdx.x < 6) s_mask[threadIdx.x >> 1][threadIdx.x & 1] = 0ull;
    if (threadIdx.x == 0) s_ticket = next_tile();
    __syncthreads();
    float va[16][2], vb[16][2];
    // prologue: X = first ticket (loaded, decided), Y = second ticket (loads in flight)
    int tile_x = s_ticket;
    if (tile_x >= n_tiles) {
        finish();
        return;
    }
    load_tile(tile_x, va);
    __syncthreads();  // (the ticket has been read)
    if (threadIdx.x == 0) s_ticket = next_tile();
    decide(tile_x, 0, va);
    __syncthreads();
    int tile_y = s_ticket;
    if (tile_y < n_tiles) load_tile(tile_y, vb);
    if (!STREAM && !RANGED && threadIdx.x == 0)
        publish_count(tile_state, tile_x, __popcll(s_mask[0][0]) + __popcll(s_mask[0][1]));
    int slot_x = 0, slot_y = 1, slot_z = 2;
    // One step: (P, Q) hold (X, Y).  Decide Y, move X to LDS, fetch Z into P's registers, write X.
    auto step = [&](float (&P)[16][2], float (&Q)[16][2]) {
        __syncthreads();  // the previous step's writes are done: s_v, s_base, s_rank, s_ticket and slot_z are free
        if (threadIdx.x == 0) s_ticket = tile_y < n_tiles ? next_tile() : n_tiles;
        if (tile_y < n_tiles) decide(tile_y, slot_y, Q);
        stage_tile(P);
        __syncthreads();  // Y's masks, the ticket and the staged tile are in place
        const int tile_z = s_ticket;
        if (tile_z < n_tiles) load_tile(tile_z, P);  // in flight during the look-back and the writes
        rank_rows(slot_x);
        if (wave == 0) {
            if (lane == 0) {
                s_mask[slot_z][0] = 0ull;  // (last read before this step's first barrier, next used after its last)
                s_mask[slot_z][1] = 0ull;
                if (!STREAM && !RANGED && tile_y < n_tiles)
                    publish_count(tile_state, tile_y, __popcll(s_mask[slot_y][0]) + __popcll(s_mask[slot_y][1]));
            }
            if (RANGED) {
                if (lane == 0) s_base = (long long)run;
                run += (unsigned)(__popcll(s_mask[slot_x][0]) + __popcll(s_mask[slot_x][1]));
            } else if (STREAM) {
                if (lane == 0) s_base = tile_base[tile_x];
            } else {
                const int count = __popcll(s_mask[slot_x][0]) + __popcll(s_mask[slot_x][1]);
                const long long base = lookback_published(tile_state, tile_x, count, ctr);
                if (lane == 0) {
                    if (tile_x == n_tiles - 1)
                        __hip_atomic_store(&ctr->n_rows, base + count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    s_base = base;
                }
            }
        }
        __syncthreads();  // s_base, s_rank
        write_tile(tile_x);
        tile_x = tile_y;
        tile_y = tile_z;
        const int t = slot_x;
        slot_x = slot_y;
        slot_y = slot_z;
        slot_z = t;
    };
    for (;;) {
        step(va, vb);
        if (tile_x >= n_tiles) break;
        step(vb, va);
        if (tile_x >= n_tiles) break;
    }
    finish();
}

// The rows that keep an entry, counted for every workgroup's consecutive tiles, so that k_select_write64 (counts) writes without
// tickets or look-back.  A row is settled by its first channel that survives: four at a time are read, and no further than the
// row of the 64 that takes longest.
__global__ __launch_bounds__(256) void k_select_count64(Geom g, int channels, int mode, int relu,
                                                        const int* __restrict__ cand_start,
                                                        const int* __restrict__ tile_start,
                                                        const float* __restrict__ resp,
                                                        const ColState* __restrict__ cols,
                                                        const Counters* __restrict__ ctr, unsigned* __restrict__ counts) {
    __shared__ unsigned s_cnt[4];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n_tiles = (int)ctr->n_tiles, per = (n_tiles + (int)gridDim.x - 1) / (int)gridDim.x;
    const int first = (int)blockIdx.x * per, last = first + per < n_tiles ? first + per : n_tiles;
    unsigned cnt = 0;
    for (int u = 2 * first + wave; u < 2 * last; u += 4) {  // half tiles
        const int tile = u >> 1;
        const int b = __builtin_amdgcn_readfirstlane(sample_of_tile(tile_start, g.batch, tile));
        const int lt = tile - tile_start[b], r = (u & 1) * 64 + lane;
        const unsigned pos = (unsigned)(lt * kTileRows + r);
        const bool live = (int)pos < cand_start[b + 1] - cand_start[b];
        const float* seg = resp + (size_t)tile * channels * kTileRows + r;
        const ColState* own = cols + (size_t)b * channels;
        bool any = false;
        for (int c0 = 0; c0 < channels; c0 += 4) {
            float x[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = seg[(size_t)(c0 + i < channels ? c0 + i : c0) * kTileRows];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const ColState* st = own + (c0 + i < channels ? c0 + i : c0);
                const unsigned tau = st->tau, cut = st->cut;
                bool keep = score_key(x[i], mode) > (pos <= cut ? tau - (tau != 0u ? 1u : 0u) : tau);
                if (relu) keep = keep && x[i] > 0.0f;
                any |= keep;
            }
            if (__ballot(live && !any) == 0ull) break;  // (uniform)
        }
        cnt += (unsigned)__popcll(__ballot(any && live));
    }
    if (lane == 0) s_cnt[wave] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) counts[blockIdx.x] = s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
}

__global__ void k_finish(const Counters* __restrict__ ctr, int which_rows, long long aux_imm, int aux_is_cand,
                         long long out_capacity, long long* __restrict__ nnz_out) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        const long long rows = which_rows ? ctr->n_pool : ctr->n_rows;
        unsigned flags = ctr->flags;
        if (rows > out_capacity) flags |= SCNN_FLAG_OUT_OVERFLOW;
        nnz_out[0] = rows;
        nnz_out[1] = aux_is_cand ? ctr->n_cand : aux_imm;
        nnz_out[2] = (long long)flags;
        nnz_out[3] = (long long)ctr->bracket_failed;
    }
}

hipError_t launch_finish(const Counters* ctr, int which_rows, long long aux_imm, int aux_is_cand,
                         long long out_capacity, long long* nnz_out, hipStream_t s) {
    hipLaunchKernelGGL(k_finish, dim3(1), dim3(64), 0, s, ctr, which_rows, aux_imm, aux_is_cand, out_capacity,
                       nnz_out);
    return hipGetLastError();
}

// The same pass for narrow layers (at most 32 channels, the widths of the paper's own networks): a tile of 128 rows holds
// too little data to pay for three barriers, so a thread owns a whole row: it reads the row's channels from the planar
// tile (coalesced across the wave), decides them, and writes the row itself.
// Zeroes a row's values that do not survive; any that does?
template <int CMAX>
__device__ __forceinline__ bool decide_row(int channels, int mode, int relu, const ColState* __restrict__ cols, unsigned pos,
                                           float (&v)[CMAX]) {
    bool any = false;
#pragma unroll
    for (int c = 0; c < CMAX; ++c) {
        if (c < channels) {
            const unsigned tau = cols[c].tau, cut = cols[c].cut;
            bool keep = score_key(v[c], mode) > (pos <= cut ? tau - (tau != 0u ? 1u : 0u) : tau);
            if (relu) keep = keep && (v[c] > 0.0f);
            v[c] = keep ? v[c] : 0.0f;
            any |= keep;
        }
    }
    return any;
}

template <int CMAX>
__device__ __forceinline__ void write_row(const Geom& g, int channels, int b, unsigned lin, const float (&v)[CMAX], long long o,
                                          int32_t* __restrict__ out_coords, float* __restrict__ out_feats) {
    int c0, c1, c2;
    site_of(g, lin, c0, c1, c2);
    store_site(g, out_coords + o * (1 + g.ndim), b, c0, c1, c2);
    float* dst = out_feats + o * channels;
    if ((channels & 3) == 0 && ((size_t)out_feats & 15) == 0) {
#pragma unroll
        for (int c = 0; c < CMAX; c += 4)
            if (c < channels) *(float4*)(dst + c) = make_float4(v[c], v[c + 1], v[c + 2], v[c + 3]);
    } else {
#pragma unroll
        for (int c = 0; c < CMAX; ++c)
            if (c < channels) dst[c] = v[c];
    }
}

// Small layers: one launch, two consecutive tiles per workgroup (one status word in tile_state), ordered by tickets and
// look-back; the launch has a workgroup for every two tiles, and those past the layer's leave at once.
template <int CMAX>
__global__ __launch_bounds__(256) void k_select_write_narrow(Geom g, int channels, int mode, int relu,
                                                             const int* __restrict__ cand_start,
                                                             const int* __restrict__ tile_start,
                                                             const unsigned* __restrict__ cand_lin,
                                                             const float* __restrict__ resp,
                                                             const ColState* __restrict__ cols,
                                                             unsigned long long* tile_state, Counters* ctr,
                                                             int32_t* __restrict__ out_coords,
                                                             float* __restrict__ out_feats, long long out_capacity,
                                                             long long* __restrict__ nnz_out, long long aux_imm,
                                                             int aux_is_cand) {
    __shared__ int s_cnt[4];  // kept rows of each wave
    __shared__ int s_ticket;
    __shared__ long long s_base;
    const int n_tiles = (int)ctr->n_tiles, n_super = (n_tiles + 1) / 2;
    if ((int)blockIdx.x >= (n_super > 0 ? n_super : 1)) return;
    if (n_super > 0) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        if (threadIdx.x == 0) s_ticket = (int)take_ticket(ctr);
        __syncthreads();
        const int st = s_ticket, tile = st * 2 + (int)(threadIdx.x >> 7), r = threadIdx.x & (kTileRows - 1);
        float v[CMAX];
        bool keep = false;
        int b = 0, row = 0;
        if (tile < n_tiles) {  // (uniform in the wave)
            b = sample_of_tile(tile_start, g.batch, tile);
            const int lt = tile - tile_start[b];
            row = cand_start[b] + lt * kTileRows + r;
            const float* seg = resp + (size_t)tile * channels * kTileRows + r;
#pragma unroll
            for (int c = 0; c < CMAX; ++c)
                if (c < channels) v[c] = seg[(size_t)c * kTileRows];
            keep = decide_row<CMAX>(channels, mode, relu, cols + (size_t)b * channels, (unsigned)(lt * kTileRows + r), v) &&
                   row < cand_start[b + 1];
        }
        const unsigned long long m = __ballot(keep);
        if (lane == 0) s_cnt[wave] = __popcll(m);
        __syncthreads();
        if (wave == 0) {
            const int total = s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
            const long long base = lookback_wave(tile_state, st, total, ctr);
            if (lane == 0) {
                if (st == n_super - 1)
                    __hip_atomic_store(&ctr->n_rows, base + total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                s_base = base;
            }
        }
        __syncthreads();
        long long o = s_base + __popcll(m & ((1ull << lane) - 1ull));
        for (int w = 0; w < wave; ++w) o += s_cnt[w];
        if (keep && o < out_capacity) write_row<CMAX>(g, channels, b, cand_lin[row], v, o, out_coords, out_feats);
    }
    finish_if_last(ctr, nnz_out, aux_imm, aux_is_cand, out_capacity, n_super > 0 ? n_super : 1);
}

// The pass in two launches, without tickets, look-back or end counters, for narrow layers of more than narrow_pair_tiles
// tiles of capacity: read-modify-writes of one address are served one after the other, and a ticket and an end mark from each of
// several hundred workgroups were half of the one launch's time.  Workgroup i of both launches owns the same consecutive
// tiles.  The first notes the rows that keep an entry (row_keep, two words per tile) and the workgroup's number of them;
// in the second a workgroup adds up the numbers before its own and writes its rows, reading no others; the last one
// writes the result counters.  A wave takes the 64 rows of half a tile at a time.
// 8 channels, us: 128^3 x 4, 5 k tiles 36 -> 9 + 11; 256^3 scattered, 13 k tiles 63 -> 17 + 20; 28 x 28 x 1024, 3 k tiles
// 34 -> 10 + 11; 32^3 x 4, capacity 1028 tiles, 11.8 -> 4.8 + 5.2.  Sixteen channels, 132 tiles: 9.5 against 7.0 + 6.7.
// More than sixteen channels are read twice at a price: one launch against this one, 24 channels, 385 of 561 tiles of
// capacity in use 16.6 against 22.7 us (the stage, by events), 727 / 1039 of 1056 23.6 / 28.7 against 23.9 / 27.5, 1092 /
// 1559 of 1584 30.1 / 39.4 against 26.4 / 31.0; 32 channels 19.1 against 26.1, 25.4 / 33.1 against 27.7 / 32.9, 33.5 / 44.6
// against 31.1 / 37.0: hence a later line for them.  There a workgroup also owns an even number of tiles: its four waves take
// two at a time, and three took as long as four (2092 tiles, 32 channels, 56.9 -> 44.6 us, 24 channels 46.5 -> 34.4; the
// launch has half as many workgroups again for it).
constexpr long long narrow_pair_tiles(int cmax) { return cmax > 16 ? 1152 : 512; }
template <int CMAX>
__device__ inline int tiles_per_workgroup(int n_tiles) {
    if constexpr (CMAX <= 16) return (n_tiles + (int)gridDim.x - 1) / (int)gridDim.x;
    const int n = (int)gridDim.x, most = n - n / 3, per = (n_tiles + most - 1) / most, even = per & ~1;
    return even > 0 && (long long)even * n >= n_tiles ? even : per;
}

template <int CMAX>
__global__ __launch_bounds__(256) void k_select_rows_narrow(Geom g, int channels, int mode, int relu,
                                                            const int* __restrict__ cand_start,
                                                            const int* __restrict__ tile_start,
                                                            const float* __restrict__ resp,
                                                            const ColState* __restrict__ cols,
                                                            const Counters* __restrict__ ctr,
                                                            unsigned long long* __restrict__ row_keep,
                                                            unsigned* __restrict__ counts) {
    __shared__ unsigned s_cnt[4];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n_tiles = (int)ctr->n_tiles, per = tiles_per_workgroup<CMAX>(n_tiles);
    const int first = (int)blockIdx.x * per, last = first + per < n_tiles ? first + per : n_tiles;
    unsigned cnt = 0;
    for (int u = 2 * first + wave; u < 2 * last; u += 4) {
        const int tile = u >> 1;
        const int b = __builtin_amdgcn_readfirstlane(sample_of_tile(tile_start, g.batch, tile));
        const int lt = tile - tile_start[b], r = (u & 1) * 64 + lane;
        const bool live = lt * kTileRows + r < cand_start[b + 1] - cand_start[b];
        const float* seg = resp + (size_t)tile * channels * kTileRows + r;
        float v[CMAX];
#pragma unroll
        for (int c = 0; c < CMAX; ++c)
            if (c < channels) v[c] = seg[(size_t)c * kTileRows];
        const bool any = decide_row<CMAX>(channels, mode, relu, cols + (size_t)b * channels, (unsigned)(lt * kTileRows + r), v);
        const unsigned long long m = __ballot(any && live);
        if (lane == 0) row_keep[u] = m;
        cnt += (unsigned)__popcll(m);
    }
    if (lane == 0) s_cnt[wave] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) counts[blockIdx.x] = s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
}

template <int CMAX>
__global__ __launch_bounds__(256) void k_select_emit_narrow(Geom g, int channels, int mode, int relu,
                                                            const int* __restrict__ cand_start,
                                                            const int* __restrict__ tile_start,
                                                            const unsigned* __restrict__ cand_lin,
                                                            const float* __restrict__ resp,
                                                            const ColState* __restrict__ cols, Counters* ctr,
                                                            const unsigned long long* __restrict__ row_keep,
                                                            const unsigned* __restrict__ counts,
                                                            int32_t* __restrict__ out_coords,
                                                            float* __restrict__ out_feats, long long out_capacity,
                                                            long long* __restrict__ nnz_out, long long aux_imm,
                                                            int aux_is_cand) {
    __shared__ unsigned s_sum[4];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n_tiles = (int)ctr->n_tiles, per = tiles_per_workgroup<CMAX>(n_tiles);
    const int first = (int)blockIdx.x * per, last = first + per < n_tiles ? first + per : n_tiles;
    if (first >= last && blockIdx.x != 0) return;
    unsigned before = 0;  // rows of the workgroups before this one (31 bits: at most as many as candidates)
    for (int i = threadIdx.x; i < (int)blockIdx.x; i += 256) before += counts[i];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) before += __shfl_xor(before, d, 64);
    if (lane == 0) s_sum[wave] = before;
    __syncthreads();
    unsigned base = s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3];
    if (last == n_tiles && threadIdx.x == 0) {
        const long long rows = (long long)base + (first < last ? counts[blockIdx.x] : 0u);
        ctr->n_rows = rows;
        write_counters(ctr, rows, nnz_out, aux_imm, aux_is_cand, out_capacity);
    }
    for (int u0 = 2 * first; u0 < 2 * last; u0 += 64) {  // 64 half tiles at a time: lane j holds the rows before the j-th
        const unsigned long long mine = u0 + lane < 2 * last ? row_keep[u0 + lane] : 0ull;
        unsigned inc = (unsigned)__popcll(mine);
        const unsigned own = inc;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const unsigned o = __shfl_up(inc, d, 64);
            if (lane >= d) inc += o;
        }
        const int n = 2 * last - u0 < 64 ? 2 * last - u0 : 64;
        for (int j = wave; j < n; j += 4) {
            const unsigned long long m =
                (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(unsigned)(mine >> 32), j) << 32 |
                (unsigned)__builtin_amdgcn_readlane((int)(unsigned)mine, j);
            if (m == 0ull) continue;
            const long long o = (long long)(base + (unsigned)__builtin_amdgcn_readlane((int)(inc - own), j)) +
                                __popcll(m & ((1ull << lane) - 1ull));
            if (!((m >> lane) & 1ull) || o >= out_capacity) continue;
            const int u = u0 + j, tile = u >> 1;
            const int b = __builtin_amdgcn_readfirstlane(sample_of_tile(tile_start, g.batch, tile));
            const int lt = tile - tile_start[b], r = (u & 1) * 64 + lane;
            const float* seg = resp + (size_t)tile * channels * kTileRows + r;
            const unsigned lin = cand_lin[cand_start[b] + lt * kTileRows + r];
            float v[CMAX];
#pragma unroll
            for (int c = 0; c < CMAX; ++c)
                if (c < channels) v[c] = seg[(size_t)c * kTileRows];
            (void)decide_row<CMAX>(channels, mode, relu, cols + (size_t)b * channels, (unsigned)(lt * kTileRows + r), v);
            write_row<CMAX>(g, channels, b, lin, v, o, out_coords, out_feats);
        }
        base += (unsigned)__builtin_amdgcn_readlane((int)inc, 63);
    }
}

constexpr long long kCountedTiles = 2048, kCountedPlainTiles = 256;
hipError_t launch_select_write(const Geom& g, int channels, int mode, int relu, const int* cand_start,
                               const int* tile_start, const unsigned* cand_lin, const float* resp,
                               const ColState* cols, unsigned long long* tile_state, long long tiles_cap,
                               Counters* ctr, int32_t* out_coords, float* out_feats, long long out_capacity,
                               long long* nnz_out, long long aux_imm, int aux_is_cand, unsigned long long* row_keep,
                               const long long* tile_base, int keeps_all, hipStream_t s) {
    // no more workgroups than can be resident at once (4 per CU by LDS), so that every ticket holder runs; three per
    // CU measured best for the wide kernels (cfg 4: 103 us against 107 with four and 110 with two)
    const long long cus = device_cu_count();
    long long blocks = tiles_cap < 1 ? 1 : (tiles_cap > cus * 3 ? cus * 3 : tiles_cap);
#define SCNN_NARROW_CASE(CMAX_)                                                                                   \
    do {                                                                                                          \
        if (tiles_cap > narrow_pair_tiles(CMAX_)) {                                                               \
            const long long most = cus * (CMAX_ > 16 ? 6 : 4);                                                    \
            const unsigned grid = (unsigned)(tiles_cap > most ? most : tiles_cap);                                \
            unsigned* counts = (unsigned*)tile_state;                                                             \
            hipLaunchKernelGGL(k_select_rows_narrow<CMAX_>, dim3(grid), dim3(256), 0, s, g, channels, mode, relu, \
                               cand_start, tile_start, resp, cols, ctr, row_keep, counts);                        \
            hipLaunchKernelGGL(k_select_emit_narrow<CMAX_>, dim3(grid), dim3(256), 0, s, g, channels, mode, relu, \
                               cand_start, tile_start, cand_lin, resp, cols, ctr, row_keep, counts, out_coords,   \
                               out_feats, out_capacity, nnz_out, aux_imm, aux_is_cand);                           \
        } else                                                                                                    \
            hipLaunchKernelGGL(k_select_write_narrow<CMAX_>, dim3((unsigned)(tiles_cap < 1 ? 1 : (tiles_cap + 1) / 2)), \
                               dim3(256), 0, s, g, channels, mode, relu, cand_start, tile_start, cand_lin, resp,  \
                               cols, tile_state, ctr, out_coords, out_feats, out_capacity, nnz_out, aux_imm,      \
                               aux_is_cand);                                                                      \
    } while (0)
    if (channels <= 4) SCNN_NARROW_CASE(4);
    else if (channels <= 8) SCNN_NARROW_CASE(8);
    else if (channels <= 16) SCNN_NARROW_CASE(16);
    else if (channels <= 32 && !tile_base) SCNN_NARROW_CASE(32);  // (with tile_base: the streaming kernel below)
    else if (channels <= 64) {
        // (streaming: four workgroups per CU; by look-back three measured best, and four cost it 5 %, which only the
        // rare launch that was given tile_base and cannot use it pays)
        if (tile_base) blocks = tiles_cap < 1 ? 1 : (tiles_cap > cus * 4 ? cus * 4 : tiles_cap);
        // Without the selection's marks: counted first on layers of many tiles, and where nothing is selected, a row being settled
        // by its first channel then, on all but small ones.  Whole calls, us, look-back against counted: plain, 33 to 64 channels,
        // 15 / 65 / 134 / 199 / 257 / 396 / 794 tiles of capacity, 34 / 38 / 46 / 51 / 53 / 69 / 85 against 36 / 40 / 47 / 51 / 53 /
        // 66 / 75 (the launch that counts is 4 us), 53 x 75 x 94 x 3 148 against 131; a tenth selected, 32 -> 64 on surfaces, 32^3 x 2,
        // 200 tiles, 99 -> 112, x 6, 570 tiles (1540 of capacity), 142 -> 147, x 16, 1500 tiles, 216 -> 209, 33 channels 198 -> 180
        const bool ranged = !tile_base && (tiles_cap > kCountedTiles || (keeps_all && tiles_cap > kCountedPlainTiles));
        if (ranged) blocks = tiles_cap < 1 ? 1 : (tiles_cap > cus * 4 ? cus * 4 : tiles_cap);
        const unsigned* counts = (const unsigned*)tile_state;
#define SCNN_WRITE64(RANGED)                                                                                           \
    hipLaunchKernelGGL(k_select_write64<RANGED>, dim3((unsigned)blocks), dim3(256), 0, s, g, channels, mode, relu,     \
                       cand_start, tile_start, cand_lin, resp, cols, tile_state, ctr, out_coords, out_feats,           \
                       out_capacity, nnz_out, aux_imm, aux_is_cand, tile_base, counts)
        if (ranged) {
            hipLaunchKernelGGL(k_select_count64, dim3((unsigned)blocks), dim3(256), 0, s, g, channels, mode, relu, cand_start,
                               tile_start, resp, cols, ctr, (unsigned*)tile_state);
            SCNN_WRITE64(true);
        } else {
            SCNN_WRITE64(false);
        }
#undef SCNN_WRITE64
    } else
        hipLaunchKernelGGL(k_select_write, dim3((unsigned)blocks), dim3(256), 0, s, g, channels, mode, relu,
                           cand_start, tile_start, cand_lin, resp, cols, tile_state, ctr, out_coords, out_feats,
                           out_capacity, nnz_out, aux_imm, aux_is_cand);
#undef SCNN_NARROW_CASE
    return hipGetLastError();
}

}  // namespace scnn
