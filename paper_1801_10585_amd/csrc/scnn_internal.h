// Internal declarations shared by the HIP translation units of libscnn.
// gfx950 only: 64-wide wavefronts, 64-bit ballots, 64-bit occupancy words.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/scnn.h"

namespace scnn {

constexpr int kTileRows = 128;    // candidate sites per response tile
constexpr int kHistBins = 2048;   // bins per radix-select pass (11-bit digits)
constexpr int kScanChunk = 2048;  // elements per block in the device scan
// matrix-core pair lists: pair = (local row of the tile << 24) | row of the other operand
constexpr unsigned kPairRowShift = 24;
constexpr unsigned kPairInMask = (1u << kPairRowShift) - 1u;

// Grid geometry, passed by value to kernels.
struct Geom {
    int ndim;
    int batch;
    int E[3];          // extent, unused axes = 1 (axis order: c_1 slowest .. c_ndim fastest)
    int K[3];          // filter size per axis, unused = 1
    int H[3];          // (K-1)/2
    int T;             // taps = prod(K)
    long long N;       // sites per sample
    long long Npad;    // N rounded up to a multiple of 64
    int Wps;           // 64-bit occupancy words per sample = Npad / 64
};

// One per (sample, channel) column of the response matrix.
struct ColState {
    unsigned tau;       // threshold key: the k-th strongest key of the column
    unsigned cut;       // entries equal to tau survive up to this position in the column (0xffffffff: all of them)
    unsigned tau_lo;    // bracket expected to hold tau, from a sample of the column: keys in [tau_lo, tau_hi] go to the
    unsigned tau_hi;    //   side buffer, keys above tau_hi are only counted
    unsigned n_nz;      // non-zero entries in the column
    unsigned n_above;   // entries above the bracket
    unsigned side_fill; // side-buffer entries written so far
    int done;           // 1 = tau and cut are final
    unsigned long long side_off;  // first side-buffer entry of the column
};

constexpr int kTicketStride = 32;  // 32-bit words between two ticket counters
// Accelerator dies (XCDs) of the part the tile orders are laid out for: MI355X has eight, each with its own L2, and
// deals the workgroups of a launch out to them in turn (workgroup i runs on XCD i % kXcds).  On a part that is
// partitioned differently the orders are still correct, the spans just stop matching the L2s.
constexpr int kXcds = 8;

// Device-resident counters produced on the way.
struct Counters {
    long long n_cand;     // candidate sites
    long long n_tiles;    // response tiles (each sample padded to a multiple of kTileRows)
    long long n_rows;     // rows after selection / ReLU
    long long n_pool;     // rows after pooling
    unsigned flags;       // SCNN_FLAG_*
    int any_tie;          // some column needs tie ranks
    unsigned finished;    // workgroups of the compaction pass that have ended
    unsigned ticket;      // next tile of the compaction pass
    unsigned bracket_failed;  // some column's threshold lay outside its sampled bracket
    unsigned cols_done;       // columns whose selection has ended
    unsigned odd;             // a row or weight of a split kernel is not split_exact
    // tiles handed out so far in each of the contraction kernels' tile spans (one per XCD); one counter per 128-byte line:
    // read-modify-writes on one line are served one after the other, whichever word they address
    // (two sets: the quad kernel runs once per group of 64 output channels, up to two groups)
    unsigned conv_ticket[2 * kXcds * kTicketStride];
};

__host__ __device__ inline long long round_up(long long x, long long m) { return (x + m - 1) / m * m; }

// Compute units of the current device (asked once per device; 256, the part the launch shapes were tuned on, if the
// runtime will not say).  The persistent kernels size their grids from it.
int device_cu_count();

__device__ inline long long lin_of(const Geom& g, int c0, int c1, int c2) {
    // unused leading axes have extent 1 and coordinate 0
    return ((long long)c0 * g.E[1] + c1) * g.E[2] + c2;
}

__device__ inline void site_of(const Geom& g, long long lin, int& c0, int& c1, int& c2) {
    c2 = (int)(lin % g.E[2]);
    lin /= g.E[2];
    c1 = (int)(lin % g.E[1]);
    c0 = (int)(lin / g.E[1]);
}
// The same for a site index inside one sample, which fits 32 bits (the candidate lists hold these): two 32-bit
// divisions instead of two 64-bit ones, which cost several times as many instructions.
__device__ inline void site_of(const Geom& g, unsigned lin, int& c0, int& c1, int& c2) {
    const unsigned e2 = (unsigned)g.E[2], e1 = (unsigned)g.E[1];
    const unsigned q = lin / e2;
    c2 = (int)(lin - q * e2);
    const unsigned q1 = q / e1;
    c1 = (int)(q - q1 * e1);
    c0 = (int)q1;
}

// coords rows are (b, c_1..c_ndim); internally sites always use three axes with
// the real axes right-aligned (2-D: axis 0 has extent 1).
__device__ inline void load_site(const Geom& g, const int32_t* row, int& b, int& c0, int& c1, int& c2) {
    b = row[0];
    if (g.ndim == 3) {
        c0 = row[1]; c1 = row[2]; c2 = row[3];
    } else {
        c0 = 0; c1 = row[1]; c2 = row[2];
    }
}

__device__ inline void store_site(const Geom& g, int32_t* row, int b, int c0, int c1, int c2) {
    row[0] = b;
    if (g.ndim == 3) {
        row[1] = c0; row[2] = c1; row[3] = c2;
    } else {
        row[1] = c1; row[2] = c2;
    }
}

__device__ inline bool site_in_grid(const Geom& g, int b, int c0, int c1, int c2) {
    return (unsigned)b < (unsigned)g.batch && (unsigned)c0 < (unsigned)g.E[0] && (unsigned)c1 < (unsigned)g.E[1] &&
           (unsigned)c2 < (unsigned)g.E[2];
}

// Order-preserving key of a response: larger key = stronger response.
// 0 is reserved for "not an entry".
__device__ inline unsigned score_key(float v, int mode) {
    unsigned u = __float_as_uint(v);
    if ((u & 0x7fffffffu) == 0u) return 0u;
    if (mode == SCNN_TOPK_ABS) return u & 0x7fffffffu;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Locate the sample of a tile: tile_start[b] <= tile < tile_start[b+1].
__device__ inline int sample_of_tile(const int* tile_start, int batch, int tile) {
    int lo = 0, hi = batch - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (tile_start[mid] <= tile) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Row index of the occupied site (b, c0, c1, c2), or -1: the inverse of get_update_id.
__device__ inline int lookup_row(const Geom& g, const unsigned long long* __restrict__ occ,
                                 const unsigned* __restrict__ occ_prefix, long long nnz_in, int b, int c0, int c1,
                                 int c2) {
    if (!site_in_grid(g, b, c0, c1, c2)) return -1;
    const long long key = (long long)b * g.Npad + lin_of(g, c0, c1, c2);
    const unsigned long long word = occ[key >> 6];
    const int bit = (int)(key & 63);
    if (!((word >> bit) & 1ull)) return -1;
    const long long row = (long long)occ_prefix[key >> 6] + __popcll(word & ((1ull << bit) - 1ull));
    return row < nnz_in ? (int)row : -1;  // only an unsorted input can trip this guard
}

// Taps k_lo <= k < k_hi of 0 .. count-1 have their site c2 + off + k on a line of `extent` sites (k_hi <= k_lo: none has).
// A line can hold 2^31 - 1 sites, so no sum here goes past its ends: taps and offsets stay below 64, and c2 and extent are
// only compared, or subtracted from something not smaller in sign.
__device__ __forceinline__ void taps_on_line(int extent, int c2, int off, int count, int& k_lo, int& k_hi) {
    k_lo = max(max(-off, 0) - c2, 0);
    k_hi = min(extent - c2, count + off) - off;
}

// Neighbour rows of one site along one filter line: the taps (t0, t1, t2_lo .. t2_lo + count - 1), count <= 32, look
// at the sites (c0 + t0 - H0, c1 + t1 - H1, c2 + t2 - H2), which are adjacent along the last axis and therefore sit
// in at most two adjacent 64-bit words of the occupancy bitmap.  Both words and their prefixes are loaded once and
// every tap of the line is resolved from them: emit(k, row) is called for k = 0 .. count-1 (count <= 32) with the
// neighbour's row or -1; bit k of `act`: tap t2_lo + k has a non-zero weight.  `live` = false (a padding lane) emits -1
// everywhere without touching memory contents that matter.
// Vector issue is what the callers are bound by, so the line's occupancy is cut out of the two words once, as 32 bits,
// and the rows, which are consecutive along a line, are counted up with it: five instructions a tap.
// 32-bit arithmetic throughout: site, row and bitmap word indices fit 31 bits.
template <typename Emit>
__device__ inline void lookup_line(const Geom& g, const unsigned long long* __restrict__ occ,
                                   const unsigned* __restrict__ occ_prefix, long long nnz_in, bool live, int b, int c0,
                                   int c1, int c2, int t0, int t1, int t2_lo, int count, unsigned act, Emit&& emit) {
    const int q0 = c0 + t0 - g.H[0], q1 = c1 + t1 - g.H[1];
    const bool line_ok = live && (unsigned)b < (unsigned)g.batch && (unsigned)q0 < (unsigned)g.E[0] &&
                         (unsigned)q1 < (unsigned)g.E[1];
    const int off = t2_lo - g.H[2];                               // site of tap k is c2 + off + k
    int k_lo, k_hi;
    taps_on_line(g.E[2], c2, off, count, k_lo, k_hi);
    const unsigned first_bit = line_ok ? (unsigned)((q0 * g.E[1] + q1) * g.E[2]) + (unsigned)c2 + (unsigned)(off + k_lo) : 0u;
    const unsigned p = first_bit & 63u;                           // position of tap k_lo's site in word_a
    const unsigned w_last = (unsigned)g.batch * (unsigned)g.Wps - 1u;
    const unsigned w0 = (unsigned)b * (unsigned)g.Wps + (first_bit >> 6);
    const unsigned wa = line_ok ? (w0 < w_last ? w0 : w_last) : 0u, wb = wa < w_last ? wa + 1u : wa;
    const unsigned long long word_a = occ[wa], word_b = occ[wb];
    const unsigned pre_a = occ_prefix[wa], pre_b = occ_prefix[wb];
    const unsigned window = (unsigned)(word_a >> p) | (unsigned)((word_b << 1) << (63u - p));
    const int n_on = k_hi - k_lo;  // taps whose site is on the line
    const unsigned raw = line_ok && n_on > 0 ? (window & (~0u >> (32 - n_on))) << k_lo : 0u;
    const unsigned win = raw & act;
    // rows count up from those of word_a before the line's first site, or, where word_a is empty (its row prefix then
    // means nothing), from the first of word_b
    unsigned row = word_a ? pre_a + (unsigned)__popcll(word_a & ((1ull << p) - 1ull)) : pre_b;
    for (int k = 0; k < count; ++k) {
        // (only an unsorted input can trip the guard)
        emit(k, ((win >> k) & 1u) && row < (unsigned)nnz_in ? (int)row : -1);
        row += (raw >> k) & 1u;
    }
}

// Bit k = tap_active[first + k] is not zero, k < count <= 32.  (whole wave)
__device__ inline unsigned active_taps(const int* __restrict__ tap_active, int first, int count) {
    const int lane = threadIdx.x & 63;
    return (unsigned)__ballot(lane < count && tap_active[first + (lane < count ? lane : 0)] != 0);
}

// Bits destined for a bitmap, one (word index, bits) per lane, where lanes that address the same word sit next to
// each other (rows sorted by site): OR the bits of each run of equal words into its first lane and report whether
// this lane is such a first lane.  Lanes with nothing to contribute pass a word index no other lane uses (negative).
// Every lane of the wave must call it.
__device__ inline bool wave_or_runs(long long word, unsigned long long& bits) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const long long ow = __shfl_down(word, d, 64);
        const unsigned long long ob = __shfl_down(bits, d, 64);
        if (lane + d < 64 && ow == word) bits |= ob;
    }
    const long long pw = __shfl_up(word, 1, 64);
    return lane == 0 || pw != word;
}

// Values that the split kernels multiply as three bf16 numbers: 0 and the magnitudes from 2^-109 (below, the third number
// runs into bf16's smallest) up to 2^58 (sums of 2^10 products stay below 2^127).  A call with any other row or weight -
// infinities and NaN among them, of which the parts' products would make NaN - multiplies in fp32 instead.
constexpr unsigned kSplitLeast = (127u - 109u) << 23, kSplitEnd = (127u + 58u) << 23;  // (as bits)
__host__ __device__ inline bool split_exact(unsigned bits) {
    const unsigned u = bits & 0x7fffffffu;
    return u == 0 || (u >= kSplitLeast && u < kSplitEnd);
}

constexpr int kTapOdd = 2;  // bit of tap_active: a weight of the tap is not split_exact

// Three bf16 numbers whose sum is x (for those values).
__device__ __forceinline__ void split3(float x, unsigned short& h, unsigned short& m, unsigned short& l) {
    auto rounded = [](float v) {
        const unsigned u = __float_as_uint(v);
        return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
    };
    const unsigned uh = rounded(x);
    const float r1 = x - __uint_as_float(uh << 16);
    const unsigned um = rounded(r1);
    const float r2 = r1 - __uint_as_float(um << 16);
    h = (unsigned short)uh;
    m = (unsigned short)um;
    l = (unsigned short)rounded(r2);
}

// Element (t, ic, oc) of a filter of c_in by c_out channels stored [T][c_in][c_out]; with `adjoint`, of the adjoint
// convolution (back-propagation to the data), whose filter is the stored one, then [T][c_out][c_in], with tap t of the
// adjoint at tap T-1-t (offset negated).
__device__ inline float filter_at(const float* __restrict__ w, int T, int c_in, int c_out, int adjoint, int t, int ic,
                                  int oc) {
    return adjoint ? w[((size_t)(T - 1 - t) * c_out + oc) * c_in + ic] : w[((size_t)t * c_in + ic) * c_out + oc];
}

// Eight fp32 values as eight h, eight m and eight l: split3 on pairs, with the conversion instruction.
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void split8(const u32x4 (&x)[2], u32x4 (&part)[3]) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f32x2 v;
        v.x = __uint_as_float(x[i >> 1][(2 * i) & 3]);
        v.y = __uint_as_float(x[i >> 1][(2 * i + 1) & 3]);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const unsigned p = __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
            part[k][i] = p;
            v.x -= __uint_as_float(p << 16);
            v.y -= __uint_as_float(p & 0xffff0000u);
        }
    }
}

// Products of a 16 x 32 by 32 x 16 block of split operands (parts h, m, l): six of the nine, each exact, as two fp32 sums.
// x_h w_h is summed by itself and the five small ones, smallest first, by themselves; one fp32 addition then joins them.  (The
// instruction cuts the sum it is given off downwards, whatever its sign, where it aligns it with the products: in one
// chain of six, x_h w_h last, that put every result 6e-9 to 8e-9 below the exact one on average and 3.4e-8 to 3.8e-8 off
// (2-norm), on rows with a sixth of their 32 entries 3.4e-8 where this gives 2.8e-8 and fp32 instructions 4.8e-8, with a
// 32nd of them 3.4e-8, 2.6e-8 and 3.1e-8; one rounding is 2.5e-8.)
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ void split_products(const u32x4 (&x)[3], const u32x4& w_h, const u32x4& w_m, const u32x4& w_l,
                                               f32x4& large, f32x4& small) {
    auto add = [](f32x4& sum, const u32x4& a, const u32x4& b) {
        sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), sum, 0, 0, 0);
    };
    large = small = f32x4{0.f, 0.f, 0.f, 0.f};
    add(large, x[0], w_h);
    add(small, x[2], w_h);
    add(small, x[0], w_l);
    add(small, x[1], w_m);
    add(small, x[1], w_h);
    add(small, x[0], w_m);
}

// Scans and reductions across a wave without the LDS pipe: shuffles are ds_bpermute, of about a hundred clocks a step, where a
// lane shift inside a vector instruction takes eight; a 64-lane scan is six steps.  (whole waves)
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned lane_shift(unsigned v) {  // (0 where the row mask or the row's end has no source)
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ unsigned wave_inclusive_add(unsigned v) {
    v += lane_shift<0x111, 0xf>(v);  // row_shr:1, 2, 4, 8: within rows of sixteen lanes
    v += lane_shift<0x112, 0xf>(v);
    v += lane_shift<0x114, 0xf>(v);
    v += lane_shift<0x118, 0xf>(v);
    v += lane_shift<0x142, 0xa>(v);  // row_bcast:15: the last lane of rows 0 and 2 to rows 1 and 3
    v += lane_shift<0x143, 0xc>(v);  // row_bcast:31: the last lane of the lower half to the upper
    return v;
}
__device__ __forceinline__ unsigned wave_add(unsigned v) { return (unsigned)__builtin_amdgcn_readlane((int)wave_inclusive_add(v), 63); }
__device__ __forceinline__ unsigned wave_max(unsigned v) {
    auto larger = [](unsigned x, unsigned y) { return x > y ? x : y; };
    v = larger(v, lane_shift<0x111, 0xf>(v));
    v = larger(v, lane_shift<0x112, 0xf>(v));
    v = larger(v, lane_shift<0x114, 0xf>(v));
    v = larger(v, lane_shift<0x118, 0xf>(v));
    v = larger(v, lane_shift<0x142, 0xa>(v));
    v = larger(v, lane_shift<0x143, 0xc>(v));
    return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ unsigned wave_min(unsigned v) { return ~wave_max(~v); }

// Exclusive scan across a 256-thread block; `total` receives the block sum.
// Contains __syncthreads(): every thread of the block must call it.
__device__ inline unsigned block_exclusive_scan_256(unsigned v, unsigned* s_wave /*[4], shared*/, unsigned& total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned inc = wave_inclusive_add(v);
    if (lane == 63) s_wave[wave] = inc;
    __syncthreads();
    unsigned base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        unsigned x = s_wave[w];
        if (w < wave) base += x;
        tot += x;
    }
    total = tot;
    __syncthreads();
    return base + inc - v;
}

// Per-sample tile ranges and 16-row group ranges from the per-sample candidate ranges (cand_start[0 .. batch], in
// global memory and visible to the block): tile_start[b] = tiles of all earlier samples, each sample rounded up to
// whole tiles; rows16_start likewise in groups of 16 rows.  Either output may be null.  Returns the number of tiles.
// A scan over the samples, 256 at a time, so that batches of thousands of small samples cost a few rounds rather
// than one thread's walk over all of them.  Contains __syncthreads(): whole block of 256 threads.
__device__ inline int sample_ranges_256(int batch, const int* cand_start, int* tile_start, int* rows16_start,
                                        unsigned* s_wave /*[4], shared*/) {
    unsigned carry_t = 0, carry_r = 0;
    for (int b0 = 0; b0 < batch; b0 += 256) {
        const int b = b0 + (int)threadIdx.x;
        const int n = b < batch ? cand_start[b + 1] - cand_start[b] : 0;
        const unsigned t = (unsigned)((n + kTileRows - 1) / kTileRows), r = (unsigned)((n + 15) / 16);
        unsigned tot_t, tot_r;
        const unsigned et = block_exclusive_scan_256(t, s_wave, tot_t);
        const unsigned er = block_exclusive_scan_256(r, s_wave, tot_r);
        if (b < batch) {
            if (tile_start) tile_start[b] = (int)(carry_t + et);
            if (rows16_start) rows16_start[b] = (int)(carry_r + er);
        }
        carry_t += tot_t;
        carry_r += tot_r;
    }
    if (threadIdx.x == 0) {
        if (tile_start) tile_start[batch] = (int)carry_t;
        if (rows16_start) rows16_start[batch] = (int)carry_r;
    }
    return (int)carry_t;
}

// First row of a sorted row list whose sample index is not below b, by 64 probes at a time.  (whole wave)
__device__ __forceinline__ long long wave_first_row(const int32_t* __restrict__ coords, int stride, long long rows, int b) {
    const int lane = threadIdx.x & 63;
    long long lo = 0, hi = rows;
    while (lo < hi) {
        const long long step = (hi - lo + 63) / 64, at = lo + lane * step;
        const unsigned long long below = __ballot(at < hi && coords[at * stride] < b);
        const int n = ~below ? __builtin_ctzll(~below) : 64;  // probes before the first row that is not below
        const long long top = lo + n * step;
        if (top < hi) hi = top;
        if (n > 0) lo += (n - 1) * step + 1;
    }
    return lo;
}

// Which of the keys that a wave holds (key u of a lane is position 64 u + lane; 0: not an entry) are the k strongest: those
// above tau, and those equal to it up to position `cut`.  Found bit by bit from the top: the largest value that at least k
// keys reach, a compare and a ballot's count per register and bit; a value that exactly k keys reach ends the search (real
// values: after about half the bits).  What a step costs is its chain of scalar instructions and its branches, hence one
// branch a step.  (whole wave)
template <int NU>
__device__ __forceinline__ void wave_threshold(const unsigned (&key)[NU], long long k, unsigned& n_nz, unsigned& tau,
                                               unsigned& cut) {
    const int lane = threadIdx.x & 63;
    auto reach = [&](unsigned at) {
        unsigned n = 0;
#pragma unroll
        for (int u = 0; u < NU; ++u) n += (unsigned)__popcll(__ballot(key[u] >= at));
        return n;
    };
    n_nz = reach(1u);
    cut = 0xffffffffu;
    tau = k <= 0 ? 0xffffffffu : 0u;  // no key is stronger: nothing survives; or fewer entries than k: all do
    const unsigned want = k < 0x7fffffffll ? (unsigned)k : 0x7fffffffu;
    if (k <= 0 || n_nz <= want) return;
    // 1 <= k < n_nz: the k-th strongest key is non-zero
    unsigned bit = 1u << 31, n = 0;
#pragma unroll 1
    do {
        const unsigned at = tau | bit;
        n = reach(at);
        tau = n >= want ? at : tau;
        bit = n == want ? 0u : bit >> 1;
    } while (bit != 0u);
    if (n == want) return;  // (all that reach it: the k-th may be stronger than tau, the next is weaker)
    unsigned left = want - (tau == 0xffffffffu ? 0u : reach(tau + 1u));  // of the entries equal to tau survive
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const unsigned long long m = __ballot(key[u] == tau);
        const unsigned c = (unsigned)__popcll(m);
        if (left >= 1u && left <= c) {  // (uniform) the q-th equal key is in this register: the lane of rank `left`
            const unsigned long long hit =
                __ballot(key[u] == tau && (unsigned)__popcll(m & ((1ull << lane) - 1ull)) + 1u == left);
            cut = (unsigned)u * 64u + (unsigned)(__ffsll((long long)hit) - 1);
            left = 0u;
        } else if (left > c) {
            left -= c;
        }
    }
}

// ---- host-side launchers (one per kernel family), all asynchronous on `s` ----
struct ScanBufs {
    unsigned* block_sums;  // ceil(capacity / kScanChunk) + 1 entries
};

// fill `words` 32-bit words with zero
hipError_t launch_zero(void* p, size_t bytes, hipStream_t s);
hipError_t launch_calibration_copy(void* dst, const void* src, size_t bytes, hipStream_t s);

// In-place exclusive scan of vals[0..n) (n read from *n_dev if n_dev != nullptr, else n_imm; n <= capacity).
// total (if non-null) receives the sum as long long.
hipError_t launch_exclusive_scan(unsigned* vals, long long capacity, long long n_imm, const long long* n_dev,
                                 unsigned* block_sums, long long* total, hipStream_t s);

}  // namespace scnn

// ---------------------------------------------------------------------------
// Launchers implemented in the individual .hip files.
// A count that lives on the device is passed as (n_imm, n_dev): n_dev wins
// when non-null.
// ---------------------------------------------------------------------------
namespace scnn {

// scnn_index.hip
hipError_t launch_index_build(const Geom& g, const int32_t* coords, long long n_imm, const long long* n_dev,
                              long long n_cap, unsigned long long* occ, unsigned* occ_prefix, Counters* ctr,
                              const float* feats /* nullable: rows of a split kernel */, int c_in,
                              unsigned short* xs /* nullable: also split them */, const int* tap_active, hipStream_t s);
hipError_t launch_index_build_pool(const Geom& g, const Geom& gp, const int32_t* coords, const float* feats, int channels,
                                   int rows_have_entries, long long n_imm, const long long* n_dev, long long n_cap,
                                   unsigned long long* occ, unsigned* occ_prefix, unsigned long long* pbits, Counters* ctr,
                                   hipStream_t s);
// wp / wb / wq / ws: the filter in the layout of the vector / fp32 pair-list / fp32 quad / split kernels (of wb, wq and
// ws at most the one that will run is non-null, or both wb and ws; wp is used when all three are null)
hipError_t launch_prepare(const Geom& g, const float* w, int c_in, int c_out, int adjoint, int c_out_pad, double* wp,
                          float* wb, float* wq, unsigned short* ws, int* tap_active, int* tap_coord, void* zero_p,
                          size_t zero_bytes, hipStream_t s);
// chunk_sums: null, or (for more than kEmitSmallWords and at most kEmitMidWords words) counters that receive the
// candidate counts of chunks of 16 words (up to 32768 words) or 256 words (beyond), for launch_cand_emit_mid
hipError_t launch_cand_dilate(const Geom& g, const unsigned long long* occ, const int* tap_active,
                              unsigned long long* cand, unsigned* cand_count, unsigned* chunk_sums, hipStream_t s);
hipError_t launch_popcount(const unsigned long long* bits, long long n_words, unsigned* out, hipStream_t s);
// bitmaps of at most this many words: the emit kernels find their offsets themselves, no scan launch
constexpr long long kEmitSmallWords = 8192;
hipError_t launch_cand_emit_small(const Geom& g, const unsigned long long* cand, const unsigned* cand_count,
                                  long long n_words, unsigned* cand_lin, long long cand_cap, int* cand_start,
                                  int* tile_start, int* rows16_start, Counters* ctr, hipStream_t s);
// up to this many words the candidate list is emitted from per-chunk counts (8192 chunks of 256 words), no scan launch
constexpr int kEmitMidChunks = 8192;
constexpr long long kEmitMidWords = (long long)kEmitMidChunks * 256;
// Lanes that share a bitmap word in the candidate dilation: 16 on small grids, where one lane per word would leave
// most of the chip idle behind a chain of dependent loads (below about half a wave per SIMD), 1 on large grids.  A
// chunk, whose candidates the dilation counts, is what one workgroup of 256 threads covers per step: 16 or 256 words.
// Batches of many small samples (fewer than 256 words each) also take 16, as long as the chunk counts fit: a sample
// then starts at most 15 words into a chunk, and those are the words the emit kernel has to add up per sample.
inline int cand_dilate_lanes(long long n_words, long long words_per_sample) {
    return (n_words <= 32768 || (words_per_sample < 256 && n_words <= 16ll * kEmitMidChunks)) ? 16 : 1;
}
inline int cand_chunk_shift(long long n_words, long long words_per_sample) {
    return cand_dilate_lanes(n_words, words_per_sample) == 16 ? 4 : 8;
}
inline long long cand_chunk_count(long long n_words, long long words_per_sample) {
    const int sh = cand_chunk_shift(n_words, words_per_sample);
    return (n_words + (1ll << sh) - 1) >> sh;
}
hipError_t launch_cand_emit_mid(const Geom& g, const unsigned long long* cand, const unsigned* cand_count,
                                const unsigned* chunk_sums, long long n_words, unsigned* cand_lin, long long cand_cap,
                                int* cand_start, int* tile_start, int* rows16_start, Counters* ctr, hipStream_t s);
hipError_t launch_cand_emit(const Geom& g, const unsigned long long* cand, const unsigned* cand_prefix,
                            long long n_words, unsigned* cand_lin, long long cand_cap, int* cand_start,
                            int* tile_start, int* rows16_start, Counters* ctr, hipStream_t s);

// scnn_conv.hip
hipError_t launch_conv_valu(const Geom& g, const unsigned long long* occ, const unsigned* occ_prefix,
                            long long nnz_in, const float* feats, int c_in, const double* wp, int c_out,
                            int c_out_pad, const float* bias, const int* tap_active, const unsigned* cand_lin,
                            const int* cand_start, const int* tile_start, const Counters* ctr, long long tiles_cap,
                            int spread /* tile i on XCD i % 8, where that can be chosen */, float* resp, hipStream_t s);

bool conv_mfma_supported(const Geom& g, int c_in, int c_out, long long nnz_in);
hipError_t launch_pair_build(const Geom& g, const unsigned long long* occ, const unsigned* occ_prefix,
                             long long nnz_in, const int* tap_active, const int* tap_coord,
                             const unsigned* cand_lin, const int* cand_start, const int* tile_start,
                             const int* rows16_start, Counters* ctr, unsigned* pairs, unsigned short* block_tap,
                             uint2* tile_hdr, long long block_cap, long long tiles_cap,
                             unsigned short* tap_first /* nullable: [tiles][T + 1] first block of each tap */,
                             hipStream_t s);
hipError_t launch_conv_mfma(const Geom& g, long long nnz_in, int only_odd, const float* feats, int c_in, const float* wb, int c_out,
                            const float* bias, const unsigned* pairs, const unsigned short* block_tap,
                            const uint2* tile_hdr, Counters* ctr, float* resp, hipStream_t s);
// (on split operands; w = the filter as it is; leave_odd: leaves a call with such values to launch_conv_mfma with only_odd,
// and does not read w)
hipError_t launch_conv_mfma_split(const Geom& g, long long nnz_in, const float* feats, int c_in, const unsigned short* ws,
                                  const float* w, int leave_odd, int c_out, const float* bias, const unsigned* pairs,
                                  const unsigned short* block_tap, const uint2* tile_hdr, Counters* ctr, float* resp,
                                  hipStream_t s);

// scnn_conv_quad.hip
constexpr int kQuadMaxCout = 128;  // two groups of 64 output channels, one launch each
// floats of the quad kernel's filter per group of 64 output channels: [tap][32-channel chunk][2048]
__host__ __device__ inline size_t quad_filter_floats(int taps, int c_in) { return (size_t)taps * ((c_in + 31) / 32) * 2048; }
inline int quad_groups(int c_out) { return (c_out + 63) / 64; }
bool conv_quad_supported(const Geom& g, int c_in, int c_out, long long nnz_in);
hipError_t launch_conv_quad(const Geom& g, const unsigned long long* occ, const unsigned* occ_prefix, long long nnz_in,
                            const float* feats, int c_in, const float* wq, int c_out, const float* bias,
                            const int* tap_active, const unsigned* cand_lin, const int* cand_start,
                            const int* tile_start, Counters* ctr, float* resp, int cus, hipStream_t s);

// scnn_conv_split.hip
// bf16 values of the split kernel's filter per group of 64 output channels: [tap][32-channel chunk][part][16 output
// channels][lane][8]; groups of at most 32 output channels use half of it
__host__ __device__ inline size_t split_filter_elems(int taps, int c_in) { return (size_t)taps * ((c_in + 31) / 32) * (3 * 4 * 512); }
bool conv_split_supported(const Geom& g, int c_in, int c_out, long long nnz_in);
hipError_t launch_conv_split(const Geom& g, const unsigned long long* occ, const unsigned* occ_prefix, long long nnz_in,
                             const float* feats, const unsigned short* xs, int c_in, const float* w,
                             const unsigned short* ws, int c_out, const float* bias,
                             const int* tap_active, const unsigned* cand_lin, const int* cand_start,
                             const int* tile_start, Counters* ctr, float* resp, int cus, hipStream_t s);

// scnn_tiny.hip
struct TinySample {  // what a sample's workgroup leaves behind
    int rows;        // output rows
    int cands;       // candidate sites
    unsigned flags;  // SCNN_FLAG_*
    unsigned first;  // where they lie in the staging area
};
// Layers that one workgroup a sample computes whole: can it, and is it the faster way for so many input rows.  The staging
// area (batch > 1) holds as many rows as the input can reach sites: stage_cap.
bool layer_tiny_shape(const Geom& g, int c_in, int c_out);
bool layer_tiny_pays(const Geom& g, int c_in, int c_out, long long rows);
hipError_t launch_layer_tiny(const Geom& g, const Geom& gp, const int32_t* coords, const float* feats, long long n_imm,
                             const long long* n_dev, int c_in, const float* w, const float* bias, int c_out, long long k,
                             int mode, int relu, int pool, long long cand_cap, long long stage_cap, unsigned* stage_lin,
                             float* stage_feats, TinySample* info, int32_t* out_coords, float* out_feats, long long out_capacity,
                             long long* nnz_out, hipStream_t s);

// scnn_bwd.hip
hipError_t launch_bwd_sites(const Geom& g, const int32_t* coords, long long rows, const int* cand_start,
                            unsigned* cand_lin, int* rows16_start, Counters* ctr, hipStream_t s);
hipError_t launch_bwd_data_write(const Geom& g, const float* resp, const float* x, int c_in, const int* cand_start,
                                 const int* tile_start, const Counters* ctr, long long tiles_cap, float* bp_data,
                                 hipStream_t s);
bool bwd_filter_mfma_supported(int c_in, int c_out, long long g_rows);
int bwd_filter_chunks(const Geom& g, int c_in, int c_out, long long tiles_cap, bool mfma);
hipError_t launch_bwd_filter_f64(const Geom& g, const unsigned long long* occ, const unsigned* occ_prefix,
                                  long long g_rows, const float* gf, int c_out, const float* x, int c_in,
                                  const int* tap_active, const unsigned* cand_lin, const int* cand_start,
                                  const int* tile_start, const Counters* ctr, long long tiles_cap, int n_chunks, double* fpart,
                                  hipStream_t s);
hipError_t launch_bwd_filter_mfma(const Geom& g, const float* x, int c_in, const float* gf, int c_out,
                                  const unsigned* pairs, const unsigned short* tap_first, const uint2* tile_hdr,
                                  const int* cand_start, const int* tile_start, const Counters* ctr, int n_chunks,
                                  double* fpart, hipStream_t s);
hipError_t launch_bwd_filter_finish(const double* fpart, int n_chunks, long long n_elem, const float* w,
                                    float* bp_filter, const Counters* ctr, long long nnz_in, long long g_rows,
                                    long long* info, hipStream_t s);

// scnn_train.hip
hipError_t launch_density_regulariser(const float* feats, long long rows_imm, const long long* rows_dev,
                                      long long rows_cap, int channels, double n_total, double rho_up, double o,
                                      double b1, double b2, double lambda, const float* w, long long n_w, float* grad,
                                      unsigned long long* count, double* partial, double* out, hipStream_t s);
hipError_t launch_prune(float* w, unsigned char* warned, long long n, float eps, unsigned long long* counts,
                        hipStream_t s);

// scnn_topk.hip
hipError_t launch_rows_sample_bounds(const Geom& g, const int32_t* coords, long long rows, int* cand_start,
                                     int* tile_start, Counters* ctr, hipStream_t s);
hipError_t launch_rows_to_planar(const Geom& g, const int32_t* coords, const float* feats, int channels,
                                 const int* cand_start, const int* tile_start, const Counters* ctr,
                                 long long tiles_cap, unsigned* cand_lin, float* resp, hipStream_t s);
// Columns short enough for the one-workgroup selection (no sampled bracket, no marked rows).
bool topk_small_columns(const Geom& g);
// Row marks (all three nullable): row_keep, two 64-bit words per tile; row_plane, kMarkPlanes times as much;
// tile_base, one word per tile.  When given, the columns are not small and k > 0, tile_base[t] becomes the output row
// at which tile t starts, unless ctr->bracket_failed is set; launch_select_write must then be given tile_base.
constexpr int kTopkPartWords = 256;  // slices of a column at most
constexpr int kMarkPlanes = 64;  // one per channel where marks are used (up to 64 channels)
// Marks pay from 17 channels on: with fewer, few rows are marked by some channel's strong response and nearly every
// surviving entry of a bracket costs the settling pass an atomic.
constexpr int kMarkMinChannels = 16;
hipError_t launch_topk(const Geom& g, int channels, long long k, int mode, int relu, const int* tile_start,
                       const float* resp, ColState* cols, uint2* side,
                       uint2* part /* kTopkPartWords entries per column */, unsigned long long* row_keep,
                       unsigned long long* row_plane, long long* tile_base, long long tiles_cap, Counters* ctr,
                       hipStream_t s);
hipError_t launch_select_write(const Geom& g, int channels, int mode, int relu, const int* cand_start,
                               const int* tile_start, const unsigned* cand_lin, const float* resp,
                               const ColState* cols, unsigned long long* tile_state, long long tiles_cap,
                               Counters* ctr, int32_t* out_coords, float* out_feats, long long out_capacity,
                               long long* nnz_out /* nullable: also write the result counters */, long long aux_imm,
                               int aux_is_cand, unsigned long long* row_keep /* two words per tile */,
                               const long long* tile_base /* nullable: from launch_topk */,
                               int keeps_all /* every entry survives the selection */, hipStream_t s);

// scnn_rows.hip
hipError_t launch_relu(const Geom& g, const int32_t* coords, const float* feats, long long rows, int channels,
                       unsigned* flags, unsigned* offs, unsigned* scan_block_sums, int32_t* out_coords, float* out_feats,
                       long long out_capacity, Counters* ctr, hipStream_t s);
hipError_t launch_maxpool(const Geom& g, const Geom& gp, const int32_t* coords, const float* feats,
                          long long n_imm, const long long* n_dev, long long n_cap, int channels,
                          int rows_have_entries, unsigned long long* occ, unsigned* occ_prefix, unsigned long long* pbits,
                          unsigned* pprefix, unsigned* scan_block_sums, long long* pool_key, long long pool_cap,
                          int32_t* out_coords, float* out_feats, long long out_capacity, Counters* ctr,
                          long long* nnz_out /* nullable: also write the result counters, as launch_finish would */,
                          long long aux_imm, int aux_is_cand, hipStream_t s);
hipError_t launch_to_dense(const Geom& g, const int32_t* coords, const float* feats, long long rows,
                           const long long* rows_dev, int channels, float* dense, hipStream_t s);
hipError_t launch_validate(const Geom& g, const int32_t* coords, long long rows, Counters* ctr, hipStream_t s);
hipError_t launch_finish(const Counters* ctr, int which_rows /*0 n_rows, 1 n_pool*/, long long aux_imm,
                         int aux_is_cand, long long out_capacity, long long* nnz_out, hipStream_t s);

}  // namespace scnn
