// Kernel of svip_warp_logits: top-k followed by top-p filtering of logits rows (a variant of the
// sampling rows of Algorithms 1, 2 and 4 that the paper does not cover; dropped logits become -inf
// and every other call treats them as tokens of probability zero).
//
// Both filters are thresholds on the logit value, found per row by a radix select over an
// order-preserving 32-bit key of the fp32 logit, most significant digit first (11 + 11 + 10 bits):
//   top-k   select on the COUNT of keys:  tau_k = k-th largest value;
//   top-p   select on the MASS  of keys >= tau_k: the first value, going down, at which the
//           cumulative softmax mass reaches top_p of the mass kept so far.
// Masses are summed as 64-bit fixed-point integers, so a row's thresholds do not depend on the
// order in which workgroup threads reach the histogram.  One workgroup owns a row.  Only the first
// digit is histogrammed over the whole row; the keys of the bin it selects go into a list in LDS
// and the other digits are found there.  Every sweep over the row is a read from memory (the rows
// in flight exceed L2), so the sweeps are few: count + maximum, mass + candidates, candidates of
// the nucleus bin if it is another one, masked copy.  A small top_k skips the histograms: a pivot
// from a sample, one sweep for the candidates above it (which also writes the output when that
// is a different buffer), everything else on the list.  top_p alone does likewise with two sweeps.
#pragma once
#include <type_traits>

#include "row_math.h"

namespace svip {

constexpr int WARP_WG = 1024;              // threads of the workgroup that owns a row
constexpr int WARP_WAVES = WARP_WG / 64;
constexpr int WARP_BINS = 2048;            // histogram bins: digits of up to 11 bits
constexpr int WARP_CAP = 8192;             // keys of one first-digit bin that fit the candidate list
constexpr int WARP_PAIRS = 7168;           // candidates of a shortcut that keeps their indices too
constexpr int DIGIT1_SHIFT = 21;           // first digit = top 11 bits of the key
// Rows from which top_p alone takes its shortcut.  On peaked rows (N(0, s^2), s from 4 to 6.5; top_p 0.9) it saves two
// sweeps for a fixed cost, the select over the list; on flat ones the estimate that turns them away is 1 to 3 us.  us,
// histogram path / shortcut, peaked rows | flat rows:
//   rows of bf16 logits      1 row                  64 rows                544 rows
//     32000           16.9 / 16.9 | 19.3 / 21.7    19.2 / 19.1 | 20.3 / 22.5    45.6 / 43.8 | 49.0 / 54.4
//     50257           22.5 / 20.5 | 26.1 / 28.5    25.0 / 22.3 | 27.7 / 30.1    65.1 / 56.9 | 71.1 / 78.0
//     65536           25.9 / 22.0 | 31.0 / 33.0    31.2 / 24.7 | 32.5 / 34.9    78.1 / 62.3 | 85.7 / 89.7
//     81920           33.1 / 25.3 | 37.5 / 39.5    35.5 / 27.7 | 39.2 / 41.6    92.9 / 71.0 | 103.9 / 108.0
//   rows of fp32 logits
//     50257           25.7 / 22.6 | 28.6 / 30.6    28.2 / 25.8 | 30.7 / 32.6    95.9 / 74.7 | 96.4 / 102.4
//     65536           29.7 / 26.6 | 34.0 / 35.8    35.0 / 28.0 | 36.2 / 38.3   122.6 / 101.0 | 123.5 / 127.0
//     81920           36.8 / 29.2 | 40.6 / 42.7    41.3 / 33.2 | 44.1 / 45.9   148.8 / 117.4 | 151.3 / 155.1
// The estimate's sample is one vector per thread: the shorter the row, the less the saving pays for a row it misjudges, and
// flat rows of 16-bit logits below 65536, of fp32 ones below 98304, would be 1 to 6 % slower than with the histograms.
constexpr int NUCLEUS_MIN_V = 98304;
static_assert(NUCLEUS_MIN_V >= 8 * WARP_WG, "every thread has a whole vector of its own");

struct WarpArgs {
    const void *in;
    void *out;                 // may equal in
    long long seq_stride, row_stride;
    int k;                     // rows per sequence
    int V;
    Scale sc;
    int top_k;                 // 0: filter off
    double top_p;              // >= 1: filter off
    int stream;                // input and output are more than the last-level cache holds (see candidate_sweep)
    float fix_scale;           // weights in [0, 1] are summed as integers in units of 1 / fix_scale
    int *kept;                 // [rows] survivors per row, or nullptr
    int no_shortcut;           // always take the histogram path (for tests and measurements)
    int *routes;               // [rows] what decided the row: 0 the histograms, 1 or 2 a shortcut; or nullptr (for tests)
};

struct WarpLds {
    union {
        struct {
            unsigned list[WARP_CAP];               // the keys of one first-digit bin, or a shortcut's candidates
            unsigned long long hist[WARP_BINS];    // mass per first digit
            unsigned cnt[WARP_BINS];               // keys per first digit
        };
        unsigned pairs[2 * WARP_PAIRS];            // a shortcut's candidates with their indices (no histogram is in use then)
    };
    unsigned long long sub[WARP_BINS];             // measure per later digit while a bin is refined
    unsigned long long wave_tot[WARP_WAVES];
    float wave_max[WARP_WAVES];
    int wave_kept[WARP_WAVES];
    unsigned digit;
    unsigned n_list;
    unsigned long long rem;
    unsigned long long acc;
};
static_assert(sizeof(unsigned[2 * WARP_PAIRS]) == sizeof(unsigned[WARP_CAP]) + sizeof(unsigned long long[WARP_BINS]) + sizeof(unsigned[WARP_BINS]),
              "the pairs take the place of list, hist and cnt");

// Order-preserving key of an fp32 value (-0 and +0 share a key) and the value of a key.
__device__ __forceinline__ unsigned value_key(float v)
{
    unsigned u = __float_as_uint(v);
    u = u == 0x80000000u ? 0u : u;
    return u ^ ((u >> 31) ? 0xFFFFFFFFu : 0x80000000u);
}
__device__ __forceinline__ float key_value(unsigned key)
{
    return __uint_as_float(key ^ ((key >> 31) ? 0x80000000u : 0xFFFFFFFFu));
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ unsigned long long dpp_mov_or_zero_u64(unsigned long long v)
{
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)v, CTRL, ROW_MASK, 0xF, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(v >> 32), CTRL, ROW_MASK, 0xF, true);
    return ((unsigned long long)hi << 32) | lo;
}
// Inclusive prefix sum over the lanes of a wave, as wave_inclusive_sum but on 64-bit integers.
__device__ __forceinline__ unsigned long long wave_inclusive_sum_u64(unsigned long long v)
{
    v += dpp_mov_or_zero_u64<0x111, 0xF>(v);
    v += dpp_mov_or_zero_u64<0x112, 0xF>(v);
    v += dpp_mov_or_zero_u64<0x114, 0xF>(v);
    v += dpp_mov_or_zero_u64<0x118, 0xF>(v);
    v += dpp_mov_or_zero_u64<0x142, 0xA>(v);
    v += dpp_mov_or_zero_u64<0x143, 0xC>(v);
    return v;
}

// Vectors v0, v0 + WARP_WG, .. of a row through the cached path (the row is read several times), all requested at once and
// without a branch between them: every thread loads, those past the end the row's last whole vector.  The vector at the
// end of a row goes element by element; past the end the caller must not look.  last_use: nothing reads the row again.
template <typename DT, int U>
__device__ __forceinline__ void warp_load_batch(const DT *row, int v0, int V, typename RawOf<DT>::type (&r)[U], bool last_use)
{
    constexpr int N = VecOf<DT>::N;
    typedef typename RawOf<DT>::type R;
    const int whole = V / N;
    if (whole > 0) {
        if (last_use) {
            asm volatile("");            // (else the compiler makes one of the two branches, and drops what differs)
#pragma unroll
            for (int u = 0; u < U; ++u) r[u] = load_raw<DT>(row, min(v0 + u * WARP_WG, whole - 1));
            asm volatile("");
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) r[u] = *(reinterpret_cast<const R *>(row) + min(v0 + u * WARP_WG, whole - 1));
        }
    }
    if (V % N != 0) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (v0 + u * WARP_WG == whole) r[u] = load_raw_edge(row, whole, V);
    }
}

// Vector vi of a row through the cached path: a vector wholly
// inside the row as one 16-byte load, the one at the end element by element, -inf past the end.
template <typename DT>
__device__ __forceinline__ typename RawOf<DT>::type warp_load(const DT *row, int vi, int V)
{
    typedef typename RawOf<DT>::type R;
    if ((vi + 1) * VecOf<DT>::N <= V) return *(reinterpret_cast<const R *>(row) + vi);
    return load_raw_edge(row, vi, V);
}

// f(vector index, its N values) for every vector of the row, U loads in flight per thread.  LONG: no branch stands between the loads,
// and no check while all U vectors are whole: 1 row of 128256 bf16 logits, two sweeps, 32.6 us so 27.6; but rows of 32000, one batch per
// thread, are 4 to 8 % slower than with a check for each, and fp32 ones that end in the histograms up to 3 %.
template <typename DT, bool LONG, int U = 4, typename F>
__device__ __forceinline__ void for_each_vector(const DT *row, int V, F f)
{
    constexpr int N = VecOf<DT>::N;
    const int nvec = (V + N - 1) / N, whole = V / N;
    int v0 = threadIdx.x;
    for (; LONG && v0 + (U - 1) * WARP_WG < whole; v0 += U * WARP_WG) {
        typename RawOf<DT>::type r[U];
#pragma unroll
        for (int u = 0; u < U; ++u) r[u] = *(reinterpret_cast<const typename RawOf<DT>::type *>(row) + v0 + u * WARP_WG);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float z[N];
            unpack<DT>(r[u], z);
            f(v0 + u * WARP_WG, z);
        }
    }
    for (; v0 < nvec; v0 += U * WARP_WG) {
        typename RawOf<DT>::type r[U];
        if (LONG) {
            warp_load_batch<DT, U>(row, v0, V, r, false);
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int v = v0 + u * WARP_WG;
                r[u] = warp_load<DT>(row, v < nvec ? v : v0, V);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int v = v0 + u * WARP_WG;
            if (v < nvec) {
                float z[N];
                unpack<DT>(r[u], z);
                f(v, z);
            }
        }
    }
}

// Sources of candidate keys: the whole row, or the list of one first-digit bin.  f(key, value).
template <typename DT, bool LONG>
struct RowSource {
    const DT *row;
    int V;
    template <typename F>
    __device__ __forceinline__ void for_each(F f) const
    {
        for_each_vector<DT, LONG>(row, V, [&](int, const float(&z)[VecOf<DT>::N]) {
#pragma unroll
            for (int e = 0; e < VecOf<DT>::N; ++e) f(value_key(z[e]), z[e]);
        });
    }
};
struct ListSource {
    const unsigned *list;
    unsigned n;
    template <typename F>
    __device__ __forceinline__ void for_each(F f) const
    {
        for (unsigned i = threadIdx.x; i < n; i += WARP_WG) f(list[i], key_value(list[i]));
    }
};

struct CountMeasure {
    __device__ __forceinline__ unsigned long long operator()(float) const { return 1ull; }
};
struct MassMeasure {
    float m;
    Scale sc;
    float fix_hi;              // fix_scale / 2^32
    // w * fix_scale truncated to an integer; fix_scale = 2^s with s >= 32.  The float is split at
    // 2^32 (both parts convert exactly), which is cheaper than a 64-bit conversion.
    __device__ __forceinline__ float weight(float z) const { return exp2_raw(scaled_diff(z, m, sc)); }
    __device__ __forceinline__ unsigned long long operator()(float z) const
    {
        const float t = weight(z) * fix_hi;          // = w * 2^(s - 32), < 2^13
        const unsigned hi = (unsigned)t;
        const unsigned lo = (unsigned)(__builtin_amdgcn_fractf(t) * 4294967296.0f);
        return ((unsigned long long)hi << 32) | lo;
    }
};

// The same masses of many logits, summed in a double of the binade whose last place is the unit: with rounding towards
// zero an addition there truncates the weight to whole units, one conversion and one addition per logit (8.4 cycles of
// issue) instead of two conversions, a fract, two multiplications and a 64-bit integer addition (26).  The rounding mode
// of doubles is the wave's, so nothing else in double precision may stand between begin() and end(); a double holds the
// sum of 2^5 weights with room to spare, and take() then adds it to the total.
struct MassSum {
    double zero;                   // 2^52 units
    unsigned long long units = 0ull;
    __device__ __forceinline__ explicit MassSum(float fix_scale) : zero(4503599627370496.0 / (double)fix_scale) {}
    __device__ __forceinline__ static void begin() { asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 2, 2), 3" ::: "memory"); }
    __device__ __forceinline__ static void end() { asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 2, 2), 0" ::: "memory"); }
    __device__ __forceinline__ static void add(double &acc, float w) { asm volatile("v_add_f64 %0, %0, %1" : "+v"(acc) : "v"((double)w)); }
    __device__ __forceinline__ void take(double acc)
    {
        units += (unsigned long long)__double_as_longlong(acc) - (unsigned long long)__double_as_longlong(zero);
    }
};

// The logits of a stored vector against a threshold key, without widening them: sign-magnitude numbers as two's complement
// ones of the same order, a saturating difference, its sign spread over the element.  A logit is below the threshold
// exactly if its 32-bit key is (so -0 counts as +0; NaN of positive sign is above, of negative sign below everything).
typedef short i16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ i16x2 ordered(i16x2 v) { return v ^ ((v >> 15) & (short)0x7FFF); }
__device__ __forceinline__ int ordered(int v) { return v ^ ((v >> 31) & 0x7FFFFFFF); }
// the 16-bit number from which on the logits of the type are at or above a key of 32 bits, in the order of ordered(); the
// key, as a signed number of the same order, need not be that of a number of the type
__device__ __forceinline__ short lowest_kept(bf16, int o)
{
    // (widened, numbers below zero end in ones and the others in zeros)
    return (short)(o == 0 ? -1 : (o < 0 ? o >> 16 : min((int)(((unsigned)o + 0xFFFFu) >> 16), 32767)));
}
__device__ __forceinline__ short lowest_kept(f16, int o)
{
    const float t = __int_as_float(ordered(o));
    if (o == 0) return -1;
    if (t != t) return (short)(o < 0 ? -32768 : 32767);
    const _Float16 h = (_Float16)t;
    const short k = ordered(i16x2{__builtin_bit_cast(short, h), 0})[0];
    return (float)h < t ? (short)(k + 1) : k;
}
template <typename DT> struct Threshold {
    i16x2 p;
    __device__ __forceinline__ explicit Threshold(unsigned key)
    {
        const short k = lowest_kept(DT{}, (int)(key ^ 0x80000000u));
        p = i16x2{k, k};
    }
    // all bits of the logits below the threshold, for one word of the vector
    __device__ __forceinline__ unsigned below(unsigned word) const
    {
        unsigned m = __builtin_bit_cast(unsigned, __builtin_elementwise_sub_sat(ordered(__builtin_bit_cast(i16x2, word)), p) >> 15);
        asm("" : "+v"(m));                         // (or it becomes a comparison and a select per logit)
        return m;
    }
};
template <> struct Threshold<float> {
    int p;
    __device__ __forceinline__ explicit Threshold(unsigned key) : p((int)(key ^ 0x80000000u)) { p = p == 0 ? -1 : p; }
    __device__ __forceinline__ unsigned below(unsigned word) const
    {
        unsigned m = (unsigned)(__builtin_elementwise_sub_sat(ordered((int)word), p) >> 31);
        asm("" : "+v"(m));
        return m;
    }
};
// The same for 16-bit logits and a threshold whose sign the whole wave branches on, in two or three instructions per word instead of five:
// among the logits of one sign the stored words have the order of the numbers or its reverse, and those of the other sign are all
// above or all below.
template <typename DT> struct SignedThreshold {
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    unsigned p;
    bool negative;                                 // -0 or below; what counts as 0 is at or above -0
    __device__ __forceinline__ explicit SignedThreshold(unsigned key)
    {
        static_assert(VecOf<DT>::N == 8, "16-bit storage");
        const i16x2 o = Threshold<DT>(key).p;
        negative = __builtin_amdgcn_readfirstlane(o[0] < 0);
        p = (unsigned)__builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, o[0] < 0 ? ordered(o) : o));
    }
    __device__ __forceinline__ void below(const u32x4 &w, unsigned (&m)[4]) const
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (negative) {
                const u16x2 d = __builtin_elementwise_sub_sat(__builtin_bit_cast(u16x2, (unsigned)w[i]), __builtin_bit_cast(u16x2, p));
                m[i] = __builtin_bit_cast(unsigned, (u16x2)(u16x2{0, 0} - __builtin_elementwise_min(d, u16x2{1, 1})));
            } else {
                m[i] = __builtin_bit_cast(unsigned, __builtin_elementwise_sub_sat(__builtin_bit_cast(i16x2, (unsigned)w[i]),
                                                                                  __builtin_bit_cast(i16x2, p)) >> 15);
            }
            asm("" : "+v"(m[i]));                  // (or it becomes a comparison and a select per logit)
        }
    }
};
template <typename DT> __device__ __forceinline__ u32x4 neg_inf_words() { return __builtin_bit_cast(u32x4, NegInfVec<DT>::value()); }

template <typename DT> struct StoreBits;
template <> struct StoreBits<float> {
    static __device__ __forceinline__ void one(float *p, float z) { *p = z; }
};
// 16-bit storage: the fp32 values came from the storage type, so converting back is exact.
template <> struct StoreBits<bf16> {
    static __device__ __forceinline__ uint32_t bits(float z) { return __float_as_uint(z) >> 16; }
};
template <> struct StoreBits<f16> {
    static __device__ __forceinline__ uint32_t bits(float z)
    {
        return (uint32_t)__builtin_bit_cast(unsigned short, (_Float16)z);
    }
};
template <typename DT>
__device__ __forceinline__ void store_one(DT *p, float z)
{
    if constexpr (VecOf<DT>::N == 4) StoreBits<DT>::one(p, z);
    else p->bits = (uint16_t)StoreBits<DT>::bits(z);
}
// Vector vi of the output; the one at the end of a row element by element.
template <typename DT>
__device__ __forceinline__ void store_words(DT *dst, int vi, int V, const u32x4 &o, bool past_caches)
{
    constexpr int N = VecOf<DT>::N;
    if ((vi + 1) * N <= V) {
        u32x4 *to = reinterpret_cast<u32x4 *>(dst + (long long)vi * N);
        if (past_caches) {
            asm volatile("");                      // (else the compiler makes one of the two branches, and drops what differs)
            __builtin_nontemporal_store(o, to);
            asm volatile("");
        } else {
            *to = o;
        }
    } else {
        float z[N];
        unpack<DT>(__builtin_bit_cast(typename RawOf<DT>::type, o), z);
#pragma unroll
        for (int e = 0; e < N; ++e)
            if (vi * N + e < V) store_one<DT>(dst + (long long)vi * N + e, z[e]);
    }
}

// Going down from the highest digit over a histogram h[WARP_BINS] in LDS (filled and barriered
// by the caller): the digit d with  sum(h above d) < target <= sum(h at and above d),  and
// rem = target - sum(h above d), the share of the target that falls inside d.  With frac >= 0
// the target is max(1, frac * sum(h)).  rem == 0: the histogram's total falls short of the target.
// Every thread of the workgroup must call it; the result is uniform.
struct Crossing {
    unsigned digit;
    unsigned long long rem;
};
template <typename T>
__device__ __forceinline__ Crossing crossing(const T *h, unsigned long long target, double frac, WarpLds &L)
{
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    // thread t owns the bins 2047 - 2t and 2046 - 2t: highest digits first
    const int b0 = WARP_BINS - 1 - 2 * tid, b1 = b0 - 1;
    const unsigned long long m0 = h[b0], m1 = h[b1];
    const unsigned long long incl = wave_inclusive_sum_u64(m0 + m1);
    if (lane == 63) L.wave_tot[wave] = incl;
    if (tid == 0) {
        L.digit = 0u;
        L.rem = 0ull;
    }
    __syncthreads();
    unsigned long long above = incl - (m0 + m1), total = 0ull;
#pragma unroll
    for (int w = 0; w < WARP_WAVES; ++w) {
        const unsigned long long t = L.wave_tot[w];
        above += w < wave ? t : 0ull;
        total += t;
    }
    if (frac >= 0.0) {
        target = (unsigned long long)llrint(frac * (double)total);
        target = target ? target : 1ull;
    }
    if (above < target && target <= above + m0) {
        L.digit = (unsigned)b0;
        L.rem = target - above;
    } else if (above + m0 < target && target <= above + m0 + m1) {
        L.digit = (unsigned)b1;
        L.rem = target - (above + m0);
    }
    __syncthreads();
    Crossing c;
    c.digit = L.digit;
    c.rem = L.rem;
    __syncthreads();                         // the next call rewrites digit, rem and wave_tot
    return c;
}

// Remaining digits of a select (11, 11 and 10 bits, most significant first) over the candidates of
// src at or above floor_key that carry `prefix` in their top `done` bits (done = 0: all, three
// digits; done = 11: inside first-digit bin `prefix`, two digits): the key v among them with
//   measure(candidates > v) < target <= measure(candidates >= v).
// BITS: the most of a key that the logits' type fills, 32 or, a 16-bit number having at most 19, 22: its last digit need not be looked for,
// and with the bits behind the others at zero a key still stands for its number, as no other number lies between the two.
template <typename DT> constexpr int KEY_BITS = VecOf<DT>::N == 8 ? 22 : 32;
template <int BITS, typename Src, typename Measure>
__device__ __forceinline__ unsigned select_digits(const Src &src, unsigned floor_key, Measure measure, unsigned prefix, int done,
                                  unsigned long long target, WarpLds &L)
{
    const int tid = threadIdx.x;
#pragma unroll 1
    while (done < BITS) {
        const int bits = done < 22 ? 11 : 10;
        const int shift = 32 - done - bits;
        const unsigned mask = (1u << bits) - 1u;
        L.sub[tid] = 0ull;
        L.sub[tid + WARP_WG] = 0ull;
        __syncthreads();
        src.for_each([&](unsigned key, float z) {
            if (key >= floor_key && (done == 0 || (key >> (32 - done)) == prefix))
                atomicAdd(&L.sub[(key >> shift) & mask], measure(z));
        });
        __syncthreads();
        const Crossing c = crossing(L.sub, target, -1.0, L);
        prefix = (prefix << bits) | c.digit;
        if (c.rem == 0ull) return prefix << shift;         // the candidates' measure falls short of the target
        target = c.rem;
        done += bits;
    }
    return prefix << (32 - BITS);
}
template <int BITS, typename Src, typename Measure>
__device__ __forceinline__ unsigned refine(const Src &src, unsigned floor_key, Measure measure, unsigned d1,
                           unsigned long long target, WarpLds &L)
{
    return select_digits<BITS>(src, floor_key, measure, d1, 11, target, L);
}

// Sum over the workgroup of one 64-bit value per thread (uniform result; uses L.acc).
__device__ __forceinline__ unsigned long long wg_sum_u64(unsigned long long mine, WarpLds &L)
{
    if (threadIdx.x == 0) L.acc = 0ull;
    __syncthreads();
    mine = wave_reduce(mine, OpSum{});
    if ((threadIdx.x & 63) == 0 && mine) atomicAdd(&L.acc, mine);
    __syncthreads();
    const unsigned long long r = L.acc;
    __syncthreads();
    return r;
}

// An LDS counter's old value, per lane.  Through atomicAdd() the compiler first adds the lanes' values up one by one, which
// takes longer than the few lanes that have something to add.
__device__ __forceinline__ unsigned lds_add(unsigned *p, unsigned n)
{
    unsigned old;
    const unsigned at = (unsigned)(unsigned long long)(__attribute__((address_space(3))) unsigned *)p;
    asm volatile("ds_add_rtn_u32 %0, %1, %2\n\ts_waitcnt lgkmcnt(0)" : "=&v"(old) : "v"(at), "v"(n) : "memory");
    return old;
}

// One sweep over the row: the keys of the logits at or above the pivot into L.list (n_list counts them, also those that do
// not fit), with `FUSED` their indices behind them (`cap` of each) and the output -- the logit itself at and above the pivot,
// -inf below; and with MASS the total mass of the row (per thread).
// What bounds it is vector-ALU issue: a wave of the nucleus path is active for 103 cycles per logit of its 64 lanes, by counters, in both
// sweeps and the select together (1088 rows of 128256 bf16 logits); with a mass it is 17 of one row's 27 us.  A row's
// chunk of 64 vectors holds some candidates more often than not, so what every logit pays for is kept apart from what a candidate
// does: the comparison works on the stored words, and the lanes that have candidates go through them one at a time.  With a mass, whole
// vectors go without a check, the comparison goes by the pivot's sign and constants stay in vector registers: top-p 0.9, 1 row
// of 128256 bf16 logits 32.7 / 27.7 us, 64 rows 39.0 / 32.4, 1088 rows 178 / 165 (with the select below).
// Tried and dropped: the row held in a workgroup's registers (one read; its phases no longer overlap another row's: 1088 rows 207 us), and
// one sweep relative to a sample's maximum with an approximate total (155 us, but 3 to 9 % more for rows that it cannot decide).
// `stream` (with a mass): for calls that move more than the last-level cache, loads and stores go past the caches, so that
// they keep the rows whose second sweep is still to come.  us, through the
// caches / past them, top_p 0.9 on inputs not used just before | the same input again and again: 1088 rows of 128256 bf16
// logits 211 / 195 | 211 / 178, 685 rows of 151936 158 / 140 | 156 / 126, 256 rows of 151936 fp32 (311 MB in all) 114 / 87 |
// 94 / 84, but 300 rows of 151936 bf16 (182 MB) 96 / 86 | 73 / 85: the line is drawn for inputs that are in the cache already.
// A call that reads the output next finds none of it there: svip_verify behind 1088 rows takes 57 us instead of 47, and the two
// together 280 / 254.  A single sweep gains nothing (top_k 50, 1088 rows 165 / 167); a plain copy does (1088 rows 114 / 110).
template <typename DT, bool FUSED, bool MASS, int U>
__device__ __forceinline__ unsigned long long candidate_sweep(const DT *row, DT *dst, int V, unsigned pivot, unsigned cap, const MassMeasure &mass,
                                                    float fix_scale, bool stream, WarpLds &L)
{
    constexpr int N = VecOf<DT>::N, PER = N / 4;                 // logits per word
    constexpr bool SIGNED = MASS && N == 8;
    const std::conditional_t<SIGNED, SignedThreshold<DT>, Threshold<DT>> pv(pivot);       // (without a mass the branch costs more than it saves)
    u32x4 low = neg_inf_words<DT>();
    if (MASS) asm("" : "+v"(low));                 // (or the masking takes two instructions per word)
    const int nvec = (V + N - 1) / N, whole = V / N;
    MassMeasure measure = mass;
    measure.sc.c_hi = in_vgpr(mass.sc.c_hi);
    measure.sc.c_lo = in_vgpr(mass.sc.c_lo);
    MassSum sum(fix_scale);
    const auto note = [&](const typename RawOf<DT>::type &r, int vi, double &acc, u32x4 &o) {
        if (MASS) {
            float z[N];
            unpack<DT>(r, z);
#pragma unroll
            for (int e = 0; e < N; ++e) MassSum::add(acc, measure.weight(z[e]));
        }
        const u32x4 w = __builtin_bit_cast(u32x4, r);
        unsigned m[4];
        if constexpr (SIGNED) {
            pv.below(w, m);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) m[i] = pv.below(w[i]);
        }
        if ((m[0] & m[1] & m[2] & m[3]) != 0xFFFFFFFFu) {
            unsigned at = 0u;                                    // one bit per candidate
#pragma unroll
            for (int i = 0; i < 4; ++i) at |= (~m[i] & (PER == 2 ? 0x00010001u : 1u)) << (PER * i);
            if (PER == 2) at = (at | (at >> 15)) & 0xFFu;
            unsigned slot = lds_add(&L.n_list, (unsigned)__popc(at));
            while (at) {
                const int e = __ffs((int)at) - 1, i = e / PER;
                at &= at - 1u;
                const unsigned word = i & 2 ? (i & 1 ? w[3] : w[2]) : (i & 1 ? w[1] : w[0]);
                float v;
                if constexpr (PER == 1) v = __uint_as_float(word);
                else v = widen(DT{(uint16_t)(e & 1 ? word >> 16 : word)});
                if (slot < cap) {
                    L.pairs[slot] = value_key(v);
                    if (FUSED) L.pairs[cap + slot] = (unsigned)(vi * N + e);
                }
                ++slot;
            }
        }
        if (FUSED) {
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = (w[i] & ~m[i]) | (low[i] & m[i]);
        }
    };
    const bool last_use = FUSED && stream && MASS;
    if (MASS) MassSum::begin();
    int v0 = threadIdx.x;
    for (; MASS && v0 + (U - 1) * WARP_WG < whole; v0 += U * WARP_WG) {       // whole vectors, without a check
        typedef typename RawOf<DT>::type R;
        R r[U];
        double acc = sum.zero;
        if (last_use) {
            asm volatile("");                      // (else the compiler makes one of the two branches, and drops what differs)
#pragma unroll
            for (int u = 0; u < U; ++u) r[u] = load_raw<DT>(row, v0 + u * WARP_WG);
            asm volatile("");
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) r[u] = *(reinterpret_cast<const R *>(row) + v0 + u * WARP_WG);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            u32x4 o;
            note(r[u], v0 + u * WARP_WG, acc, o);
            if (FUSED) {
                u32x4 *to = reinterpret_cast<u32x4 *>(dst) + v0 + u * WARP_WG;
                if (last_use) {
                    asm volatile("");
                    __builtin_nontemporal_store(o, to);
                    asm volatile("");
                } else {
                    *to = o;
                }
            }
        }
        if (MASS) sum.take(acc);
    }
    for (; v0 < nvec; v0 += U * WARP_WG) {
        typename RawOf<DT>::type r[U];
        double acc = sum.zero;
        if (MASS) {
            warp_load_batch<DT, U>(row, v0, V, r, last_use);
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) r[u] = warp_load<DT>(row, v0 + u * WARP_WG < nvec ? v0 + u * WARP_WG : v0, V);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int vi = v0 + u * WARP_WG;
            if (vi >= nvec) continue;
            u32x4 o;
            note(r[u], vi, acc, o);
            if (FUSED) store_words<DT>(dst, vi, V, o, last_use);
        }
        if (MASS) sum.take(acc);
    }
    if (MASS) MassSum::end();
    return sum.units;
}

// The largest value of the list (uniform; ends behind a barrier).
__device__ __forceinline__ float list_max(const ListSource &ls, WarpLds &L)
{
    float m = neg_inf();
    ls.for_each([&](unsigned, float z) { m = vmax(m, z); });
    m = wave_max(m);
    if ((threadIdx.x & 63) == 0) L.wave_max[threadIdx.x >> 6] = m;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < WARP_WAVES; ++w) m = vmax(m, L.wave_max[w]);
    return m;
}

template <typename DT> constexpr int KEY_LOW = VecOf<DT>::N == 4 ? 0 : 13;       // low bits of a key that are the same in all numbers of one sign
// The key v of the list with  measure(> v) < target <= measure(>= v), as select_digits, for keys between lo and hi: the first digit is as
// fine as 2048 bins over that span are.  The upper digits of the keys themselves put a list into some ten bins, where the atomics of
// as many lanes wait for one another; here 16-bit numbers come one to a bin, mostly, and one digit does.  us, top-k 50 and top-p 0.9 by
// three such digits / so: 1 row of 128256 bf16 logits 29.0 / 22.3, 544 of 32000 51.1 / 35.8, 1088 of 128256 161 / 143; top-k alone 24.1 / 20.3,
// 41.5 / 32.8, 148 / 138.  Keys of fp32 logits take three digits either way.  The low bits that all numbers share are zero in v.
// *rem = target - measure(> v), 0 if the list falls short of the target.
template <typename DT, typename Measure>
__device__ __forceinline__ unsigned select_span(const ListSource &ls, unsigned lo, unsigned hi, Measure measure, unsigned long long target,
                                                unsigned long long *rem, WarpLds &L)
{
    constexpr int LOW = KEY_LOW<DT>;
    const int tid = threadIdx.x;
    unsigned base = lo >> LOW << LOW;
    int shift = 21 - __clz((int)((hi - base) | 1u));              // (hi - base) >> shift < 2048
    if (shift < LOW) shift = LOW;
    unsigned width = 0xFFFFFFFFu;                                 // keys of [base, base + width]
#pragma unroll 1
    for (;;) {
        L.sub[tid] = 0ull;
        L.sub[tid + WARP_WG] = 0ull;
        __syncthreads();
        ls.for_each([&](unsigned key, float z) {
            if (key >= base && key - base <= width) atomicAdd(&L.sub[min((key - base) >> shift, WARP_BINS - 1u)], measure(z));      // (a NaN's is above hi)
        });
        __syncthreads();
        const Crossing c = crossing(L.sub, target, -1.0, L);
        base += c.digit << shift;
        *rem = c.rem;
        if (shift == LOW || c.rem == 0ull) return base;
        width = (1u << shift) - 1u;
        target = c.rem;
        shift = shift - 11 > LOW ? shift - 11 : LOW;
    }
}

// The output behind a sweep that has written it down to its pivot: the candidates below tau become -inf as well.  (The sweep's stores
// are complete: every barrier since waited for them.)  Returns how many logits are kept.
template <typename DT>
__device__ __forceinline__ int drop_candidates(DT *dst, int V, unsigned tau, unsigned n, WarpLds &L)
{
    unsigned long long kept = 0ull;
    for (unsigned i = threadIdx.x; i < n; i += WARP_WG) {
        const unsigned idx = L.pairs[WARP_PAIRS + i];
        if (idx < (unsigned)V) {
            if (L.list[i] >= tau) kept += 1ull;
            else store_one<DT>(dst + idx, neg_inf());
        }
    }
    return (int)wg_sum_u64(kept, L);
}

// Shortcut for a small top_k: a pivot from a sample of the row (one vector per thread), aimed at
// about three times top_k keys above it; one sweep puts every key >= pivot into L.list.  If at
// least top_k keys arrive and all of them fit, the list holds the row's largest keys, the row
// maximum among them, and both thresholds follow from the list alone -- with the same integer
// arithmetic as the histogram path, hence the same result.
// With `fused` (output is not the input, top_k <= 1024) the same sweep already writes the output:
// -inf below the pivot, the logit itself at and above it, and the list also keeps the candidates'
// indices (WARP_PAIRS of each); afterwards only the candidates below the final threshold are overwritten,
// so the row is read once.
// Returns 0: nothing decided (the sample misjudged the row; the caller takes the histogram path,
// which rewrites the whole output), 1: *tau_out is the threshold, 2: output and *kept_out are done.
template <typename DT, bool fused>
__device__ __forceinline__ int small_k_shortcut(const DT *row, DT *dst, int V, const WarpArgs &a, bool P,
                                             unsigned *tau_out, int *kept_out, WarpLds &L)
{
    constexpr int N = VecOf<DT>::N;
    const int tid = threadIdx.x;
    const int nvec = (V + N - 1) / N;
    const int nsamp = nvec < WARP_WG ? nvec : WARP_WG;            // sampled vectors
    constexpr unsigned cap = fused ? WARP_PAIRS : WARP_CAP;
    const long long want = 3ll * a.top_k * ((long long)nsamp * N) / V + 8;
    if (a.top_k > (int)cap / 4 || want > (long long)nsamp * N / 4) return 0;
    if (tid < nsamp) {
        // sixteen evenly spaced runs of 64 consecutive vectors: whole cache lines, spread over the row
        const int vi = nvec <= WARP_WG ? tid : (int)((long long)(tid >> 6) * (nvec - 64) / 15) + (tid & 63);
        float z[N];
        unpack<DT>(warp_load<DT>(row, vi, V), z);
#pragma unroll
        for (int e = 0; e < N; ++e) L.list[tid * N + e] = value_key(z[e]);
    }
    __syncthreads();
    const ListSource sample{L.list, (unsigned)(nsamp * N)};
    const unsigned pivot = select_digits<KEY_BITS<DT>>(sample, 0u, CountMeasure{}, 0u, 0, (unsigned long long)want, L);
    if (tid == 0) L.n_list = 0u;
    __syncthreads();
    candidate_sweep<DT, fused, false, 2>(row, dst, V, pivot, cap, MassMeasure{}, a.fix_scale, a.stream, L);
    __syncthreads();
    const unsigned n = L.n_list;
    __syncthreads();
    if (n < (unsigned)a.top_k || n > cap) return 0;
    const ListSource ls{L.list, n};
    // (fp32 keys take three digits either way)
    const float m = N == 8 || P ? list_max(ls, L) : 0.f;
    unsigned long long rem;
    unsigned tau = N == 8 ? select_span<DT>(ls, pivot, value_key(m), CountMeasure{}, (unsigned long long)a.top_k, &rem, L)
                          : select_digits<32>(ls, 0u, CountMeasure{}, 0u, 0, (unsigned long long)a.top_k, L);
    if (P) {
        const MassMeasure mass{m, a.sc, a.fix_scale * (1.0f / 4294967296.0f)};
        unsigned long long mine = 0ull;
        ls.for_each([&](unsigned key, float z) { mine += key >= tau ? mass(z) : 0ull; });
        const unsigned long long Zk = wg_sum_u64(mine, L);
        unsigned long long target = (unsigned long long)llrint(a.top_p * (double)Zk);
        target = target ? target : 1ull;
        if (Zk >= target) {
            const unsigned tau_p = select_span<DT>(ls, tau, value_key(m), mass, target, &rem, L);
            tau = tau_p > tau ? tau_p : tau;
        }
    }
    *tau_out = tau;
    if (!fused) return 1;
    *kept_out = drop_candidates(dst, V, tau, n, L);
    return 2;
}

// Shortcut for top_p alone.  A row's nucleus is usually some hundreds of tokens; the histogram path finds it with a
// 64-bit LDS atomic for every logit, a further sweep for the keys of one bin and one that copies.  Here
//   sweep 1: every thread's maximum.  The smallest maximum of four threads is the pivot: whatever the row's
//            distribution, about 256 ln 256 = 1600 logits are at or above it; where that will not do the smallest of two
//            threads (about 512 ln 512 = 3500);
//   sweep 2: the keys >= pivot into L.list, the total mass in registers with the same integer arithmetic, hence the same
//            threshold; with `fused` (output is not the input) it also writes the logits >= pivot, -inf below, and
//            afterwards only the candidates below the threshold are overwritten.
// Between the two an estimate tells whether the list will reach top_p of the total: the mass above the pivot is at least
// that of the threads' maxima, and the mass below comes from a sample, which cannot miss much as no logit below the pivot
// outweighs it.  A row that is too flat leaves here with the sweep behind it that the histogram path needs first anyway.
// For rows of at least NUCLEUS_MIN_V logits: every thread has at least one vector in sweep 1 and one in the sample.
// Returns 0: nothing decided (*m_out is the row maximum); 1, 2: as small_k_shortcut.
template <typename DT, bool fused>
__device__ __forceinline__ int nucleus_shortcut(const DT *row, DT *dst, int V, const WarpArgs &a, unsigned *tau_out,
                                             int *kept_out, float *m_out, WarpLds &L)
{
    constexpr int N = VecOf<DT>::N;
    constexpr float LOWEST = -3.402823466e38f;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int nvec = (V + N - 1) / N;
    constexpr unsigned cap = fused ? WARP_PAIRS : WARP_CAP;
    float mine_max = neg_inf();
    for_each_vector<DT, N == 8>(row, V, [&](int, const float(&z)[N]) { mine_max = vmax(mine_max, tree_max<N>(z)); });
    const float pair = vmax(mine_max, __shfl_xor(mine_max, 1));
    const float group = vmax(pair, __shfl_xor(pair, 2));
    // the same runs of whole cache lines as in small_k_shortcut
    const typename RawOf<DT>::type sample = warp_load<DT>(row, (int)((long long)(tid >> 6) * (nvec - 64) / 15) + (tid & 63), V);
    {
        const float hi = wave_max(mine_max), lo4 = -wave_max(-group), lo2 = -wave_max(-pair);
        if (lane == 0) {
            L.wave_max[wave] = hi;
            L.wave_tot[wave] = ((unsigned long long)__float_as_uint(lo2) << 32) | __float_as_uint(lo4);
        }
    }
    if (tid == 0) L.n_list = 0u;
    __syncthreads();
    float m = neg_inf(), pz = neg_inf(), pz2 = neg_inf();
#pragma unroll
    for (int w = 0; w < WARP_WAVES; ++w) {
        m = vmax(m, L.wave_max[w]);
        pz = vmax(pz, -__uint_as_float((unsigned)L.wave_tot[w]));
        pz2 = vmax(pz2, -__uint_as_float((unsigned)(L.wave_tot[w] >> 32)));
    }
    pz = vmax(-pz, LOWEST);                                       // masked logits are no candidates
    pz2 = vmax(-pz2, LOWEST);
    *m_out = m;
    float head = exp2_raw(scaled_diff(mine_max, m, a.sc)), tail = 0.f, tail2 = 0.f;
    float zs[N];
    unpack<DT>(sample, zs);
#pragma unroll
    for (int e = 0; e < N; ++e) {
        const float w = exp2_raw(scaled_diff(zs[e], m, a.sc));
        tail += zs[e] < pz ? w : 0.f;
        tail2 += zs[e] < pz2 ? w : 0.f;
    }
    head = wave_reduce(head, OpSum{});
    tail = wave_reduce(tail, OpSum{});
    tail2 = wave_reduce(tail2, OpSum{});
    if (lane == 0) {
        L.sub[wave] = ((unsigned long long)__float_as_uint(head) << 32) | __float_as_uint(tail);
        L.sub[WARP_WAVES + wave] = __float_as_uint(tail2);
    }
    __syncthreads();
    head = tail = tail2 = 0.f;
#pragma unroll
    for (int w = 0; w < WARP_WAVES; ++w) {
        head += __uint_as_float((unsigned)(L.sub[w] >> 32));
        tail += __uint_as_float((unsigned)L.sub[w]);
        tail2 += __uint_as_float((unsigned)L.sub[WARP_WAVES + w]);
    }
    // a wrong yes costs a sweep, a wrong no the saving: a fifth of the tail allowed is kept as a margin
    const float per = (float)V / (float)(WARP_WG * N) * (float)a.top_p, room = 0.8f * (1.f - (float)a.top_p) * head;
    if (!(room >= per * tail)) {
        if (!(room >= per * tail2)) return 0;
        pz = pz2;
    }
    const MassMeasure mass{m, a.sc, a.fix_scale * (1.0f / 4294967296.0f)};
    unsigned long long mine = candidate_sweep<DT, fused, true, 4>(row, dst, V, value_key(pz), cap, mass, a.fix_scale, a.stream, L);
    const unsigned long long Z = wg_sum_u64(mine, L);             // its barriers also cover the list
    const unsigned n = L.n_list;
    if (n > cap) return 0;
    const ListSource ls{L.list, n};
    unsigned long long target = (unsigned long long)llrint(a.top_p * (double)Z), rem;
    target = target ? target : 1ull;
    const unsigned tau = select_span<DT>(ls, value_key(pz), value_key(m), mass, target, &rem, L);
    if (rem == 0ull) return 0;                                    // the list falls short of it
    *tau_out = tau;
    if (!fused) return 1;
    *kept_out = drop_candidates(dst, V, tau, n, L);
    return 2;
}

// The output: the logits whose keys are at or above tau, -inf for the others.  Returns how many this thread kept.
template <typename DT, int U = 4>
__device__ __forceinline__ int masked_copy(const DT *row, DT *dst, int V, unsigned tau, bool stream)
{
    constexpr int N = VecOf<DT>::N, BITS = 128 / N;
    const Threshold<DT> th(tau);
    const u32x4 low = neg_inf_words<DT>();
    const int nvec = (V + N - 1) / N;
    int bits = 0;                                                // of the logits kept
    for (int v0 = threadIdx.x; v0 < nvec; v0 += U * WARP_WG) {
        typename RawOf<DT>::type r[U];
        warp_load_batch<DT, U>(row, v0, V, r, stream);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int vi = v0 + u * WARP_WG;
            if (vi >= nvec) continue;
            const u32x4 w = __builtin_bit_cast(u32x4, r[u]);
            u32x4 o;
            int here = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const unsigned m = th.below(w[i]);
                o[i] = (w[i] & ~m) | (low[i] & m);
                here += __popc(~m);
            }
            if ((vi + 1) * N > V) {                              // -inf stands past the end of the row, kept or not
                here = 0;
#pragma unroll
                for (int e = 0; e < N; ++e)
                    if (vi * N + e < V) here += __popc(~(N == 4 ? th.below(w[e & 3]) : th.below(w[e / 2]) | (e & 1 ? 0x0000FFFFu : 0xFFFF0000u)));
            }
            bits += here;
            store_words<DT>(dst, vi, V, o, stream);
        }
    }
    return bits / BITS;
}

// No filter: the row as it is.  us, as a masked copy that keeps everything / so: 1 row of 128256 bf16 logits 10.2 / 7.0, 512 of 32000 bf16
// 17.9 / 15.2, 1088 of 128256 bf16 114 / 113, 512 of 151936 fp32 127 / 125, 512 of 32000 fp32 29.4 / 30.0.
template <typename DT, int U = 4>
__device__ __forceinline__ void plain_copy(const DT *row, DT *dst, int V, bool stream)
{
    constexpr int N = VecOf<DT>::N;
    const int nvec = (V + N - 1) / N;
    for (int v0 = threadIdx.x; v0 < nvec; v0 += U * WARP_WG) {
        typename RawOf<DT>::type r[U];
        warp_load_batch<DT, U>(row, v0, V, r, stream);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int vi = v0 + u * WARP_WG;
            if (vi < nvec) store_words<DT>(dst, vi, V, __builtin_bit_cast(u32x4, r[u]), stream);
        }
    }
}

// The keys of first-digit bin d1 into L.list (the caller has checked that they fit).
template <typename Row>
__device__ __forceinline__ void collect(const Row &rs, unsigned d1, WarpLds &L)
{
    if (threadIdx.x == 0) L.n_list = 0u;
    __syncthreads();
    rs.for_each([&](unsigned key, float) {
        if ((key >> DIGIT1_SHIFT) == d1) {
            const unsigned i = atomicAdd(&L.n_list, 1u);
            if (i < (unsigned)WARP_CAP) L.list[i] = key;
        }
    });
    __syncthreads();
}

// grid (rows), WARP_WG threads.  Instances of their own, because the shortcuts' code costs the other paths registers: NUCLEUS for
// top_p alone over rows that have a shortcut, HISTOGRAMS for top_p alone without one (rows of 65536 bf16 logits 4 % slower otherwise).
enum WarpKind { GENERAL, NUCLEUS, HISTOGRAMS };
template <typename DT, WarpKind KIND>
__global__ __launch_bounds__(WARP_WG, 8) void k_warp(WarpArgs a)
{
    constexpr int N = VecOf<DT>::N;
    __shared__ WarpLds L;
    const int y = blockIdx.x, b = y / a.k, j = y - b * a.k;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const long long off = (long long)b * a.seq_stride + (long long)j * a.row_stride;
    const DT *row = static_cast<const DT *>(a.in) + off;
    DT *dst = static_cast<DT *>(a.out) + off;
    const int V = a.V;

    const bool K = KIND == GENERAL && a.top_k > 0 && a.top_k < V, P = KIND != GENERAL || a.top_p < 1.0;
    if (!K && !P) {
        plain_copy<DT>(row, dst, V, a.stream);
        if (tid == 0) {
            if (a.routes) a.routes[y] = 0;
            if (a.kept) a.kept[y] = V;
        }
        return;
    }
    constexpr bool LONG = KIND == NUCLEUS && N == 8;
    const RowSource<DT, LONG> rs{row, V};
    unsigned tau = 0u;                      // keep keys >= tau
    int kept = 0;
    int decided = 0;
    if (K && !a.no_shortcut)
        decided = a.in != a.out && a.top_k <= WARP_CAP / 8
                      ? small_k_shortcut<DT, true>(row, dst, V, a, P, &tau, &kept, L)
                      : small_k_shortcut<DT, false>(row, dst, V, a, P, &tau, &kept, L);
    float m = neg_inf();
    const bool m_known = KIND == NUCLEUS;
    if constexpr (KIND == NUCLEUS)
        decided = a.in != a.out ? nucleus_shortcut<DT, true>(row, dst, V, a, &tau, &kept, &m, L)
                                : nucleus_shortcut<DT, false>(row, dst, V, a, &tau, &kept, &m, L);
    if (a.routes && tid == 0) a.routes[y] = decided;
    if (decided == 0) {
        // sweep 1: keys per first digit (top-k), row maximum (reference of the top-p weights)
        unsigned d_k = 0u;
        unsigned long long k_rem = 0ull;
        if (K) {
            L.cnt[tid] = 0u;
            L.cnt[tid + WARP_WG] = 0u;
            __syncthreads();
        }
        if (!m_known) for_each_vector<DT, LONG>(row, V, [&](int, const float(&z)[N]) {
            if (P) m = vmax(m, tree_max<N>(z));
            if (K) {
#pragma unroll
                for (int e = 0; e < N; ++e) atomicAdd(&L.cnt[value_key(z[e]) >> DIGIT1_SHIFT], 1u);
            }
        });
        if (P && !m_known) {
            m = wave_max(m);
            if (lane == 0) L.wave_max[wave] = m;
        }
        __syncthreads();
        if (P && !m_known) {
            m = L.wave_max[0];
#pragma unroll
            for (int w = 1; w < WARP_WAVES; ++w) m = vmax(m, L.wave_max[w]);
        }
        if (K) {
            const Crossing c = crossing(L.cnt, (unsigned long long)a.top_k, -1.0, L);
            d_k = c.digit;
            k_rem = c.rem;
        }
        const MassMeasure mass{m, a.sc, a.fix_scale * (1.0f / 4294967296.0f)};

        // sweep 2: mass per first digit from d_k upwards (top-p), the keys of bin d_k (top-k)
        const bool listA = K && L.cnt[d_k] <= (unsigned)WARP_CAP;
        if (P) {
            L.hist[tid] = 0ull;
            L.hist[tid + WARP_WG] = 0ull;
        }
        if (tid == 0) L.n_list = 0u;
        __syncthreads();
        if (P || listA) {
            rs.for_each([&](unsigned key, float z) {
                const unsigned d = key >> DIGIT1_SHIFT;
                if (P && d >= d_k) atomicAdd(&L.hist[d], mass(z));
                if (listA && d == d_k) {
                    const unsigned i = atomicAdd(&L.n_list, 1u);
                    if (i < (unsigned)WARP_CAP) L.list[i] = key;
                }
            });
        }
        __syncthreads();
        const ListSource ls{L.list, listA ? L.n_list : 0u};
        if (K) tau = listA ? refine<KEY_BITS<DT>>(ls, 0u, CountMeasure{}, d_k, k_rem, L) : refine<KEY_BITS<DT>>(rs, 0u, CountMeasure{}, d_k, k_rem, L);
        if (P) {
            if (K) {
                // bin d_k counts only with its keys >= tau
                if (tid == 0) L.acc = 0ull;
                __syncthreads();
                unsigned long long mine = 0ull;
                const auto add = [&](unsigned key, float z) {
                    if ((key >> DIGIT1_SHIFT) == d_k && key >= tau) mine += mass(z);
                };
                if (listA) ls.for_each(add);
                else rs.for_each(add);
                mine = wave_reduce(mine, OpSum{});
                if (lane == 0 && mine) atomicAdd(&L.acc, mine);
                __syncthreads();
                if (tid == 0) L.hist[d_k] = L.acc;
                __syncthreads();
            }
            const Crossing c = crossing(L.hist, 0ull, a.top_p, L);
            unsigned tau_p = 0u;
            if (c.rem != 0ull) {
                if (K && c.digit == d_k) {
                    tau_p = listA ? refine<KEY_BITS<DT>>(ls, tau, mass, d_k, c.rem, L) : refine<KEY_BITS<DT>>(rs, tau, mass, d_k, c.rem, L);
                } else {
                    // sweep 3; a bin too crowded for the list is refined by sweeps over the row instead
                    const bool fits = !K || L.cnt[c.digit] <= (unsigned)WARP_CAP;
                    if (fits) collect(rs, c.digit, L);
                    if (fits && L.n_list <= (unsigned)WARP_CAP) {
                        const ListSource lp{L.list, L.n_list};
                        tau_p = refine<KEY_BITS<DT>>(lp, tau, mass, c.digit, c.rem, L);
                    } else {
                        tau_p = refine<KEY_BITS<DT>>(rs, tau, mass, c.digit, c.rem, L);
                    }
                }
            }
            tau = tau_p > tau ? tau_p : tau;
        }
    }

    if (decided == 2) {
        if (a.kept && tid == 0) a.kept[y] = kept;
        return;
    }
    kept = masked_copy<DT>(row, dst, V, tau, a.stream);
    if (a.kept) {
        kept = wave_reduce(kept, OpSum{});
        if (lane == 0) L.wave_kept[wave] = kept;
        __syncthreads();
        if (tid == 0) {
            int n = 0;
#pragma unroll
            for (int w = 0; w < WARP_WAVES; ++w) n += L.wave_kept[w];
            a.kept[y] = n;
        }
    }
}

}  // namespace svip
