// Quantile estimation for the quantile map (App. F.2, App. G, "SRAM-Quantiles"):
// the tensor is cut into chunks of kQChunk values; one workgroup per chunk finds
// its 257 sample quantiles Q_c(i / 257) = sorted[floor(i L / 257)] on chip (by
// counting into buckets, or a sort where the buckets do not separate the
// values); the estimate of each quantile is the average of the chunk
// quantiles, weighted by chunk length.
// Instead of the atomic averaging in DRAM that App. G describes, the chunk
// quantiles are summed in a fixed order -- sequentially within groups of
// kQGroup consecutive chunks (one workgroup per group), then sequentially over
// the groups -- so the result is deterministic.  From the averaged quantiles
// Q(p) the map follows Eq. 5: q_i = (Q(i / 257) + Q((i + 1) / 257)) / 2,
// divided by max |q_i|, rounded to fp32, equal entries moved up by one ulp.
#include "bq_device.h"

namespace bq {
namespace {

using namespace dev;

constexpr int kQThreads = 256;                    // threads per chunk sort
constexpr int kQPerThread = kQChunk / kQThreads;  // keys per thread
static_assert(kQChunk == kQThreads * kQPerThread && kQPerThread % 4 == 0, "chunk shape");
constexpr int kCombineThreads = 512;              // >= 257

// fp32 bit pattern -> unsigned key of the same order, and back
__device__ inline uint32_t order_key(uint32_t u)
{
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ inline uint32_t key_bits(uint32_t k)
{
    return (k & 0x80000000u) ? (k & 0x7fffffffu) : ~k;
}

// Bitonic sort of KMAX keys, P per thread, by one workgroup (KMAX = kQChunk) or
// one wave (64 P): thread or lane t holds sorted positions P t .. P t + P - 1 when
// done.  A pass compares position p with p ^ J (the lower position keeps the
// smaller key when (p & K) == 0, the larger otherwise).  Partners at distance
// J < P are in the same thread, at P <= J < 64 P in another lane of the same wave
// (exchanged by lane shuffles), at J >= 64 P in another wave (exchanged through
// LDS).  The whole network is unrolled at compile time so the keys stay in
// registers.

// The key of lane (lane ^ M) of the wave: DPP for M = 1, 2 (quad permutes)
// and 8 (rotation of a 16-lane row by 8), a swizzle within 32 lanes for
// M = 4, 16, a permute through the LDS crossbar for M = 32.
template <int M>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v)
{
    const int x = (int)v;
    if constexpr (M == 1)
        return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, false);
    else if constexpr (M == 2)
        return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0x4E, 0xF, 0xF, false);
    else if constexpr (M == 8)
        return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0x128, 0xF, 0xF, false);
    else if constexpr (M == 4 || M == 16)
        return (uint32_t)__builtin_amdgcn_ds_swizzle(x, 0x1F | (M << 10));
    else
        return (uint32_t)__shfl_xor(x, M);
}

// median of three: med3(a, b, 0) = min(a, b), med3(a, b, ~0) = max(a, b), so
// one instruction takes the kept key of a compare-exchange given a per-lane
// selector
__device__ __forceinline__ uint32_t med3u(uint32_t a, uint32_t b, uint32_t s)
{
    uint32_t r;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(s));
    return r;
}

template <int P, int K, int J>
__device__ __forceinline__ void bitonic_pass(uint32_t (&a)[P], uint32_t *keys, int tid)
{
    if constexpr (J >= 64 * P) {
        constexpr int m = J / P;  // partner thread distance (another wave)
        constexpr int V = P / 4;  // 16-byte vectors per thread
#pragma unroll
        for (int v = 0; v < V; ++v)
            reinterpret_cast<vu4 *>(keys)[V * tid + v] =
                vu4{a[4 * v], a[4 * v + 1], a[4 * v + 2], a[4 * v + 3]};
        __syncthreads();
        const int pt = tid ^ m;
        uint32_t b[P];
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const vu4 bv = reinterpret_cast<const vu4 *>(keys)[V * pt + v];
            b[4 * v] = bv.x;
            b[4 * v + 1] = bv.y;
            b[4 * v + 2] = bv.z;
            b[4 * v + 3] = bv.w;
        }
        __syncthreads();
        const bool keep_min = ((tid & m) == 0) == (((P * tid) & K) == 0);
        const uint32_t sel = keep_min ? 0u : ~0u;
#pragma unroll
        for (int i = 0; i < P; ++i)
            a[i] = med3u(a[i], b[i], sel);
    } else if constexpr (J >= P) {
        constexpr int m = J / P;  // partner lane distance, < 64
        const bool keep_min = ((tid & m) == 0) == (((P * tid) & K) == 0);
        const uint32_t sel = keep_min ? 0u : ~0u;
#pragma unroll
        for (int i = 0; i < P; ++i)
            a[i] = med3u(a[i], lane_xor<m>(a[i]), sel);
    } else {
#pragma unroll
        for (int i = 0; i < P; ++i) {
            if ((i & J) == 0) {
                const bool asc = ((P * tid + i) & K) == 0;
                const uint32_t lo = asc ? 0u : ~0u;
                const uint32_t x = a[i], y = a[i | J];
                a[i] = med3u(x, y, lo);
                a[i | J] = med3u(x, y, ~lo);
            }
        }
    }
    if constexpr (J > 1)
        bitonic_pass<P, K, J / 2>(a, keys, tid);
}

template <int P, int KMAX, int K = 2>
__device__ __forceinline__ void bitonic_sort(uint32_t (&a)[P], uint32_t *keys, int tid)
{
    bitonic_pass<P, K, K / 2>(a, keys, tid);
    if constexpr (K < KMAX)
        bitonic_sort<P, KMAX, 2 * K>(a, keys, tid);
}

// ---------------------------------------------------------------------------
// Quantiles by buckets
// ---------------------------------------------------------------------------

// Only 257 of a chunk's ranks are needed, so a full sort does too much: the
// values are counted into kQBuckets buckets that preserve order, placed in
// bucket order (unsorted inside a bucket), and each wanted rank is selected
// among the few values of its bucket.  A bucket of many different values is sorted
// by a wave; a chunk in which these are too many, as a whole.
//
// Buckets.  With u the magnitude bits of a value, [lo, hi] a range of u and
// m = min(u, 1) + (min(max(u - lo, 0), hi - lo) >> shift), a value counts in
// bucket base + m when its sign bit is clear and in base - 1 - m when it is set:
// monotone in the order of the values, -0 before +0, for any bit pattern.
// Each value belongs to one of four classes.  lo is the largest of the classes'
// smallest nonzero u and hi the smallest of their largest (of those that have a
// nonzero u), so that about 8 of 4096 values lie below lo and 8 above hi, whereupon
// both move outwards by an eighth of the range if there are values: a few
// outliers, in the buckets of m = 1 and in the last ones, do not take the buckets
// away from the others.  shift is the smallest that fits the range into
// half of the buckets (all of them when the signs agree).  Normal values then
// take about 11 binades at 256 buckets each, 2 to 3 values per occupied bucket;
// a wider range gets fewer buckets per binade.
//
// VALU and LDS instructions and the waits between them bound it, not HBM: 646 VALU
// instructions per wave for 16 values per lane, of which about 21 a value for the
// counting and placing.  256 threads: a rank each (512 x 8 values took 1.2 times as
// long).  Reading all the first places before the first value is placed is 2 % slower.
//
// Times of the whole estimate for 2^24 values (MI355X, HIP graph), us, against a
// sort of every chunk:
//   normal                             37   65    ReLU of normal          59   81
//   uniform                            38   65    zeros                   61   84
//   normal in order                    35   64    sigmoid(3 normal)       55   66
//   normal, one 1e38 a chunk           37   65    tanh(3 normal)          85   64
//   sixteen values                     77   81    half normal, half within
//   4 normal clamped to [0, 6]         89   81    1e-6 of 0.5            115   80
// (Ties in the map take one thread about 20 us in either column.)  A chunk that is
// sorted pays for the count before it.
constexpr int kQBuckets = 8192;                // two 16-bit counters per word
constexpr int kQWords = kQBuckets / 2;
constexpr int kQScanWords = kQWords / kQThreads;  // consecutive words per thread
// A bucket of more than kQBig values that differ is sorted by one wave (a run); a
// chunk is sorted as a whole when a wave finds more than kQWaveRuns of them, or
// one of more than kQRunMost values.
constexpr int kQBig = 32;
constexpr int kQRuns = kQChunk / (kQBig + 1);  // there are no more big buckets
constexpr int kQWaveRuns = 8;
constexpr int kQRunKeys = 2;  // per lane
constexpr int kQRunMost = 64 * kQRunKeys;
// A value of which a wave sees at least kQOften among 128 is set aside.
constexpr int kQOften = 24;
static_assert(kQScanWords % 4 == 0, "a thread scans whole 16-byte groups");

// Byte offset of the word that counts bucket b (two buckets per word): groups
// of 4 words are permuted so that the scan's 16-byte reads of consecutive
// words per thread spread over all banks.
__device__ __forceinline__ uint32_t bucket_offset(uint32_t b)
{
    return ((b << 1) & ~3u) ^ ((b >> 1) & 0x70u);
}
__device__ __forceinline__ uint32_t &bucket_word(uint32_t *count, uint32_t b)
{
    return *reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(count) + bucket_offset(b));
}
// First place of bucket b once the counts are scanned.
__device__ __forceinline__ uint32_t bucket_first(uint32_t *count, uint32_t b)
{
    return __builtin_amdgcn_ubfe(bucket_word(count, b), b << 4, 16);  // 16 (b & 1)
}

struct BucketMap {
    uint32_t lo, range, shift, base;
};

__device__ __forceinline__ uint32_t bucket_index(const BucketMap &M, uint32_t bits)
{
    const uint32_t u = bits & 0x7fffffffu;
    const uint32_t m =
        min(u, 1u) + (min(__builtin_elementwise_sub_sat(u, M.lo), M.range) >> M.shift);
    return (m ^ (uint32_t)((int)bits >> 31)) + M.base;  // base + ~m = base - 1 - m
}

// Max over the wave, in every lane (rows by DPP, then the four rows).
__device__ __forceinline__ uint32_t wave_umax(uint32_t v)
{
    const int r = (int)row_umax(v);
    return max(max((uint32_t)__builtin_amdgcn_readlane(r, 0),
                   (uint32_t)__builtin_amdgcn_readlane(r, 16)),
               max((uint32_t)__builtin_amdgcn_readlane(r, 32),
                   (uint32_t)__builtin_amdgcn_readlane(r, 48)));
}

// Maxima of the four classes, value h of lane l in class (l + h) mod 4, over a row
// of 16 lanes: class c in the lanes l = c (mod 4).  Neighbouring values, values at
// any stride and values in order are spread evenly over the classes.
__device__ __forceinline__ uint32_t rotate_classes(uint32_t v)
{
    v = dpp_umax<0x124, 0xf>(v);     // row_ror 4
    return dpp_umax<0x128, 0xf>(v);  // row_ror 8
}
__device__ __forceinline__ uint32_t class_umax(const uint32_t (&v)[4])
{
    const int a = __builtin_amdgcn_mov_dpp((int)v[1], 0x93, 0xf, 0xf, false);  // lane l - 1
    const int b = __builtin_amdgcn_mov_dpp((int)v[2], 0x4e, 0xf, 0xf, false);  // l - 2
    const int c = __builtin_amdgcn_mov_dpp((int)v[3], 0x39, 0xf, 0xf, false);  // l - 3
    return rotate_classes(max(max(v[0], (uint32_t)a), max((uint32_t)b, (uint32_t)c)));
}

// Sorts c[0 .. N) in registers by Batcher's odd-even mergesort network.
template <int N>
__device__ __forceinline__ void sort_network(uint32_t *c)
{
#pragma unroll
    for (int p = 1; p < N; p *= 2)
#pragma unroll
        for (int h = p; h >= 1; h /= 2)
#pragma unroll
            for (int j = h % p; j + h < N; j += 2 * h)
#pragma unroll
                for (int i = 0; i < h; ++i)
                    if (i + j + h < N && (i + j) / (2 * p) == (i + j + h) / (2 * p)) {
                        const uint32_t x = c[i + j], y = c[i + j + h];
                        c[i + j] = min(x, y);
                        c[i + j + h] = max(x, y);
                    }
}

// The value of rank t among vals[s .. s + k), k <= N, all of one sign (so that
// their bits order like their magnitudes; counted from the other end for negative
// values).  Two sorted halves, the second taken backwards, are a bitonic sequence:
// the smaller (larger) of each pair of opposite values are its smaller (larger)
// half and bitonic again, so each bit of t takes one instruction per value kept
// (27 instructions of 8 values against 45 with a sort of all, 91 against 141 of
// 16).  Reads up to N - 1 words past the bucket.
template <int N>
__device__ __forceinline__ uint32_t select_network(const uint32_t *vals, int s, int k, int t)
{
    uint32_t c[N];
#pragma unroll
    for (int i = 0; i < N; ++i)
        c[i] = vals[s + i];
    t = (int)c[0] < 0 ? k - 1 - t : t;
    if constexpr (N > 8) {
        // buckets this full often hold one value (small whole numbers, bf16)
        uint32_t other = 0u;
#pragma unroll
        for (int i = 1; i < N; ++i)
            other |= i < k ? c[i] ^ c[0] : 0u;
        if (!__any(other != 0u))
            return c[0];
    }
#pragma unroll
    for (int i = 1; i < N; ++i)
        c[i] = i < k ? c[i] : 0xffffffffu;
    sort_network<N / 2>(c);
    sort_network<N / 2>(c + N / 2);
#pragma unroll
    for (int w = N / 2; w >= 1; w /= 2) {
        const uint32_t larger = (t & w) ? ~0u : 0u;
#pragma unroll
        for (int i = 0; i < w; ++i)
            c[i] = med3u(c[i], c[w == N / 2 ? N - 1 - i : i + w], larger);
    }
    return c[0];
}

// The same by a whole wave, for s, k <= kQBig and t that are the same in all lanes:
// each lane counts the values before its own.  Taken for a wave's single rank in a
// bucket of more than 8 values (19 % of the waves of normal values), for which all
// lanes would otherwise go through the network of 16: 2^26 normal values 110.7 us
// against 113.8; up to 3 ranks one after the other 112.1, and uniform values, which
// have more of them, 119.1 against 116.0.
__device__ __forceinline__ uint32_t select_by_wave(const uint32_t *vals, int s, int k, int t)
{
    const int lane = threadIdx.x & 63;
    const uint32_t key = lane < k ? order_key(vals[s + lane]) : 0xffffffffu;
    int less = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j)
        less += (uint32_t)__builtin_amdgcn_readlane((int)key, j) < key ? 1 : 0;
    if (k > 16) {
#pragma unroll
        for (int j = 16; j < kQBig; ++j)
            less += (uint32_t)__builtin_amdgcn_readlane((int)key, j) < key ? 1 : 0;
    }
    return key_bits(wave_umax(less <= t ? key : 0u));
}

// One wave sorts vals[s .. s + k), k <= 64 P, in place unless the values are
// equal; whether they are not.
template <int P>
__device__ __forceinline__ bool sort_run(uint32_t *vals, int s, int k)
{
    const int lane = threadIdx.x & 63;
    uint32_t a[P], other = 0u;
#pragma unroll
    for (int i = 0; i < P; ++i)
        a[i] = vals[s + min(64 * i + lane, k - 1)];
    const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)a[0]);
#pragma unroll
    for (int i = 0; i < P; ++i) {
        other |= a[i] ^ first;
        a[i] = 64 * i + lane < k ? order_key(a[i]) : 0xffffffffu;
    }
    if (!__any(other != 0u))
        return false;
    bitonic_sort<P, 64 * P>(a, nullptr, lane);
#pragma unroll
    for (int i = 0; i < P; ++i)
        if (P * lane + i < k)
            vals[s + P * lane + i] = key_bits(a[i]);
    return true;
}

// One workgroup per chunk writes the chunk's 257 sample quantiles.  Value 4h + r of
// thread t is element 4t + 4 kQThreads h + r (coalesced loads; any arrangement
// will do).
__global__ __launch_bounds__(kQThreads, 4) void chunk_quantiles_kernel(const float *__restrict__ xs,
                                                                       int64_t n,
                                                                       float *__restrict__ partial)
{
    // the values, the counters (which select_network may read into); two words and
    // one word per wave, the number of big buckets and the buckets
    constexpr int kWaves = kQThreads / 64;
    __shared__ __attribute__((aligned(16))) uint32_t
        lds[kQChunk + kQWords + 3 * kWaves + 1 + kQRuns];
    uint32_t *const vals = lds, *const count = vals + kQChunk, *const tallies = count + kQWords;
    uint32_t *const slots = tallies + 2 * kWaves;
    const int64_t c0 = (int64_t)blockIdx.x * kQChunk;
    const float *const x = xs + c0;
    const int L = n - c0 >= kQChunk ? kQChunk : (int)(n - c0);
    const bool full = L == kQChunk;
    float *const out = partial + (int64_t)blockIdx.x * 257;
    const int tid = threadIdx.x;
    const int wave = tid >> 6;
    const auto element = [&](int i) { return 4 * tid + 4 * kQThreads * (i / 4) + (i & 3); };
    uint32_t a[kQPerThread];
    // 16-byte loads need x itself 16-byte aligned (the chunk starts at a
    // multiple of 4096 values); a view that is only 4-byte aligned takes the
    // scalar loads
    const bool aligned = (reinterpret_cast<uintptr_t>(x) & 15u) == 0;
    const auto load = [&](int h) {
        const vf4 v = ld_nt(reinterpret_cast<const vf4 *>(x + 4 * tid + 4 * kQThreads * h));
        a[4 * h] = __float_as_uint(v.x);
        a[4 * h + 1] = __float_as_uint(v.y);
        a[4 * h + 2] = __float_as_uint(v.z);
        a[4 * h + 3] = __float_as_uint(v.w);
    };
    if (full && aligned) {
#pragma unroll
        for (int h = 0; h < kQPerThread / 4; ++h)
            load(h);
    } else {
        // past the end: values that are there, evenly, for the statistics
        const int in = (int)(0x7fffffffu >> __builtin_clz(L));  // 2^floor(log2 L) - 1
#pragma unroll
        for (int h = 0; h < kQPerThread / 4; ++h) {
            if (aligned && 4 * kQThreads * (h + 1) <= L) {
                load(h);
            } else if (4 * kQThreads * h < L) {
#pragma unroll
                for (int i = 4 * h; i < 4 * h + 4; ++i)
                    a[i] = __float_as_uint(G(x)[element(i) < L ? element(i) : element(i) & in]);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    a[4 * h + r] = a[r];
            }
        }
    }
    // counters cleared while the loads are in flight
#pragma unroll
    for (int v = 0; v < kQScanWords / 4; ++v)
        reinterpret_cast<vu4 *>(count)[tid + kQThreads * v] = vu4{0u, 0u, 0u, 0u};

    // whether there are signs of either kind; per class the smallest nonzero and the
    // largest magnitude (taken as -u, zero is the least).  The slots lie in vals,
    // which is filled later.
    static_assert(kQPerThread == 16, "four values per class and thread");
    uint32_t low[4], top[4];
    int least = (int)a[0], greatest = (int)a[0];
#pragma unroll
    for (int i = 0; i < kQPerThread; ++i) {
        least = min(least, (int)a[i]);
        greatest = max(greatest, (int)a[i]);
        const uint32_t u = a[i] & 0x7fffffffu;
        low[i / 4] = i % 4 ? max(low[i / 4], 0u - u) : 0u - u;
        top[i / 4] = i % 4 ? max(top[i / 4], u) : u;
    }
    const uint32_t signs = (__any(least < 0) ? 1u : 0u) | (__any(greatest >= 0) ? 2u : 0u);
    const uint32_t low_row = class_umax(low), top_row = class_umax(top);
    // the more frequent of two values, among 128
    const auto frequency = [&](uint32_t v) {
        return (uint32_t)(__popcll(__ballot(a[0] == v)) + __popcll(__ballot(a[10] == v)));
    };
    const uint32_t one = (uint32_t)__builtin_amdgcn_readlane((int)a[0], 5);
    const uint32_t two = (uint32_t)__builtin_amdgcn_readlane((int)a[10], 40);
    const uint32_t times_one = frequency(one), times_two = frequency(two);
    if ((tid & 63) == 0)
        reinterpret_cast<vu2 *>(vals)[wave] = vu2{times_one > times_two ? one : two,
                                                  max(times_one, times_two) << 2 | signs};
    constexpr int kRows = kQThreads / 16;
    uint32_t *const lows = vals + 2 * kWaves, *const tops = lows + 4 * kRows;
    if ((tid & 15) < 4) {
        lows[kRows * (tid & 3) + (tid >> 4)] = low_row;
        tops[kRows * (tid & 3) + (tid >> 4)] = top_row;
    }
    __syncthreads();
    uint32_t often = 0u, times = 0u, either = 0u;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const vu2 v = reinterpret_cast<const vu2 *>(vals)[w];
        often = v.y >> 2 > times ? v.x : often;
        times = max(times, v.y >> 2);
        either |= v.y;
    }
    often = (uint32_t)__builtin_amdgcn_readfirstlane((int)often);
    const bool aside = __builtin_amdgcn_readfirstlane((int)times) >= kQOften;
    const bool all = full && !aside;
    either = (uint32_t)__builtin_amdgcn_readfirstlane((int)either);
    const bool neg = (either & 1u) != 0u, both = (either & 3u) == 3u;
    static_assert(kRows == 16, "a row of lanes reads every row's maxima");
    const auto over_rows = [&](const uint32_t *rows) {  // of the class tid % 4
        const vu4 v = reinterpret_cast<const vu4 *>(rows)[4 * (tid & 3) + ((tid >> 2) & 3)];
        return rotate_classes(max(max(v.x, v.y), max(v.z, v.w)));
    };
    const auto over_classes = [](uint32_t v) {
        v = dpp_umax<0xb1, 0xf>(v);
        v = dpp_umax<0x4e, 0xf>(v);
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
    };
    const uint32_t low_class = over_rows(lows), top_class = over_rows(tops);
    const uint32_t ends[2] = {over_classes(0u - low_class), 0u - over_classes(0u - top_class)};
    uint32_t lo = min(ends[0], ends[1]), hi = max(ends[0], ends[1]);
    const uint32_t more = (hi - lo) / 8;
    lo = max(0u - over_classes(low_class), __builtin_elementwise_sub_sat(lo, more));
    hi = min(over_classes(top_class), hi + more);
    BucketMap M;
    M.lo = lo;
    // values that do not take part go to the last kQThreads buckets
    const uint32_t buckets = all ? kQBuckets : kQBuckets - kQThreads;
    M.base = both ? kQBuckets / 2 : neg ? buckets : 0;
    M.range = hi - lo;
    const uint32_t most = buckets - (both ? kQBuckets / 2 : 0) - 2;
    M.shift = (uint32_t)max(32 - __builtin_clz(M.range | 1u) - (both ? 12 : 13), 0);
    M.shift += (M.range >> M.shift) > most ? 1u : 0u;

    uint32_t b[kQPerThread], before[kQPerThread];
#pragma unroll
    for (int i = 0; i < kQPerThread; ++i)
        b[i] = bucket_index(M, a[i]);
    // A value that is a large part of the chunk takes no part from here on, lest its
    // counter be added to by most lanes at once, and is brought back into the ranks:
    // `equal` values are it, `below` lie before it.  Each thread gives those that
    // take no part a bucket after all others.
    uint32_t mine = (1u << kQPerThread) - 1u;  // bit i: value i takes part
    int equal = 0, below = 0;
    if (!all) {
        const auto signed_key = [](uint32_t v) {
            return (int)(v ^ ((uint32_t)((int)v >> 31) >> 1));
        };
#pragma unroll
        for (int i = 0; i < kQPerThread; ++i) {
            if (element(i) >= L || (aside && a[i] == often)) {
                mine &= ~(1u << i);
                b[i] = (uint32_t)(kQBuckets - kQThreads + tid);
            }
        }
        if (aside) {
#pragma unroll
            for (int i = 0; i < kQPerThread; ++i) {
                const bool there = element(i) < L;
                equal += (int)__popcll(__ballot(there && a[i] == often));
                below += (int)__popcll(__ballot(there && signed_key(a[i]) < signed_key(often)));
            }
            if ((tid & 63) == 0)
                reinterpret_cast<vu2 *>(tallies)[wave] = vu2{(uint32_t)equal, (uint32_t)below};
            __syncthreads();
            equal = below = 0;
#pragma unroll
            for (int k = 0; k < kWaves; ++k) {
                const vu2 v = reinterpret_cast<const vu2 *>(tallies)[k];
                equal += (int)v.x;
                below += (int)v.y;
            }
            equal = __builtin_amdgcn_readfirstlane(equal);
            below = __builtin_amdgcn_readfirstlane(below);
        }
    }
    const int placed = L - equal;
    const auto end = [&](uint32_t bk) {
        return bk + 1 < (uint32_t)kQBuckets ? bucket_first(count, bk + 1) : (uint32_t)kQChunk;
    };
    // OR over the workgroup
    static_assert(kWaves == 4, "the slots are read at once");
    const auto over_waves = [&](uint32_t of_wave) {
        if ((tid & 63) == 0)
            slots[wave] = of_wave;
        __syncthreads();
        const vu4 v = *reinterpret_cast<const vu4 *>(slots);
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)(v.x | v.y | v.z | v.w));
    };
    if (tid == 0)
        slots[kWaves] = 0u;  // runs
    // count; `before` is the counters' word before the add: the number of a bucket's
    // values so far is a value's place in it
    uint32_t some = 0u, kinds = 0u;
#pragma unroll
    for (int i = 0; i < kQPerThread; ++i)
        before[i] = atomicAdd(&bucket_word(count, b[i]), 1u << ((b[i] << 4) & 31u));
#pragma unroll
    for (int i = 0; i < kQPerThread; ++i)
        some |= before[i];
    const auto place = [&](int i) { return __builtin_amdgcn_ubfe(before[i], b[i] << 4, 16); };
    // bit 0: a big bucket; bit 1: one too large for a run whose values differ (each
    // wave looks at the first that it meets, from the last values counted)
    static_assert((kQBig & (kQBig - 1)) == 0, "a bit of both counters tells");
    if (__any((some & (0x10001u * (0x10000u - kQBig))) != 0u)) {
        uint64_t met = 0u;
        uint32_t bucket = 0u, value = 0u;
        bool differ = false;
#pragma unroll
        for (int i = kQPerThread - 1; i >= 0; --i) {
            if (met == 0u) {
                met = __ballot(place(i) >= (uint32_t)kQRunMost);
                const int lane = met != 0u ? __builtin_ctzll(met) : 0;
                bucket = (uint32_t)__builtin_amdgcn_readlane((int)b[i], lane);
                value = (uint32_t)__builtin_amdgcn_readlane((int)a[i], lane);
            }
            differ = differ || (met != 0u && b[i] == bucket && a[i] != value);
        }
        kinds = __any(differ) ? 3u : 1u;
    }
    kinds = over_waves(kinds);
    bool sort = (kinds & 2u) != 0u;
    if (!sort) {
        // counts to first places: a thread scans 2 kQScanWords consecutive
        // buckets, with the running count in both halves of a word
        uint32_t w[kQScanWords], total = 0;
#pragma unroll
        for (int v = 0; v < kQScanWords / 4; ++v) {
            const vu4 c = *reinterpret_cast<const vu4 *>(
                &bucket_word(count, (uint32_t)(2 * kQScanWords * tid + 8 * v)));
            w[4 * v] = c.x;
            w[4 * v + 1] = c.y;
            w[4 * v + 2] = c.z;
            w[4 * v + 3] = c.w;
            total += c.x + c.y + c.z + c.w;
        }
        // (at most 4096 values: no carry between halves)
        total = (total & 0xffffu) + (total >> 16);
        const uint32_t incl = wave_scan(total);
        if ((tid & 63) == 63)
            vals[wave] = incl;
        __syncthreads();
        uint32_t run = incl - total;
        const vu4 of_waves = *reinterpret_cast<const vu4 *>(vals);
        run += wave > 0 ? of_waves.x : 0u;
        run += wave > 1 ? of_waves.y : 0u;
        run += wave > 2 ? of_waves.z : 0u;
        run |= run << 16;
#pragma unroll
        for (int v = 0; v < kQScanWords / 4; ++v) {
            uint32_t o[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t c = w[4 * v + k];
                o[k] = run + (c << 16);
                run += c + __builtin_amdgcn_alignbit(c, c, 16);
            }
            *reinterpret_cast<vu4 *>(
                &bucket_word(count, (uint32_t)(2 * kQScanWords * tid + 8 * v))) =
                vu4{o[0], o[1], o[2], o[3]};
        }
        __syncthreads();

        // values in bucket order (first place and place in the bucket in one add: no
        // carry between halves)
#pragma unroll
        for (int i = 0; i < kQPerThread; ++i)
            vals[__builtin_amdgcn_ubfe(bucket_word(count, b[i]) + before[i], b[i] << 4, 16)] =
                a[i];
        if (kinds != 0u) {
            // each big bucket's value at place kQBig makes the bucket known
#pragma unroll
            for (int i = 0; i < kQPerThread; ++i) {
                if (place(i) == (uint32_t)kQBig) {
                    const uint32_t at_run = atomicAdd(&slots[kWaves], 1u);
                    slots[kWaves + 1 + at_run] = b[i];
                }
            }
            __syncthreads();
            const int runs = __builtin_amdgcn_readfirstlane((int)slots[kWaves]);
            int mixed = 0;
            for (int j = wave; j < runs && mixed <= kQWaveRuns; j += kWaves) {
                const uint32_t bk =
                    (uint32_t)__builtin_amdgcn_readfirstlane((int)slots[kWaves + 1 + j]);
                const int s = __builtin_amdgcn_readfirstlane((int)bucket_first(count, bk));
                const int k = __builtin_amdgcn_readfirstlane((int)end(bk)) - s;
                if (k <= kQRunMost) {
                    mixed += sort_run<kQRunKeys>(vals, s, k) ? 1 : 0;
                } else {
                    uint32_t other = 0u;
                    for (int i = tid & 63; i < k; i += 64)
                        other |= vals[s + i] ^ vals[s];
                    mixed += __any(other != 0u) ? kQWaveRuns + 1 : 0;
                }
            }
            sort = over_waves(mixed > kQWaveRuns ? 1u : 0u) != 0u;
        } else {
            __syncthreads();
        }
    }
    if (sort) {
#pragma unroll
        for (int i = 0; i < kQPerThread; ++i)
            a[i] = (mine >> i & 1u) != 0u ? order_key(a[i]) : 0xffffffffu;
        bitonic_sort<kQPerThread, kQChunk>(a, vals, tid);
        constexpr int V = kQPerThread / 4;
#pragma unroll
        for (int v = 0; v < V; ++v)
            reinterpret_cast<vu4 *>(vals)[V * tid + v] =
                vu4{key_bits(a[4 * v]), key_bits(a[4 * v + 1]), key_bits(a[4 * v + 2]),
                    key_bits(a[4 * v + 3])};
        __syncthreads();
    }
    // ranks floor(i L / 257), i = 1 .. 256, one per thread; i = 0 is the minimum
    static_assert(kQThreads == 256, "one rank per thread");
    const int rank = (int)((uint32_t)((tid + 1) * L) / 257u);
    uint32_t v = often;
    if (placed > 0) {
        const bool is_often = rank >= below && rank < below + equal;
        const int p = is_often ? 0 : rank - (rank < below ? 0 : equal);
        uint32_t c = vals[p];
        if (!sort) {
            const uint32_t bk = bucket_index(M, c);
            const int s = (int)bucket_first(count, bk), t = p - s;
            const int k = is_often ? 1 : (int)end(bk) - s;
            const uint64_t more_than_8 = __ballot(k > 8 && k <= kQBig);
            if ((more_than_8 & (more_than_8 - 1u)) == 0u) {
                if (k > 1 && k <= 8)
                    c = select_network<8>(vals, s, k, t);
                if (more_than_8 != 0u) {
                    // a single rank: by the whole wave
                    const int l = __builtin_ctzll(more_than_8);
                    const uint32_t of_l = select_by_wave(vals, __builtin_amdgcn_readlane(s, l),
                                                         __builtin_amdgcn_readlane(k, l),
                                                         __builtin_amdgcn_readlane(t, l));
                    c = (tid & 63) == l ? of_l : c;
                }
            } else if (k > 1 && k <= kQBig) {
                // one network for the wave, the size its largest bucket needs
                if (!__any(k > 16))
                    c = select_network<16>(vals, s, k, t);
                else
                    c = select_network<32>(vals, s, k, t);
            }
        }
        v = is_often ? often : c;
    }
    G(out)[tid + 1] = __uint_as_float(v);
    // i = 0 is the minimum, of the first bucket or the value set aside
    if (wave == 0) {
        uint32_t m = ~0u;
        if (placed > 0) {
            const uint32_t c = vals[0];
            const int k = sort ? 1 : (int)end(bucket_index(M, c));
            m = order_key(tid < min(k, kQBig) ? vals[tid] : c);
        }
        m = ~wave_umax(~(aside ? min(m, order_key(often)) : m));
        if (tid == 0)
            G(out)[0] = __uint_as_float(key_bits(m));
    }
}

// One workgroup per group of kQGroup chunks: length-weighted sums of the chunk
// quantiles, in chunk order, in double.  A full group's kQGroup loads are all
// issued before the first add (the adds keep chunk order).
__global__ __launch_bounds__(320) void group_sums_kernel(const float *__restrict__ partial,
                                                         int64_t n, int64_t nchunks,
                                                         double *__restrict__ gsum)
{
    const int tid = threadIdx.x;
    if (tid > 256)
        return;
    const int64_t c0 = (int64_t)blockIdx.x * kQGroup;
    const int64_t c1 = c0 + kQGroup < nchunks ? c0 + kQGroup : nchunks;
    double s = 0.0;
    if (c1 - c0 == kQGroup) {
        float v[kQGroup];
#pragma unroll
        for (int k = 0; k < kQGroup; ++k)
            v[k] = G(partial)[(c0 + k) * 257 + tid];
#pragma unroll
        for (int k = 0; k < kQGroup; ++k) {
            const int64_t rem = n - (c0 + k) * kQChunk;
            const double L = (double)(rem >= kQChunk ? kQChunk : rem);
            s += L * (double)v[k];
        }
    } else {
        for (int64_t c = c0; c < c1; ++c) {
            const int64_t rem = n - c * kQChunk;
            const double L = (double)(rem >= kQChunk ? kQChunk : rem);
            s += L * (double)G(partial)[c * 257 + tid];
        }
    }
    G(gsum)[(int64_t)blockIdx.x * 257 + tid] = s;
}

// One workgroup: sum the group sums in order, average, then Eq. 5.
__global__ __launch_bounds__(kCombineThreads) void combine_quantiles_kernel(
    const double *__restrict__ gsum, int64_t n, int64_t ngroups, float *__restrict__ out)
{
    __shared__ double Q[257];
    __shared__ double q[256];
    __shared__ double red[256];
    __shared__ float map[256];
    __shared__ int tie;
    const int tid = threadIdx.x;
    if (tid == 0)
        tie = 0;
    if (tid <= 256) {
        // in group order; loads issued 32 at a time
        double s = 0.0;
        int64_t g = 0;
        for (; g + 32 <= ngroups; g += 32) {
            double v[32];
#pragma unroll
            for (int k = 0; k < 32; ++k)
                v[k] = G(gsum)[(g + k) * 257 + tid];
#pragma unroll
            for (int k = 0; k < 32; ++k)
                s += v[k];
        }
        for (; g < ngroups; ++g)
            s += G(gsum)[g * 257 + tid];
        Q[tid] = s / (double)n;
    }
    __syncthreads();
    if (tid < 256) {
        q[tid] = (Q[tid] + Q[tid + 1]) * 0.5;
        red[tid] = fabs(q[tid]);
    }
    __syncthreads();
    // max |q_i| by a tree (a maximum is exact in any order)
    for (int h = 128; h > 0; h >>= 1) {
        if (tid < h)
            red[tid] = fmax(red[tid], red[tid + h]);
        __syncthreads();
    }
    const double amax = red[0];
    if (tid < 256)
        map[tid] = (float)(amax > 0.0 ? q[tid] / amax : q[tid]);
    __syncthreads();
    // equal neighbours (ties in the sample) moved up by one ulp, in order; the
    // serial pass runs only when some neighbour is not strictly above its
    // predecessor
    if (tid >= 1 && tid < 256 && !(map[tid] > map[tid - 1]))
        tie = 1;
    __syncthreads();
    if (tid == 0 && tie) {
        for (int i = 1; i < 256; ++i)
            if (!(map[i] > map[i - 1]))
                map[i] = next_up(map[i - 1]);
    }
    __syncthreads();
    if (tid < 256)
        G(out)[tid] = map[tid];
}

}  // namespace

hipError_t launch_quantile_codebook(const float *x, int64_t n, void *workspace, float *out,
                                    hipStream_t stream)
{
    const int64_t nchunks = (n + kQChunk - 1) / kQChunk;
    const int64_t ngroups = (nchunks + kQGroup - 1) / kQGroup;
    float *partial = static_cast<float *>(workspace);
    double *gsum = reinterpret_cast<double *>(static_cast<char *>(workspace) +
                                              quantile_partial_bytes(n));
    hipLaunchKernelGGL(chunk_quantiles_kernel, dim3((unsigned)nchunks), dim3(kQThreads), 0,
                       stream, x, n, partial);
    hipLaunchKernelGGL(group_sums_kernel, dim3((unsigned)ngroups), dim3(320), 0, stream, partial,
                       n, nchunks, gsum);
    hipLaunchKernelGGL(combine_quantiles_kernel, dim3(1), dim3(kCombineThreads), 0, stream, gsum,
                       n, ngroups, out);
    return hipGetLastError();
}

}  // namespace bq
