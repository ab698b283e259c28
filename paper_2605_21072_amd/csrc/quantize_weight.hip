// Offline weight step for gfx950 (Sec. 3.2): input-channel L2 norms, Modified-Z-score +
// minimum-magnitude outlier detection (Eqs. (mad), (new_threshold)), alignment of the outlier
// count (Fig. "outlier patterns" caption), [outlier | normal] permutation and dual per-row scales
// with INT8 / INT4 rounding (Eq. (dual_scale), Eq. (quantization)).
//
// Every result is defined bit for bit, some of them through sums taken in a fixed order.  The kernels take
// those sums in parallel and PROVE that the order cannot matter: a sum of n non-negative doubles lies within
// n 2^-53 (relative) of the exact sum in any order, so when the whole interval around the parallel sum leads to the
// same fp32 norm (or the same comparison), the ordered sum does too.  The rare sums that fail the test (about
// 3 columns in 10^5 at 8960 rows) are redone in order.  W is streamed twice: once for the norms, once by
// the row quantizer; detection between them is one workgroup that sorts the norms.
//   kernel times, us        norms       detection    scales and codes
//   8960 x 1536, INT8       15 (397)    10.5 (258)   19 (32)
//   1536 x 8960, INT4, clip 14 (70)     18 (1316)    50 (4697: search, codes, packing)
// In brackets one thread per column, O(K^2) rankings, one thread per (row, block) for the search and byte stores.
#include "qarvd_common.h"

namespace {

struct DetectScalars {   // lives in the workspace
    int32_t n_det, K_o;
};

// ---- norms -------------------------------------------------------------------------------
// v[k] = (float) sqrt(sum_j W[j,k]^2), the sum in fp64 in ascending j.  A product of two floats is exact in fp64, so
// fma(d, d, S) rounds exactly as S + d * d does.
//
// Pass 1, bound by the 4 N K bytes it reads: a workgroup sums a chunk of rows for a slab of 256 columns (four waves
// take every fourth row, 1 KB of a row per load).  At most NORM_BLOCKS workgroups (four per CU), so the partial
// sums never exceed NORM_BLOCKS x 256 doubles whatever N and K are.
constexpr int NORM_BLOCKS = 1024;

template <bool VEC>
__global__ __launch_bounds__(256) void norm_partial_kernel(const float *__restrict__ W, int N, int K, int64_t ldw,
                                                           int rows_per_chunk, double *__restrict__ partial)
{
    __shared__ double part[4][256];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col0 = blockIdx.x * 256;
    const int r0 = blockIdx.y * rows_per_chunk, r1 = min(N, r0 + rows_per_chunk);
    double S[4] = {0.0, 0.0, 0.0, 0.0};
    // VEC: columns col0 + 4 lane + u by one 16-byte load; else columns col0 + lane + 64 u
    int col[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) col[u] = min(col0 + (VEC ? 4 * lane + u : lane + 64 * u), K - 1);
    auto row4 = [&](int r, float (&t)[4]) {
        const float *w = W + (size_t)r * ldw;
        if constexpr (VEC) {      // K % 4 == 0: the four columns are inside the matrix or the whole chunk is clamped
            const float4 f = *reinterpret_cast<const float4 *>(w + min(col0 + 4 * lane, K - 4));
            t[0] = f.x; t[1] = f.y; t[2] = f.z; t[3] = f.w;
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) t[u] = w[col[u]];
        }
    };
    auto add = [&](const float (&t)[4]) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double d = (double)t[u];
            S[u] = fma(d, d, S[u]);
        }
    };
    int r = r0 + wave;
    for (; r + 28 < r1; r += 32) {        // eight rows of this wave in flight
        float t[8][4];
#pragma unroll
        for (int i = 0; i < 8; ++i) row4(r + 4 * i, t[i]);
#pragma unroll
        for (int i = 0; i < 8; ++i) add(t[i]);
    }
    for (; r < r1; r += 4) {
        float t[4];
        row4(r, t);
        add(t);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) part[wave][VEC ? 4 * lane + u : lane + 64 * u] = S[u];
    __syncthreads();
    const int k = col0 + threadIdx.x;
    if (k < K)
        partial[(size_t)blockIdx.y * K + k] =
            (part[0][threadIdx.x] + part[1][threadIdx.x]) + (part[2][threadIdx.x] + part[3][threadIdx.x]);
}

// Pass 2: 64 columns per workgroup, sixteen threads per column.  With S the parallel sum and n = N terms, both S and the
// ordered sum are within n u / (1 - n u) of the exact one (u = 2^-53), so the ordered sum lies in
// S (1 -+ 2.5 (n + 2) u), which leaves room for the roundings of the bounds themselves.  sqrt and the conversion
// to float are monotone: equal ends mean that the ordered sum gives this float.  A sum is NaN if a term is, in any order.
__global__ __launch_bounds__(1024) void norm_final_kernel(const double *__restrict__ partial, int chunks,
                                                         const float *__restrict__ W, int N, int K, int64_t ldw,
                                                         float *__restrict__ v, float *__restrict__ v_out)
{
    __shared__ double part[16][64];
    __shared__ unsigned long long redo;
    __shared__ float stage[1024];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int k = blockIdx.x * 64 + lane;
    const double *p = partial + min(k, K - 1);
    double S = 0.0;
    int c = wave;
    for (; c + 112 < chunks; c += 128) {
        double t[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) t[i] = p[(size_t)(c + 16 * i) * K];
#pragma unroll
        for (int i = 0; i < 8; ++i) S += t[i];
    }
#pragma unroll 4
    for (; c < chunks; c += 16) S += p[(size_t)c * K];
    part[wave][lane] = S;
    __syncthreads();
    if (wave == 0) {
        S = 0.0;
#pragma unroll
        for (int w = 0; w < 16; ++w) S += part[w][lane];
        const double e = 2.5 * ((double)N + 2.0) * 0x1p-53;
        const float lo = (float)sqrt(S * (1.0 - e)), hi = (float)sqrt(S * (1.0 + e));
        const bool settled = lo == hi || S != S;
        const unsigned long long bad = __ballot(k < K && !settled);
        if (k < K && settled) {
            v[k] = lo;
            if (v_out) v_out[k] = lo;
        }
        if (lane == 0) redo = bad;
    }
    __syncthreads();
    for (unsigned long long m = redo; m; m &= m - 1) {       // in order, 1024 rows at a time through LDS
        const int kr = blockIdx.x * 64 + __builtin_ctzll(m);
        double T = 0.0;
        for (int r0 = 0; r0 < N; r0 += 1024) {
            if (r0 + (int)threadIdx.x < N) stage[threadIdx.x] = W[(size_t)(r0 + threadIdx.x) * ldw + kr];
            __syncthreads();
            if (threadIdx.x == 0) {
                const int lim = min(1024, N - r0);
                for (int i = 0; i < lim; ++i) {
                    const double d = (double)stage[i];
                    T = fma(d, d, T);
                }
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            const float f = (float)sqrt(T);
            v[kr] = f;
            if (v_out) v_out[kr] = f;
        }
    }
}

// ---- detection by searches --------------------------------------------------------------------
// For more than 16384 channels, and for norms that the sort below gives up on.  Norms are non-negative floats, so their
// bit patterns order as they do, and any order statistic is found by bisecting the pattern range with counts, and once at most 64
// values are left in the range they are ranked directly: three selections (median, MAD, the K_o-th largest norm) of
// about ten counts each.  The MAD's doubles are bisected by their upper 32 bits first.
// KPT: keys per thread, kept in registers through a selection's counts, the norms in LDS; 0 (K > 16384): keys are recomputed from
// memory.  Code that runs once is fetched from memory at about a microsecond per kilobyte, so every loop but the count itself is
// rolled.
template <int KPT, int NT>
__device__ __forceinline__ void detect_by_search(const float *v, int K, double c, double alpha, int align, const uint8_t *__restrict__ forced,
                                                 DetectScalars *sc, int32_t *__restrict__ perm)
{
    constexpr int R = KPT > 0 ? KPT : 1, NW = NT / 64;
    __shared__ int red[2][NW];
    __shared__ __align__(16) unsigned long long cand[64];
    __shared__ int n_cand, rank[64];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    int buf = 0;

    double med = 0.0;
    bool devs = false;                         // keys: deviations from the median (upper halves) instead of norms
    auto value = [&](int i) { return v[i]; };
    auto dev = [&](float f) { return (unsigned long long)__double_as_longlong(fabs((double)f - med)); };
    auto key_of = [&](float f) { return devs ? (unsigned)(dev(f) >> 32) : __float_as_uint(f); };
    unsigned key[R];                           // keys of the selection at hand, ~0 past the end
    // workgroup sum / minimum: one barrier each, two alternating LDS buffers
    auto all_sum = [&](int n) {
        n = wave_sum_all(n);
        if (lane == 0) red[buf][wave] = n;
        __syncthreads();
        n = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) n += red[buf][w];
        buf ^= 1;
        return __builtin_amdgcn_readfirstlane(n);      // (keeps the bisection in scalar registers)
    };
    auto all_min = [&](unsigned m) {
        m = wave_min_all(m);
        if (lane == 0) red[buf][wave] = (int)m;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < NW; ++w) m = min(m, (unsigned)red[buf][w]);
        buf ^= 1;
        return (unsigned)__builtin_amdgcn_readfirstlane((int)m);
    };
    auto count = [&](auto pred) __attribute__((always_inline)) {              // number of values with pred(index, value)
        int n = 0;
#pragma unroll 4
        for (int i = t; i < K; i += NT) n += pred(i, value(i)) ? 1 : 0;
        return all_sum(n);
    };

    int K_o = 0;
    unsigned sel_min = ~0u;                    // selected: channels with a pattern above this one,
    int cut = K - 1;                           // and those equal to it up to this index
    // selections: 0 the median of the norms, 1 the median of the deviations, 2 the smallest of the K_o largest norms
#pragma unroll 1
    for (int stage = forced ? 3 : 0; stage < 3; ++stage) {
        devs = stage == 1;
        unsigned min_key = ~0u, max_inv = ~0u;
        if constexpr (KPT > 0) {
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const int i = u * NT + t;
                key[u] = i < K ? key_of(v[i]) : ~0u;
                min_key = min(min_key, key[u]);
                max_inv = i < K ? min(max_inv, ~key[u]) : max_inv;
            }
        } else {
            for (int i = t; i < K; i += NT) {
                const unsigned q = key_of(v[i]);
                min_key = min(min_key, q);
                max_inv = min(max_inv, ~q);
            }
        }
        min_key = all_min(min_key);
        const unsigned max_key = ~all_min(max_inv);
        // k-th smallest (from 0) of the 32- or (deviations) 64-bit patterns; `second` is the next order statistic
        int k = stage < 2 ? (K - 1) / 2 : K - K_o;
        unsigned long long first = 0, second = 0;
#pragma unroll 1
        for (int rep = 0; rep < 2; ++rep) {
            unsigned lo = min_key, hi = max_key;
            int below = 0, upto = K;           // values below the range, and up to its end
            while (lo < hi && upto - below > 64) {
                const unsigned mid = lo + ((hi - lo) >> 1);       // < hi: never the key past the end
                int n = 0;
                if constexpr (KPT > 0) {
#pragma unroll
                    for (int u = 0; u < R; ++u) n += key[u] <= mid ? 1 : 0;
                } else {
                    for (int i = t; i < K; i += NT) n += key_of(v[i]) <= mid ? 1 : 0;
                }
                n = all_sum(n);
                if (n > k) {
                    hi = mid;
                    upto = n;
                } else {
                    lo = mid + 1;
                    below = n;
                }
            }
            unsigned long long lo2 = devs ? (unsigned long long)lo << 32 : lo;
            unsigned long long hi2 = devs ? ((unsigned long long)hi << 32) | 0xFFFFFFFFull : hi;
            while (lo2 < hi2 && upto - below > 64) {              // more than 64 deviations share the upper half
                const unsigned long long mid = lo2 + ((hi2 - lo2) >> 1);
                const int n = count([&](int, float f) { return dev(f) <= mid; });
                if (n > k) {
                    hi2 = mid;
                    upto = n;
                } else {
                    lo2 = mid + 1;
                    below = n;
                }
            }
            unsigned long long kth = lo2;      // lo2 == hi2: every value left is this one
            bool have_next = false;
            if (lo2 < hi2) {
                if (t == 0) n_cand = 0;
                if (t < 64) rank[t] = 0;
                __syncthreads();
#pragma unroll 4
                for (int i = t; i < K; i += NT) {
                    const float f = value(i);
                    const unsigned long long q = devs ? dev(f) : (unsigned long long)__float_as_uint(f);
                    if (q >= lo2 && q <= hi2) {
                        const int slot = atomicAdd(&n_cand, 1);
                        if (slot < 64) cand[slot] = q;
                    }
                }
                __syncthreads();
                const int m = min(n_cand, 64);
                const unsigned long long mine = lane < m ? cand[lane] : ~0ull;
                int r = 0;                     // every wave compares with its share of the candidates
#pragma unroll
                for (int u = 0; u < 64 / NW; ++u) {
                    const int j = wave * (64 / NW) + u;
                    const unsigned long long o = cand[j];
                    r += j < m && (o < mine || (o == mine && j < lane)) ? 1 : 0;
                }
                if (r) atomicAdd(&rank[lane], r);
                __syncthreads();
                r = rank[lane];
                const unsigned long long who = __ballot(lane < m && r == k - below);
                const unsigned long long next = __ballot(lane < m && r == k + 1 - below);
                if (who) kth = cand[__builtin_ctzll(who)];
                if (next) {
                    have_next = true;
                    second = cand[__builtin_ctzll(next)];
                }
                __syncthreads();               // cand and n_cand may be rewritten
            } else if (k + 1 < upto) {
                have_next = true;
                second = kth;
            }
            if (rep == 0) first = kth;
            else second = kth;
            if (stage == 2 || (K & 1) || have_next) break;
            ++k;                               // even K and the upper middle lies beyond the range: select it too
        }
        if (stage < 2) {                       // median: mean of the two middle order statistics (odd K: the middle one)
            const double a = devs ? __longlong_as_double((long long)first) : (double)__uint_as_float((unsigned)first);
            const double b = devs ? __longlong_as_double((long long)second) : (double)__uint_as_float((unsigned)second);
            const double middle = (K & 1) ? a : (b + a) / 2.0;
            if (stage == 0) {
                med = middle;
            } else {
                double T1 = c * middle;        // middle = MAD
                T1 = med + T1;
                const double T2 = alpha * med;
                const double T = T1 > T2 ? T1 : T2;
                const int n_det = count([&](int, float f) { return (double)f > T; });
                if (t == 0) sc->n_det = n_det;
                if (n_det == 0) break;
                const long long up = ((long long)n_det + align - 1) / align * align;
                K_o = up > K ? K : (int)up;
            }
        } else {
            sel_min = (unsigned)first;
            const int need = K_o - count([&](int, float f) { return __float_as_uint(f) > sel_min; });
            const int equal = count([&](int, float f) { return __float_as_uint(f) == sel_min; });
            for (int lo = 0; need < equal && lo < cut;) {         // ties: the smaller indices
                const int mid = (lo + cut) / 2;
                if (count([&](int i, float f) { return __float_as_uint(f) == sel_min && i <= mid; }) >= need) cut = mid;
                else lo = mid + 1;
            }
        }
    }
    // Stable partition: perm = [selected ascending | rest ascending].  A thread takes P consecutive channels (P odd: no
    // bank conflicts); the selected channels before them are counted over the lanes below it, bit by bit of their
    // counts, and over the waves before.
    auto selected = [&](int i) {
        if (i >= K) return false;
        if (forced) return forced[i] != 0;
        const unsigned q = __float_as_uint(value(i));
        return K_o > 0 && (q > sel_min || (q == sel_min && i <= cut));
    };
    const int P = ((K + NT - 1) / NT) | 1, i0 = t * P;
    int n = 0;
#pragma unroll 4
    for (int j = 0; j < P; ++j) n += selected(i0 + j) ? 1 : 0;
    int so = 0, wave_n = 0;
#pragma unroll
    for (int b = 0; b < (KPT > 0 ? 6 : 9); ++b) {        // P <= 33 (K <= 16384), 131 (K <= QARVD_MAX_K)
        const unsigned long long bits = __ballot((n >> b) & 1);
        so += __popcll(bits & ((1ull << lane) - 1)) << b;
        wave_n += __popcll(bits) << b;
    }
    if (lane == 0) red[buf][wave] = wave_n;
    __syncthreads();
    int all = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        so += w < wave ? red[buf][w] : 0;
        all += red[buf][w];
    }
    if (forced) K_o = all;
#pragma unroll 4
    for (int j = 0; j < P; ++j) {
        const int i = i0 + j;
        const bool s = selected(i);
        if (i < K) perm[s ? so : K_o + (i - so)] = i;
        so += s ? 1 : 0;
    }
    if (t == 0) sc->K_o = K_o;
}

template <int NT>
__global__ __launch_bounds__(NT) void detect_long_kernel(const float *__restrict__ v, int K, double c, double alpha, int align,
                                                         const uint8_t *__restrict__ forced, DetectScalars *sc, int32_t *__restrict__ perm)
{
    detect_by_search<0, NT>(v, K, c, alpha, align, forced, sc, perm);
}

// ---- detection and permutation: one workgroup ------------------------------------------------
// The norms are sorted first; then the median is read off.  The deviations from it fall towards the median and rise after it, so the
// k + 1 smallest of them are k + 1 neighbours, and the k-th (from 0) is the smallest over all windows of k + 1 neighbours of the larger
// of the two deviations at the window's ends: one pass and one reduction for the MAD (for an even K the next one too).  (Subtraction
// and rounding are monotone, and infinities and NaNs have the largest patterns, so this holds for the rounded values.)
//
// The sort: bit patterns (which order as the norms do) are counted in 511 coarse bins over their range, zeros in one of their own (they
// would make a bin a quarter of an octave wide, and nearly all others would fall into one or two); a pattern's place within its
// bin, times the number of patterns there, points to one of 2 K fine bins (K beyond 9216, where the LDS holds no more); the
// fine counts summed up give every pattern its bin's first place, and within a bin (5 to 8 patterns at most in ordinary layers) each
// counts the smaller ones.
// A bin of more than 48 patterns is not counted through.  It is nearly always one of equal norms (channels that are dead, padding or
// copies), whose order is of no matter; up to 32 patterns that differ from their crowded bins' first ones are placed among
// them one by one.  More, thousands of norms within bits of each other but not equal, take the searches above.
// One workgroup on an otherwise idle chip is bound by latency, a barrier and an LDS round trip per step; the coarse counters
// are kept sixteen times, since nearly all norms fall into a few of those bins.
// Against the three searches alone (about ten counts of all values each), us at K = 1536, 5120 and 8960: ordinary norms 22.7 -> 10.9, 28.8
// -> 16.0, 33.8 -> 18.3; 64 channels zero 24.1 -> 11.9, 31.9 -> 17.7, 36.8 -> 20.4 (by the searches behind the sort's first half, from
// LDS, 39, 55 and 63); half of them zero 46 -> 12, 62 -> 20, 74 -> 23; 300 equal ones among the others 21.5 -> 11.1, 28.5 -> 18.3,
// 34.9 -> 21.7; half of them within 20 bits of 1 (the searches take over) 31 -> 36, 40 -> 45, 87 -> 96.  All-pairs ranks
// counted by the whole chip and summed up by one workgroup took 10 and 24.  Half of what is left at 8960 is LDS reads at random
// places: counting within bins (5 us; with one fine bin a norm instead of two 6.2), scattering and sorting back.
constexpr int COARSE = 512, COPIES = 16, BIN_MAX = 48, ODD_MAX = 32;
constexpr int fine_per_norm(int R) { return R <= 10 ? 2 : 1; }      // (what the LDS holds)

template <int R, int NT>      // K <= R NT
__global__ __launch_bounds__(NT) void detect_kernel(const float *__restrict__ v, int K, double c, double alpha, int align,
                                                    const uint8_t *__restrict__ forced, DetectScalars *sc, int32_t *__restrict__ perm)
{
    constexpr int NW = NT / 64, E = R * NW, F = fine_per_norm(R);       // E: groups of 64 channels
    static_assert(E <= 256, "four groups a lane");
    typedef unsigned long long u64;
    __shared__ u64 least[2][NW];
    __shared__ int red[4][NW], before[E], coarse_first[COARSE + 1], n_odd;
    __shared__ int2 odd[ODD_MAX];
    extern __shared__ __align__(16) unsigned lds[];        // sorted [K] (first the coarse counters) | fine [F K + 1]
    unsigned *const sorted = lds;
    int *const coarse = reinterpret_cast<int *>(lds);
    int *const fine = reinterpret_cast<int *>(lds) + max(K, COARSE * COPIES);
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;

    // running sums over the workgroup: what the threads before this one hold together; one barrier (slot: a buffer of its own)
    auto sum_before = [&](int n, int slot) {
        const int run = wave_scan(n);
        if (lane == 63) red[slot][wave] = run;
        __syncthreads();
        int base = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) base += w < wave ? red[slot][w] : 0;
        return base + run - n;
    };
    auto total = [&](int slot) {
        int n = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) n += red[slot][w];
        return n;
    };

    unsigned key[R];
    int K_o = 0, cut = K - 1;
    unsigned sel_min = ~0u;                    // selected: channels with a pattern above this one, and those equal to it up to `cut`
    if (!forced) {
#pragma unroll
        for (int u = 0; u < R; ++u) key[u] = __float_as_uint(v[min(u * NT + t, K - 1)]);
        for (int i = t; i < COARSE * COPIES / 4; i += NT) reinterpret_cast<int4 *>(coarse)[i] = make_int4(0, 0, 0, 0);
        for (int i = t; i <= F * K; i += NT) fine[i] = 0;
        if (t == 0) n_odd = 0;
        unsigned lo = ~0u, hi_inv = ~0u;
#pragma unroll
        for (int u = 0; u < R; ++u) {          // (the last one again past the end)
            lo = min(lo, key[u] ? key[u] : ~0u);
            hi_inv = min(hi_inv, ~key[u]);
        }
        lo = wave_min_all(lo);
        hi_inv = wave_min_all(hi_inv);
        if (lane == 0) {
            red[0][wave] = (int)lo;
            red[1][wave] = (int)hi_inv;
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            lo = min(lo, (unsigned)red[0][w]);
            hi_inv = min(hi_inv, (unsigned)red[1][w]);
        }
        const unsigned range = ~hi_inv - lo;                           // (all zero: 1)
        int shift = max(0, 32 - 9 - __clz((int)range));                // (a range of 0 has 32 leading zeros)
        if (range >> shift > COARSE - 2) ++shift;                      // bin 0 holds the zeros
        auto coarse_bin = [&](unsigned q) { return q ? 1 + ((q - lo) >> shift) : 0; };
#pragma unroll
        for (int u = 0; u < R; ++u)
            if (u * NT + t < K) atomicAdd(&coarse[coarse_bin(key[u]) * COPIES + (lane & (COPIES - 1))], 1);
        __syncthreads();
        {
            constexpr int B = COARSE / NT > 0 ? COARSE / NT : 1;       // bins of a thread
            int n[B], all = 0;
#pragma unroll
            for (int b = 0; b < B; ++b) {
                n[b] = 0;
                if (t * B + b < COARSE) {
#pragma unroll
                    for (int q = 0; q < COPIES / 4; ++q) {
                        const int4 o = reinterpret_cast<const int4 *>(coarse)[(t * B + b) * (COPIES / 4) + q];
                        n[b] += (o.x + o.y) + (o.z + o.w);
                    }
                }
                all += n[b];
            }
            int first = sum_before(all, 2);
#pragma unroll
            for (int b = 0; b < B; ++b) {
                if (t * B + b <= COARSE) coarse_first[t * B + b] = first;
                first += n[b];
            }
            if (t == NT - 1 && NT * B == COARSE) coarse_first[COARSE] = first;
        }
        __syncthreads();
        int place[R], slot[R];
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const unsigned b = coarse_bin(key[u]), in_bin = key[u] ? (key[u] - lo) & ((1u << shift) - 1) : 0;
            const int first = coarse_first[b], n = coarse_first[b + 1] - first;
            place[u] = F * first + (int)(((u64)in_bin * (unsigned)(F * n)) >> shift);
            slot[u] = u * NT + t < K ? atomicAdd(&fine[place[u]], 1) : 0;
        }
        __syncthreads();
        {
            constexpr int P = (F * R) | 1;                                   // neighbouring fine bins (odd: no bank conflicts)
            const int i0 = t * P;
            int n[P], all = 0, most = 0;
#pragma unroll
            for (int j = 0; j < P; ++j) n[j] = i0 + j < F * K ? fine[i0 + j] : 0;
#pragma unroll
            for (int j = 0; j < P; ++j) {
                all += n[j];
                most = max(most, n[j]);
            }
            if (__ballot(most > BIN_MAX) && lane == 0) least[0][wave] = 1;
            else if (lane == 0) least[0][wave] = 0;
            int first = sum_before(all, 3);
#pragma unroll
            for (int j = 0; j < P; ++j) {
                if (i0 + j < F * K) fine[i0 + j] = first;
                first += n[j];
            }
            if (t == 0) fine[F * K] = K;
        }
        u64 crowded = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) crowded |= least[0][w];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const int first = fine[place[u]];
            if (u * NT + t < K) sorted[first + slot[u]] = key[u];
            slot[u] += first;
        }
        __syncthreads();
        int at[R], end[R];
#pragma unroll
        for (int u = 0; u < R; ++u) {
            end[u] = fine[place[u] + 1];
            at[u] = place[u] = fine[place[u]];
        }
        if (crowded) {                         // (the same for all threads)
#pragma unroll
            for (int u = 0; u < R; ++u)
                if (u * NT + t < K && end[u] - place[u] > BIN_MAX && sorted[place[u]] != key[u]) {
                    const int n = atomicAdd(&n_odd, 1);
                    if (n < ODD_MAX) odd[n] = make_int2(slot[u], (int)key[u]);
                }
            __syncthreads();
            const int n = n_odd;
            if (n > ODD_MAX) {
#pragma unroll
                for (int u = 0; u < R; ++u)
                    if (u * NT + t < K) sorted[u * NT + t] = key[u];
                __syncthreads();
                detect_by_search<R, NT>(reinterpret_cast<const float *>(sorted), K, c, alpha, align, nullptr, sc, perm);
                return;
            }
            // In a crowded bin `most` is the pattern in its first place.  Places of equal patterns follow their slots, less the odd ones
            // before them, plus the smaller odd ones; an odd one counts the smaller odd ones, and all others if it is above them.
#pragma unroll
            for (int u = 0; u < R; ++u) {
                if (end[u] - place[u] <= BIN_MAX) continue;
                const unsigned most = sorted[place[u]];
                int smaller = 0, ahead = 0, here = 0;          // odd ones of this bin
                for (int j = 0; j < n; ++j) {
                    const int2 o = odd[j];
                    if (o.x < place[u] || o.x >= end[u]) continue;
                    smaller += (unsigned)o.y < key[u] || ((unsigned)o.y == key[u] && o.x < slot[u]) ? 1 : 0;
                    ahead += o.x < slot[u] ? 1 : 0;
                    ++here;
                }
                at[u] = key[u] == most ? slot[u] + smaller - ahead : place[u] + smaller + (key[u] > most ? end[u] - place[u] - here : 0);
                end[u] = place[u];             // nothing left to count below
            }
        }
        auto count_smaller = [&](int u, int s0) {                      // among four patterns of the bin from s0 on, read together
            unsigned o[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) o[s] = sorted[min(place[u] + s0 + s, K - 1)];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int j = place[u] + s0 + s;
                at[u] += j < end[u] && (o[s] < key[u] || (o[s] == key[u] && j < slot[u])) ? 1 : 0;
            }
        };
#pragma unroll
        for (int u = 0; u < R; ++u) count_smaller(u, 0);
#pragma unroll
        for (int u = 0; u < R; ++u)
            for (int s0 = 4; __ballot(place[u] + s0 < end[u]); s0 += 4) count_smaller(u, s0);
        __syncthreads();
#pragma unroll
        for (int u = 0; u < R; ++u)
            if (u * NT + t < K) sorted[at[u]] = key[u];
        __syncthreads();

        const int k = (K - 1) / 2;
        auto norm = [&](int i) { return (double)__uint_as_float(sorted[i]); };
        // median: mean of the two middle order statistics (odd K: the middle one)
        const double m0 = norm(k), m1 = norm(min(k + 1, K - 1));
        const double med = (K & 1) ? m0 : (m1 + m0) / 2.0;
        auto dev = [&](int i) { return (u64)__double_as_longlong(fabs(norm(i) - med)); };
        u64 m[2] = {~0ull, ~0ull};
        for (int i = t; i + k < K; i += NT) {
            const u64 d = dev(i), e = dev(i + k);
            m[0] = min(m[0], max(d, e));
            if (i + k + 1 < K) m[1] = min(m[1], max(d, dev(i + k + 1)));
        }
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const unsigned h = wave_min_all((unsigned)(m[r] >> 32));
            const unsigned l = wave_min_all((unsigned)(m[r] >> 32) == h ? (unsigned)m[r] : ~0u);
            if (lane == 0) least[r][wave] = (u64)h << 32 | l;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            m[r] = least[r][0];
#pragma unroll
            for (int w = 1; w < NW; ++w) m[r] = min(m[r], least[r][w]);
        }
        const double a = __longlong_as_double((long long)m[0]), b = __longlong_as_double((long long)m[1]);
        const double mad = (K & 1) ? a : (b + a) / 2.0;
        double T1 = c * mad;
        T1 = med + T1;
        const double T2 = alpha * med;
        const double T = T1 > T2 ? T1 : T2;
        int n_det = 0;
#pragma unroll
        for (int u = 0; u < R; ++u) n_det += __popcll(__ballot(u * NT + t < K && (double)__uint_as_float(key[u]) > T));
        if (lane == 0) red[0][wave] = n_det;
        __syncthreads();
        n_det = total(0);
        if (t == 0) sc->n_det = n_det;
        const long long up = ((long long)n_det + align - 1) / align * align;
        K_o = up > K ? K : (int)up;
        if (K_o > 0) {
            sel_min = sorted[K - K_o];
            // equal norms at the edge of the block: the smaller channels
            const bool tie = K_o < K && sorted[K - K_o - 1] == sel_min;
            if (tie) {
                int above = 0;
#pragma unroll
                for (int u = 0; u < R; ++u) above += __popcll(__ballot(u * NT + t < K && key[u] > sel_min));
                if (lane == 0) red[1][wave] = above;
                __syncthreads();
                const int need = K_o - total(1);
                for (int first = 0; first < cut;) {
                    const int mid = (first + cut) / 2;
                    int n = 0;
#pragma unroll
                    for (int u = 0; u < R; ++u) n += __popcll(__ballot(u * NT + t <= mid && key[u] == sel_min));
                    __syncthreads();
                    if (lane == 0) red[1][wave] = n;
                    __syncthreads();
                    if (total(1) >= need) cut = mid;
                    else first = mid + 1;
                }
            }
        }
    }
    // Stable partition: perm = [selected ascending | rest ascending].  A group is 64 neighbouring channels; the selected ones before
    // a channel are those of the groups before its own and those of the lanes below.
    u64 mask[R];
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const int i = u * NT + t;
        mask[u] = __ballot(i < K && (forced ? forced[i] != 0 : K_o > 0 && (key[u] > sel_min || (key[u] == sel_min && i <= cut))));
        if (lane == 0) before[u * NW + wave] = __popcll(mask[u]);
    }
    __syncthreads();
    if (wave == 0) {                            // running sums over the groups, four (or fewer) a lane
        constexpr int G = (E + 63) / 64;
        int n[G], all = 0;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int e = lane * G + g;
            n[g] = e < E ? before[e] : 0;
            all += n[g];
        }
        int run = wave_scan(all);
        if (lane == 63) red[2][0] = run;
        run -= all;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int e = lane * G + g;
            if (e < E) before[e] = run;
            run += n[g];
        }
    }
    __syncthreads();
    if (forced) K_o = red[2][0];
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const int i = u * NT + t;
        const int so = before[u * NW + wave] + __popcll(mask[u] & ((1ull << lane) - 1));
        if (i < K) perm[(mask[u] >> lane) & 1 ? so : K_o + (i - so)] = i;
    }
    if (t == 0) sc->K_o = K_o;
}

// ---- dual scales + codes -------------------------------------------------------------------
// A row of W in PACKED order in the registers of a workgroup (NT = 64: of one wave).  Wave w holds the chunks of 256 packed
// positions w, w + NT / 64, ...: in chunk c its lane l holds the positions 256 chunk + 64 e + l, e < 4.  The
// permutation is applied by the loads themselves: the channel offsets of a lane's positions are the same for every row
// and stay in registers, and since [outlier | normal] keeps both blocks in ascending order, the 64 addresses of a
// load are consecutive but for the outliers left out.  So there is no LDS image, no position table and no byte
// scatter, and rows of any length and alignment take the same path.  (Four consecutive positions per lane instead,
// which need no transpose before the store, spread each load over 1 KB: 26 us against 21 for 8960 x 1536.)
template <int CH, int NT>
struct PackedRow {
    uint32_t off[CH][4];     // byte offset in the row of every position (pads: some channel of the same block)
    int n_off, end_o, end_n; // outlier block [0, end_o), normal block [n_off, end_n)
    int kp;                  // packed extent
    int base[CH];            // first position of the chunk (wave-uniform)

    // wave: index of the wave among those that share the row
    __device__ __forceinline__ void init(const int32_t *__restrict__ perm, int K, int K_o, int wave, int lane)
    {
        n_off = (K_o + 31) / 32 * 32;
        end_o = K_o;
        end_n = n_off + (K - K_o);
        kp = (end_n + 127) / 128 * 128;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            base[c] = 256 * (wave + c * (NT / 64));
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int p = base[c] + 64 * e + lane;
                const int q = p < n_off ? min(p, K_o - 1) : min(K_o + (p - n_off), K - 1);
                off[c][e] = 4u * (uint32_t)perm[max(q, 0)];
            }
        }
    }
    // w wave-uniform.  Raw buffer loads: the row's base sits in scalar registers and a position costs one 32-bit offset
    // (the compiler keeps 64-bit addresses per position for global loads: twice the registers).
    __device__ __forceinline__ void load(const float *w, int K, float (&x)[CH][4]) const
    {
#if defined(__HIP_DEVICE_COMPILE__)
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(w), 0, 4 * K, 0x00020000);
#pragma unroll
        for (int c = 0; c < CH; ++c)
            if (base[c] < kp) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    x[c][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)off[c][e], 0, 0));
            }
#endif
    }
};

struct RowsArgs {
    const float *W;
    int64_t ldw;
    const int32_t *perm;
    const DetectScalars *sc;
    uint8_t *out;            // INT8: one byte per position; INT4: two positions per byte
    int64_t ldo;             // bytes
    float *s_normal, *s_outlier;
    float qmax;              // 127 or 7
    int32_t N, K;
};

// Codes of a row and their store.  A lane's four codes of a chunk lie 64 positions apart; two exchanges inside each group of
// four lanes (bytes i of lanes 4a .. 4a+3 belong together) turn them into the dword of positions 64 (l & 3) + 4 (l >> 2) ..+3
// of the chunk, so that one store writes the 256 bytes.
//
// INT4 packing: the codes of each aligned group of 16 packed positions g go into 8 bytes; byte i < 4
// holds positions 16g+i (low nibble) and 16g+4+i (high nibble), byte 4+i positions 16g+8+i and
// 16g+12+i.  (Shifting a packed dword left by 4 and masking 0xF0F0F0F0 then yields four consecutive
// codes, each times 16, in byte order; masking the dword itself the next four.)  So an even dword of codes and
// the odd one after it, four lanes up, make one packed dword.
template <int CH, int NT>
__device__ __forceinline__ void store_codes(const RowsArgs &a, const PackedRow<CH, NT> &pr, const float (&x)[CH][4], int row, int lane,
                                            const ExactQuotient &qo, const ExactQuotient &qn)
{
    constexpr float MAGIC = 12582912.0f;       // 1.5 * 2^23: the sum rounds half-to-even, the code is its low byte
    uint8_t *out = a.out + (size_t)row * a.ldo;
    const bool w4 = a.qmax < 8.0f;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        if (pr.base[c] >= pr.kp) continue;
        uint32_t b[4];
        if (pr.base[c] >= pr.n_off && pr.base[c] + 256 <= pr.end_n) {        // normal channels only
#pragma unroll
            for (int e = 0; e < 4; ++e)
                b[e] = __float_as_uint(qn.clamped(x[c][e]) + MAGIC);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int p = pr.base[c] + 64 * e + lane;
                const bool is_o = p < pr.n_off;
                ExactQuotient q = qn;
                q.s = is_o ? qo.s : qn.s;
                q.rs = is_o ? qo.rs : qn.rs;
                q.bound = is_o ? qo.bound : qn.bound;
                const float f = p < (is_o ? pr.end_o : pr.end_n) ? x[c][e] : 0.0f;      // pads
                b[e] = __float_as_uint(q.clamped(f) + MAGIC);
            }
        }
        uint32_t w = __builtin_amdgcn_perm(__builtin_amdgcn_perm(b[3], b[2], 0x0c0c0400u), __builtin_amdgcn_perm(b[1], b[0], 0x0c0c0400u),
                                           0x05040100u);
        // 4 x 4 byte transpose over lanes 4a .. 4a+3: bytes of odd / even pairs with lane ^ 1, then halves with lane ^ 2
        const uint32_t w1 = (uint32_t)__builtin_amdgcn_mov_dpp((int)w, 0xB1, 0xF, 0xF, true);
        w = __builtin_amdgcn_perm(w1, w, (lane & 1) ? 0x03070105u : 0x06020400u);
        const uint32_t w2 = (uint32_t)__builtin_amdgcn_mov_dpp((int)w, 0x4E, 0xF, 0xF, true);
        w = __builtin_amdgcn_perm(w2, w, (lane & 2) ? 0x03020706u : 0x05040100u);
        const int p0 = pr.base[c] + 64 * (lane & 3) + 4 * (lane >> 2);
        if (!w4) {
            if (p0 < pr.kp) *reinterpret_cast<uint32_t *>(out + p0) = w;
        } else {
            const uint32_t up = (uint32_t)__builtin_amdgcn_ds_swizzle((int)w, 0x101F);     // lane ^ 4
            if (!(lane & 4) && p0 < pr.kp)
                *reinterpret_cast<uint32_t *>(out + p0 / 2) = (w & 0x0F0F0F0Fu) | ((up & 0x0F0F0F0Fu) << 4);
        }
    }
}

// The same for scales outside the range of the exact quotient above (rows of magnitudes around 1e-30 and below, or 1e30 and
// above): IEEE divisions, one position per thread, the row gathered again.
template <int NT>
__device__ __forceinline__ void store_codes_far(const RowsArgs &a, int row, int t, int K_o, float so, float sn)
{
    const float *w = a.W + (size_t)row * a.ldw;
    uint8_t *out = a.out + (size_t)row * a.ldo;
    const int n_off = (K_o + 31) / 32 * 32, end_n = n_off + (a.K - K_o), kp = (end_n + 127) / 128 * 128;
    auto code = [&](int p) {
        if (p < n_off) return p < K_o ? quantize_sym(w[a.perm[p]], so, a.qmax) : 0;
        return p < end_n ? quantize_sym(w[a.perm[K_o + (p - n_off)]], sn, a.qmax) : 0;
    };
    if (a.qmax > 8.0f)
        for (int p = t; p < kp; p += NT) out[p] = (uint8_t)code(p);
    else
        for (int b = t; b < kp / 2; b += NT) {
            const int p = 16 * (b >> 3) + (b & 3) + 8 * ((b >> 2) & 1);
            out[b] = (uint8_t)((code(p) & 15) | ((code(p + 4) & 15) << 4));
        }
}

// Absmax scales.  NT = 64: four independent rows per workgroup, one per wave, no barrier; else one row per workgroup.
// Bound by the 4 N K bytes read and N K written (3.6 TB/s at 8960 x 1536, of which 4 us are the first row's latency).
template <int CH, int NT>
__global__ __launch_bounds__(NT == 64 ? 256 : NT) void weight_rows_kernel(RowsArgs a)
{
    constexpr int RW = NT == 64 ? 4 : 1, NWAVE = NT / 64;
    __shared__ float red[2][2][NWAVE];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int K_o = a.sc->K_o;
    PackedRow<CH, NT> pr;
    pr.init(a.perm, a.K, K_o, NT == 64 ? 0 : wave, lane);
    const int stride = gridDim.x * RW;
    int row = blockIdx.x * RW + (NT == 64 ? wave : 0);
    float x[CH][4], xn[CH][4];
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) x[c][e] = xn[c][e] = 0.0f;
    if (row < a.N) pr.load(a.W + (size_t)row * a.ldw, a.K, x);
    for (int buf = 0; row < a.N; row += stride, buf ^= 1) {
        if (row + stride < a.N) pr.load(a.W + (size_t)(row + stride) * a.ldw, a.K, xn);      // in flight under this row's work
        float m_o = 0.0f, m_n = 0.0f;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            if (pr.base[c] >= pr.n_off) {
                m_n = fmaxf(m_n, fmaxf(fmaxf(fabsf(x[c][0]), fabsf(x[c][1])), fmaxf(fabsf(x[c][2]), fabsf(x[c][3]))));
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool is_o = pr.base[c] + 64 * e + lane < pr.n_off;
                    m_o = fmaxf(m_o, is_o ? fabsf(x[c][e]) : 0.0f);
                    m_n = fmaxf(m_n, is_o ? 0.0f : fabsf(x[c][e]));
                }
            }
        }
        m_o = wave_max_all(m_o);
        m_n = wave_max_all(m_n);
        if constexpr (NT > 64) {
            if (lane == 0) {
                red[buf][0][wave] = m_o;
                red[buf][1][wave] = m_n;
            }
            __syncthreads();
#pragma unroll
            for (int w = 0; w < NWAVE; ++w) {
                m_o = fmaxf(m_o, red[buf][0][w]);
                m_n = fmaxf(m_n, red[buf][1][w]);
            }
        }
        // a block without channels holds only pads (which load some channel of the row): its scale is zero
        const float so = K_o > 0 ? m_o / a.qmax : 0.0f, sn = K_o < a.K ? m_n / a.qmax : 0.0f;
        if (lane == 0 && (NT == 64 || wave == 0)) {
            a.s_outlier[row] = so;
            a.s_normal[row] = sn;
        }
        const ExactQuotient qo(so, a.qmax), qn(sn, a.qmax);
        if (qo.exact() && qn.exact()) store_codes<CH, NT>(a, pr, x, row, lane, qo, qn);
        else store_codes_far<NT>(a, row, NT == 64 ? lane : (int)threadIdx.x, K_o, so, sn);
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) x[c][e] = xn[c][e];
    }
}

// Packed rows of more than 18432 positions: two passes over the row, gathered through perm from memory.
__global__ __launch_bounds__(256) void weight_rows_long_kernel(RowsArgs a)
{
    __shared__ float red[2][4];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, row = blockIdx.x;
    const int K_o = a.sc->K_o;
    const float *w = a.W + (size_t)row * a.ldw;
    float m_o = 0.0f, m_n = 0.0f;
    for (int q = t; q < a.K; q += 256) {
        const float m = fabsf(w[a.perm[q]]);
        if (q < K_o) m_o = fmaxf(m_o, m);
        else m_n = fmaxf(m_n, m);
    }
    m_o = wave_max_all(m_o);
    m_n = wave_max_all(m_n);
    if (lane == 0) {
        red[0][wave] = m_o;
        red[1][wave] = m_n;
    }
    __syncthreads();
    const float so = fmaxf(fmaxf(red[0][0], red[0][1]), fmaxf(red[0][2], red[0][3])) / a.qmax;
    const float sn = fmaxf(fmaxf(red[1][0], red[1][1]), fmaxf(red[1][2], red[1][3])) / a.qmax;
    if (t == 0) {
        a.s_outlier[row] = so;
        a.s_normal[row] = sn;
    }
    store_codes_far<256>(a, row, t, K_o, so, sn);
}

// ---- percentile-clip scales ----------------------------------------------------------------
// Percentile-clip initialisation of the two scales of every output row (Sec. 4.1 "Quantization
// Implementation": the clipping percentile is searched over {0.999, 0.9999, 0.99999}).  Per row and block,
// with the block's n values taken in packed order:
//     clip_p = linear-interpolated p-quantile of |w|  (h = (n-1) p, a[floor h] + frac (a[floor h + 1] - a[floor h]),
//              in double, rounded to float),  s_p = clip_p / qmax,
//     SSE_p  = sum (double) e^2,  e = fmaf(-s_p, q(w, s_p), w),  summed in packed order in double;
//     the smallest SSE wins, the larger percentile on a tie.
// One workgroup per row, values in registers in packed order (PackedRow), both blocks in each phase.  The quantiles need
// the T = n - floor(0.999 (n-1)) largest magnitudes only (T <= 18 for n <= 16384).  The T-th largest of the NT / 16 maxima
// of groups of sixteen lanes is a lower bound of the T-th largest value; the few dozen values that reach it go to
// LDS and are ranked there.
// The three sums are taken in parallel.  They decide an integer, so a comparison counts only where it holds for every order of
// summation: serial and parallel sums are both within n u / (1 - n u) of the exact one (u = 2^-53; e^2 is exact).
// Candidates with equal scales have equal sums term by term.  Anything else (intervals that overlap, scales outside the exact
// quotient's range, NaN) is summed in order: the errors taken by the whole workgroup, then one thread per candidate (1536 x 8960 with
// every row so: 0.35 ms a call; with the gather and the quotients in that thread too 8.2).  Bound by the latency of its phases
// (14 us a row) and by vector-ALU issue (about 35 instructions per value), so one row per workgroup and registers held low enough
// for three workgroups per CU, at the price of a few spilled ones (28 bytes of scratch a lane at <5, 512>) (1536 x 8960: 50 us;
// with the offsets kept for three rows 79, one workgroup per CU).
constexpr int CLIP_MAX_T = 20, CLIP_CAND = 512;

template <int CH, int NT>
__global__ __launch_bounds__(NT, CH > 5 ? 4 : 6) void weight_rows_clip_kernel(RowsArgs a)
{
    constexpr int NWAVE = NT / 64, G = NT / 16;
    static_assert(G <= 64, "one group maximum per lane");
    __shared__ float gmax[2][G], top[2][CLIP_MAX_T], redf[NWAVE], scale[2][3], chosen[2];
    __shared__ __align__(16) float cand[2][CLIP_CAND];
    __shared__ double sums[2][NWAVE][3];
    __shared__ float err[3][NT];
    __shared__ int n_cand[2], redi[NWAVE], open[2];
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int K_o = a.sc->K_o;
    PackedRow<CH, NT> pr;
    pr.init(a.perm, a.K, K_o, wave, lane);
    auto block_n = [&](int blk) { return blk ? a.K - K_o : K_o; };
    auto block_T = [&](int blk) { return block_n(blk) - (int)floor((double)(block_n(blk) - 1) * 0.999); };
    {
        const int row = blockIdx.x;
        const float *w = a.W + (size_t)row * a.ldw;
        float x[CH][4];
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) x[c][e] = 0.0f;
        pr.load(w, a.K, x);
        // f(value, real) over the chunks that hold positions of block blk (whole waves)
        auto for_each = [&](int blk, auto f) {
            const int b0 = blk ? pr.n_off : 0, b1 = blk ? pr.end_n : pr.end_o;
#pragma unroll
            for (int c = 0; c < CH; ++c)
                if (pr.base[c] < b1 && pr.base[c] + 256 > b0) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int p = pr.base[c] + 64 * e + lane;
                        f(x[c][e], p >= b0 && p < b1);
                    }
                }
        };
        // ---- the T largest magnitudes of each block, descending, in top[] ----
#pragma unroll 1
        for (int blk = 0; blk < 2; ++blk) {
            float m = -1.0f;
            for_each(blk, [&](float f, bool real) { m = fmaxf(m, real ? fabsf(f) : -1.0f); });
#pragma unroll
            for (int off = 8; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
            if ((lane & 15) == 0) gmax[blk][t >> 4] = m;
            if (t == 0) n_cand[blk] = 0;
            if (t < CLIP_MAX_T) top[blk][t] = -1.0f;
        }
        __syncthreads();
#pragma unroll 1
        for (int blk = 0; blk < 2; ++blk) {
            const int T = block_T(blk);
            float L = -1.0f;                   // at least T values reach the T-th largest group maximum
            const float mine = lane < G ? gmax[blk][lane] : -2.0f;
            int r = 0;
#pragma unroll
            for (int j = 0; j < G; ++j) {
                const float o = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mine), j));
                r += (o > mine || (o == mine && j < lane)) ? 1 : 0;
            }
            const unsigned long long who = __ballot(lane < G && r == T - 1);
            if (who) L = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mine), __builtin_ctzll(who)));
            for_each(blk, [&](float f, bool real) {
                if (real && fabsf(f) >= L) {
                    const int slot = atomicAdd(&n_cand[blk], 1);
                    if (slot < CLIP_CAND) cand[blk][slot] = fabsf(f);
                }
            });
        }
        __syncthreads();
        {
            const int blk = t < NT / 2 ? 1 : 0;        // half of the workgroup ranks each block's candidates
            const int nc = n_cand[blk], T = block_T(blk);
            if (nc <= CLIP_CAND)
                for (int i = t & (NT / 2 - 1); i < nc; i += NT / 2) {
                    const float mine = cand[blk][i];
                    int r = 0;
#pragma unroll 4
                    for (int j = 0; j < nc; j += 4) {
                        const float4 o = *reinterpret_cast<const float4 *>(&cand[blk][j]);
                        r += (o.x > mine || (o.x == mine && j < i)) ? 1 : 0;
                        r += j + 1 < nc && (o.y > mine || (o.y == mine && j + 1 < i)) ? 1 : 0;
                        r += j + 2 < nc && (o.z > mine || (o.z == mine && j + 2 < i)) ? 1 : 0;
                        r += j + 3 < nc && (o.w > mine || (o.w == mine && j + 3 < i)) ? 1 : 0;
                    }
                    if (r < T) top[blk][r] = mine;
                }
        }
#pragma unroll 1
        for (int blk = 0; blk < 2; ++blk) {
            if (n_cand[blk] <= CLIP_CAND) continue;
            // many ties or a crowded group: one distinct magnitude per round
            const int T = block_T(blk);
            float prev = __builtin_inff();
            bool first = true;
            for (int have = 0; have < T;) {
                float mx = -1.0f;
                for_each(blk, [&](float f, bool real) {
                    const float v = fabsf(f);
                    if (real && (first || v < prev)) mx = fmaxf(mx, v);
                });
                mx = wave_max_all(mx);
                if (lane == 0) redf[wave] = mx;
                __syncthreads();
#pragma unroll
                for (int i = 0; i < NWAVE; ++i) mx = fmaxf(mx, redf[i]);
                int eq = 0;
                for_each(blk, [&](float f, bool real) { eq += (real && fabsf(f) == mx) ? 1 : 0; });
                eq = wave_sum_all(eq);
                if (lane == 0) redi[wave] = eq;
                __syncthreads();
                eq = 0;
#pragma unroll
                for (int i = 0; i < NWAVE; ++i) eq += redi[i];
                if (eq == 0) mx = -1.0f;       // nothing left to find (NaN in the row): no further rounds
                const int upto = eq == 0 ? T : min(T, have + eq);
                if (t >= have && t < upto) top[blk][t] = mx;
                have = upto;
                prev = mx;
                first = false;
                __syncthreads();
            }
        }
        __syncthreads();
        // ---- candidate scales: thread 3 blk + c ----
        if (t < 6) {
            const int blk = t / 3, c = t - 3 * blk, n = block_n(blk);
            const double h = (double)(n - 1) * (c == 0 ? 0.999 : c == 1 ? 0.9999 : 0.99999);
            const int lo = (int)floor(h);
            const int hi = lo + 1 < n ? lo + 1 : n - 1;
            const double frac = h - (double)lo;
            const double alo = n > 0 ? (double)top[blk][n - 1 - lo] : 0.0, ahi = n > 0 ? (double)top[blk][n - 1 - hi] : 0.0;
            const float clip = (float)(alo + frac * (ahi - alo));
            scale[blk][c] = clip / a.qmax;
        }
        __syncthreads();
        // ---- squared errors ----
#pragma unroll 1
        for (int blk = 0; blk < 2; ++blk) {
            const ExactQuotient qt[3] = {ExactQuotient(scale[blk][0], a.qmax), ExactQuotient(scale[blk][1], a.qmax), ExactQuotient(scale[blk][2], a.qmax)};
            double sse[3] = {0.0, 0.0, 0.0};
            for_each(blk, [&](float f0, bool real) {
                const float f = real ? f0 : 0.0f;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const float q = rintf(qt[c].clamped(f));
                    const double e = (double)fmaf(-qt[c].s, q, f);
                    sse[c] = fma(e, e, sse[c]);
                }
            });
            // scales outside the exact quotient's range: the sums prove nothing
            if (!(qt[0].exact() && qt[1].exact() && qt[2].exact())) sse[0] = sse[1] = sse[2] = __builtin_nan("");
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                sse[c] = wave_sum_all(sse[c]);
                if (lane == 0) sums[blk][wave][c] = sse[c];
            }
        }
        __syncthreads();
        if (t < 2) {                           // thread blk decides
            const int blk = t, n = block_n(blk);
            const float s0 = scale[blk][0], s1 = scale[blk][1], s2 = scale[blk][2];
            double q0 = 0.0, q1 = 0.0, q2 = 0.0;
#pragma unroll
            for (int i = 0; i < NWAVE; ++i) {
                q0 += sums[blk][i][0];
                q1 += sums[blk][i][1];
                q2 += sums[blk][i][2];
            }
            const double e = 2.5 * ((double)n + 2.0) * 0x1p-53;
            bool proven = true;
            auto less = [&](float sp, double p, float sq, double q) {        // ordered sum p < ordered sum q
                if (sp == sq) return false;
                if (p * (1.0 + e) < q * (1.0 - e)) return true;
                if (!(p * (1.0 - e) >= q * (1.0 + e))) proven = false;
                return false;
            };
            const bool one = less(s1, q1, s2, q2);
            float best = one ? s1 : s2;
            if (less(s0, q0, best, one ? q1 : q2)) best = s0;
            open[blk] = proven ? 0 : 1;
            if (n == 0) best = 0.0f;
            chosen[blk] = best;
        }
        __syncthreads();
#pragma unroll 1
        for (int blk = __builtin_expect(open[0] + open[1], 0) ? 0 : 2; blk < 2; ++blk) {
            if (!open[blk]) continue;
            // in order: all threads take errors, NT values at a time, and thread c sums those of candidate c
            const int n = block_n(blk);
            double T = 0.0;
            for (int p0 = 0; p0 < n; p0 += NT) {
                if (p0 + t < n) {
                    const float f = w[a.perm[(blk ? K_o : 0) + p0 + t]];
#pragma unroll
                    for (int c = 0; c < 3; ++c) err[c][t] = fmaf(-scale[blk][c], (float)quantize_sym(f, scale[blk][c], a.qmax), f);
                }
                __syncthreads();
                if (t < 3) {
                    const int lim = min(NT, n - p0);
#pragma unroll 8
                    for (int i = 0; i < lim; ++i) {
                        const double d = (double)err[t][i];
                        T = fma(d, d, T);
                    }
                }
                __syncthreads();
            }
            if (t < 3) sums[blk][0][t] = T;
            __syncthreads();
            if (t == 0) {
                const double q0 = sums[blk][0][0], q1 = sums[blk][0][1], q2 = sums[blk][0][2];
                float best = q1 < q2 ? scale[blk][1] : scale[blk][2];
                if (q0 < (q1 < q2 ? q1 : q2)) best = scale[blk][0];
                chosen[blk] = best;
            }
            __syncthreads();
        }
        if (t < 2) (t ? a.s_normal : a.s_outlier)[row] = chosen[t];
        const ExactQuotient qo(chosen[0], a.qmax), qn(chosen[1], a.qmax);
        if (qo.exact() && qn.exact()) store_codes<CH, NT>(a, pr, x, row, lane, qo, qn);
        else store_codes_far<NT>(a, row, t, K_o, chosen[0], chosen[1]);
    }
}

// ---- host ------------------------------------------------------------------------------------
struct Workspace {
    DetectScalars *sc;
    float *v;
    double *partial;
    uint8_t *forced;
};

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

int norm_chunks(int32_t N, int32_t K)
{
    const int slabs = (K + 255) / 256;
    const int most = NORM_BLOCKS / slabs > 0 ? NORM_BLOCKS / slabs : 1;
    const int want = (N + 15) / 16;              // at least four rows per wave
    return want < most ? want : most;
}

// The partial sums get what they need at most, whatever N and K: a workspace that is large enough for a layer is large enough for
// every layer of no more channels, as callers that allocate one for several layers expect.
size_t carve(void *base, int32_t K, Workspace *ws)
{
    unsigned char *p = reinterpret_cast<unsigned char *>(base);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        void *r = p ? p + off : nullptr;
        off += align256(bytes);
        return r;
    };
    void *sc = take(sizeof(DetectScalars)), *v = take((size_t)K * 4), *forced = take((size_t)K);
    void *partial = take((size_t)NORM_BLOCKS * 256 * 8);
    if (ws) {
        ws->sc = reinterpret_cast<DetectScalars *>(sc);
        ws->v = reinterpret_cast<float *>(v);
        ws->forced = reinterpret_cast<uint8_t *>(forced);
        ws->partial = reinterpret_cast<double *>(partial);
    }
    return off;
}

template <int R, int NT>
qarvd_status launch_sorting_detect(const Workspace &ws, int32_t K, double f, const qarvd_detect_cfg &c, const uint8_t *forced, int32_t *perm, hipStream_t st)
{
    static unsigned long long raised = 0;      // one mask per kernel
    if (qarvd_status s_a = qarvd_raise_lds_limit_once(detect_kernel<R, NT>, 132 * 1024, raised); s_a != QARVD_OK) return s_a;
    // the sorted norms (or the coarse counters) and the fine bins: 36 KB and 72 KB at K = 9216, 64 KB and 64 KB at 16384
    const size_t lds = ((size_t)(K > COARSE * COPIES ? K : COARSE * COPIES) + (size_t)K * fine_per_norm(R) + 1) * 4;
    hipLaunchKernelGGL((detect_kernel<R, NT>), dim3(1), dim3(NT), lds, st, ws.v, K, f, c.alpha, c.align, forced, ws.sc, perm);
    return qarvd_launch_status();
}

qarvd_status launch_detect(const Workspace &ws, int32_t K, const qarvd_detect_cfg &c, int32_t *perm, hipStream_t st)
{
    const uint8_t *forced = c.forced_mask ? ws.forced : nullptr;
    const double f = c.tau / 0.6745;
    if (K > 16384) {
        hipLaunchKernelGGL((detect_long_kernel<1024>), dim3(1), dim3(1024), 0, st, ws.v, K, f, c.alpha, c.align, forced, ws.sc, perm);
        return qarvd_launch_status();
    }
    if (K <= 6 * 256) return launch_sorting_detect<6, 256>(ws, K, f, c, forced, perm, st);
    if (K <= 10 * 512) return launch_sorting_detect<10, 512>(ws, K, f, c, forced, perm, st);
    if (K <= 9 * 1024) return launch_sorting_detect<9, 1024>(ws, K, f, c, forced, perm, st);
    return launch_sorting_detect<16, 1024>(ws, K, f, c, forced, perm, st);
}

template <int CH, int NT>
void launch_rows(const RowsArgs &a, int cus, hipStream_t st)
{
    constexpr int RW = NT == 64 ? 4 : 1, TH = NT == 64 ? 256 : NT;
    // as many workgroups as the registers let run at once (sixteen waves per CU), so that the offsets are set up once
    // for several rows, trimmed to whole rounds
    const int slots = cus * 1024 / TH;
    const int groups = (a.N + RW - 1) / RW;
    const int rounds = (groups + slots - 1) / slots;
    hipLaunchKernelGGL((weight_rows_kernel<CH, NT>), dim3((groups + rounds - 1) / rounds), dim3(TH), 0, st, a);
}

template <int CH, int NT>
void launch_rows_clip(const RowsArgs &a, hipStream_t st)
{
    hipLaunchKernelGGL((weight_rows_clip_kernel<CH, NT>), dim3(a.N), dim3(NT), 0, st, a);
}

}  // namespace

extern "C" void qarvd_default_detect_cfg(qarvd_detect_cfg *cfg)
{
    if (!cfg) return;
    cfg->tau = 3.5;
    cfg->alpha = 1.2;
    cfg->align = 32;
    cfg->clip_search = 0;
    cfg->forced_mask = nullptr;
}

extern "C" const char *qarvd_status_string(qarvd_status s)
{
    switch (s) {
        case QARVD_OK: return "QARVD_OK";
        case QARVD_ERR_INVALID_ARG: return "QARVD_ERR_INVALID_ARG";
        case QARVD_ERR_UNSUPPORTED: return "QARVD_ERR_UNSUPPORTED";
        case QARVD_ERR_WORKSPACE: return "QARVD_ERR_WORKSPACE";
        case QARVD_ERR_HIP: return "QARVD_ERR_HIP";
    }
    return "QARVD_ERR_UNKNOWN";
}

extern "C" int32_t qarvd_packed_normal_offset(int32_t K_o) { return K_o < 0 ? 0 : qarvd_round_up(K_o, 32); }

extern "C" int32_t qarvd_packed_k(int32_t K, int32_t K_o)
{
    if (K <= 0 || K > QARVD_MAX_K || K_o > K) return 0;
    if (K_o >= 0) return qarvd_packed(K, K_o).kp;
    // worst case over K_o: the outlier padding adds at most 31 bytes
    return qarvd_round_up(K + 31, 128);
}

extern "C" int32_t qarvd_packed_ld(int32_t K, int32_t K_o)
{
    const int32_t kp = qarvd_packed_k(K, K_o);
    if (kp <= 0) return 0;
    const int32_t ld = kp + 128;                  // multiples of 128, skipping the multiples of 512
    return (ld % 512) == 0 ? ld + 128 : ld;
}

extern "C" size_t qarvd_quantize_weight_workspace(int32_t N, int32_t K)
{
    if (N <= 0 || K <= 0 || K > QARVD_MAX_K) return 0;
    return carve(nullptr, K, nullptr);
}

namespace {

// bits = 8: Wq is the INT8 output [N, ldwq].  bits = 4: Wq is the packed INT4 output [N, ldwq bytes].
qarvd_status quantize_weight_impl(int bits, const float *W, int32_t N, int32_t K, int64_t ldw,
                                  const qarvd_detect_cfg *cfg, void *Wq, int64_t ldwq, float *s_normal,
                                  float *s_outlier, int32_t *perm, int32_t *K_o_host, float *v_out,
                                  void *workspace, size_t workspace_bytes, void *stream)
{
    if (!W || !Wq || !s_normal || !s_outlier || !perm || !K_o_host) return QARVD_ERR_INVALID_ARG;
    if (N <= 0 || K <= 0 || K > QARVD_MAX_K || ldw < K) return QARVD_ERR_INVALID_ARG;
    qarvd_detect_cfg c;
    qarvd_default_detect_cfg(&c);
    if (cfg) c = *cfg;
    if (!c.forced_mask && (!(c.tau >= 0.0) || !(c.alpha >= 0.0) || c.align <= 0)) return QARVD_ERR_INVALID_ARG;
    if (c.clip_search != 0 && c.clip_search != 1) return QARVD_ERR_INVALID_ARG;
    if (c.clip_search && K > 16384) return QARVD_ERR_UNSUPPORTED;     // the search keeps the 20 largest magnitudes
    // The split is not known yet, so the row stride must hold the widest packed row the call can
    // produce: K rounded up to 128 when the aligned count is a multiple of 32 (no inner padding),
    // else the general worst case.
    const bool no_inner_pad = !c.forced_mask && (c.align % 32) == 0;
    const int64_t kp_max = no_inner_pad ? qarvd_round_up(K, 128) : qarvd_packed_k(K, -1);
    if (ldwq < (bits == 8 ? kp_max : kp_max / 2)) return QARVD_ERR_INVALID_ARG;
    if (!qarvd_aligned16(Wq) || (ldwq % 16) != 0 || (reinterpret_cast<uintptr_t>(W) & 3u)) return QARVD_ERR_UNSUPPORTED;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u)) return QARVD_ERR_WORKSPACE;
    if (workspace_bytes < carve(nullptr, K, nullptr)) return QARVD_ERR_WORKSPACE;

    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    Workspace ws;
    carve(workspace, K, &ws);
    int cus = 0;
    if (qarvd_status s_d = qarvd_current_device(nullptr, &cus); s_d != QARVD_OK) return s_d;
    if (c.forced_mask) QARVD_HIP_TRY(hipMemcpyAsync(ws.forced, c.forced_mask, (size_t)K, hipMemcpyHostToDevice, st));

    const int chunks = norm_chunks(N, K), per_chunk = (N + chunks - 1) / chunks;
    const bool vec = (K % 4) == 0 && (ldw % 4) == 0 && qarvd_aligned16(W);
    const dim3 ng((K + 255) / 256, chunks);
    if (vec) hipLaunchKernelGGL((norm_partial_kernel<true>), ng, dim3(256), 0, st, W, N, K, ldw, per_chunk, ws.partial);
    else hipLaunchKernelGGL((norm_partial_kernel<false>), ng, dim3(256), 0, st, W, N, K, ldw, per_chunk, ws.partial);
    hipLaunchKernelGGL(norm_final_kernel, dim3((K + 63) / 64), dim3(1024), 0, st, ws.partial, chunks, W, N, K, ldw, ws.v, v_out);
    if (qarvd_status s_l = launch_detect(ws, K, c, perm, st); s_l != QARVD_OK) return s_l;

    RowsArgs a;
    a.W = W; a.ldw = ldw; a.perm = perm; a.sc = ws.sc;
    a.out = reinterpret_cast<uint8_t *>(Wq); a.ldo = ldwq;
    a.s_normal = s_normal; a.s_outlier = s_outlier;
    a.qmax = bits == 8 ? 127.0f : 7.0f; a.N = N; a.K = K;
    // threads per row and dwords per thread by the longest packed row the call can produce
    if (c.clip_search) {
        if (kp_max <= 2 * 1024) launch_rows_clip<2, 256>(a, st);
        else if (kp_max <= 5 * 1024) launch_rows_clip<5, 256>(a, st);
        else if (kp_max <= 5 * 2048) launch_rows_clip<5, 512>(a, st);
        else launch_rows_clip<9, 512>(a, st);
    } else {
        if (kp_max <= 6 * 256) launch_rows<6, 64>(a, cus, st);
        else if (kp_max <= 5 * 512) launch_rows<5, 128>(a, cus, st);
        else if (kp_max <= 5 * 1024) launch_rows<5, 256>(a, cus, st);
        else if (kp_max <= 9 * 1024) launch_rows<9, 256>(a, cus, st);
        else if (kp_max <= 9 * 2048) launch_rows<9, 512>(a, cus, st);
        else hipLaunchKernelGGL(weight_rows_long_kernel, dim3(N), dim3(256), 0, st, a);
    }
    if (qarvd_status s_l = qarvd_launch_status(); s_l != QARVD_OK) return s_l;
    DetectScalars host_sc;
    QARVD_HIP_TRY(hipMemcpyAsync(&host_sc, ws.sc, sizeof(host_sc), hipMemcpyDeviceToHost, st));
    QARVD_HIP_TRY(hipStreamSynchronize(st));
    *K_o_host = host_sc.K_o;
    return QARVD_OK;
}

}  // namespace

extern "C" qarvd_status qarvd_quantize_weight(const float *W, int32_t N, int32_t K, int64_t ldw,
                                              const qarvd_detect_cfg *cfg, int8_t *Wq, int64_t ldwq,
                                              float *s_normal, float *s_outlier, int32_t *perm,
                                              int32_t *K_o_host, float *v_out, void *workspace,
                                              size_t workspace_bytes, void *stream)
{
    return quantize_weight_impl(8, W, N, K, ldw, cfg, Wq, ldwq, s_normal, s_outlier, perm, K_o_host, v_out, workspace,
                                workspace_bytes, stream);
}

// ---- the same offline step for callers that cannot allocate ----------------------------------------------
// The workspace (partial norm sums, norms, mask, the scalars) lives in a file-scope device array instead of a caller
// buffer: 2.2 MB per GPU the library runs on, held until the process ends.  In host code the array's name is only a stand-in;
// its device address is looked up once per device with hipGetSymbolAddress and that pointer is what the kernels get.
namespace {
constexpr int32_t STATIC_SCRATCH_MAX_K = 16384;
// carve() for K <= 16384: 256 (scalars) + 65536 (norms) + 16384 (mask) + partial sums (at most NORM_BLOCKS slabs of 256 columns)
constexpr size_t STATIC_SCRATCH_BYTES = 256 + 65536 + 16384 + (size_t)NORM_BLOCKS * 256 * 8;      // 2179328
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

// device address of `scratch` on the current device (each GPU holds its own copy at its own address)
qarvd_status static_scratch_ptr(void **out)
{
    static void *ptr[64] = {nullptr};
    int dev = 0;
    QARVD_HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) return QARVD_ERR_UNSUPPORTED;
    void *p = __atomic_load_n(&ptr[dev], __ATOMIC_ACQUIRE);
    if (!p) {
        QARVD_HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return QARVD_ERR_HIP;
        __atomic_store_n(&ptr[dev], p, __ATOMIC_RELEASE);
    }
    *out = p;
    return QARVD_OK;
}
}  // namespace

extern "C" int32_t qarvd_quantize_weight_static_max_k(void) { return STATIC_SCRATCH_MAX_K; }

extern "C" qarvd_status qarvd_quantize_weight_static(const float *W, int32_t N, int32_t K, int64_t ldw,
                                                     const qarvd_detect_cfg *cfg, int8_t *Wq, int64_t ldwq,
                                                     float *s_normal, float *s_outlier, int32_t *perm,
                                                     int32_t *K_o_host, float *v_out, void *stream)
{
    if (K > STATIC_SCRATCH_MAX_K) return QARVD_ERR_WORKSPACE;      // the fixed array holds the workspace of K <= 16384
    if (K > 0 && carve(nullptr, K, nullptr) > STATIC_SCRATCH_BYTES) return QARVD_ERR_WORKSPACE;
    void *ws = nullptr;
    if (qarvd_status st = static_scratch_ptr(&ws); st != QARVD_OK) return st;
    // Every kernel of the step writes the part of the workspace it owns before anything reads it (the existing
    // entry point is given uninitialised memory too), so what an earlier call left behind is never read.
    return quantize_weight_impl(8, W, N, K, ldw, cfg, Wq, ldwq, s_normal, s_outlier, perm, K_o_host, v_out, ws,
                                STATIC_SCRATCH_BYTES, stream);
}

extern "C" size_t qarvd_quantize_weight_w4_workspace(int32_t N, int32_t K)
{
    if (N <= 0 || K <= 0 || K > QARVD_MAX_K) return 0;
    return carve(nullptr, K, nullptr);
}

extern "C" qarvd_status qarvd_quantize_weight_w4(const float *W, int32_t N, int32_t K, int64_t ldw,
                                                 const qarvd_detect_cfg *cfg, uint8_t *Wq4, int64_t ldwq4,
                                                 float *s_normal, float *s_outlier, int32_t *perm,
                                                 int32_t *K_o_host, float *v_out, void *workspace,
                                                 size_t workspace_bytes, void *stream)
{
    return quantize_weight_impl(4, W, N, K, ldw, cfg, Wq4, ldwq4, s_normal, s_outlier, perm, K_o_host, v_out, workspace,
                                workspace_bytes, stream);
}
