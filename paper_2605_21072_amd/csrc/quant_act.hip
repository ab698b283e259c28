// Activation quantization for gfx950: fused gather-permute + per-token dynamic (or static)
// symmetric INT8 (appendix "Quantization Kernels", kernel (i) and the online permutation;
// Sec. 2.2 Eq. (quantization)).
//
// HBM-bound: every X element is read from memory exactly once and one byte is written.
//
// A token row is owned by one wave (K <= 1536) or one workgroup.  It is read with coalesced 16-byte loads in
// natural channel order and stays in registers; the per-token absmax is a reduction inside the wave (plus an LDS exchange
// between waves); the codes go to LDS in natural order, four to a dword, and every thread picks the four bytes of
// its dwords of the packed row from there, with the entries of `perm` as byte addresses: no inverse table to build, no
// byte stores, nothing to clear, and at most one barrier between a row's arrival and its way out.
#include "qarvd_common.h"

namespace {

constexpr int TPB = 256;

// Four consecutive elements of X as loaded, at any element's address (one instruction whatever the alignment), and widened
// (exactly) to fp32.
template <typename T> struct Elem;
template <> struct Elem<float> {
    typedef float4 raw;
    typedef float raw_any __attribute__((ext_vector_type(4), aligned(4)));
    static __device__ __forceinline__ raw zero() { return make_float4(0.0f, 0.0f, 0.0f, 0.0f); }
    static __device__ __forceinline__ raw of(raw_any r) { return make_float4(r.x, r.y, r.z, r.w); }
    static __device__ __forceinline__ raw scale(raw r, float f) { return make_float4(r.x * f, r.y * f, r.z * f, r.w * f); }
    static __device__ __forceinline__ float4 widen(raw r) { return r; }
    static __device__ __forceinline__ float load1(const float *p) { return *p; }
    static __device__ __forceinline__ raw drop(raw r, int n)        // the first n elements, 0 < n < 4, moved out, zeros behind
    {
        return n == 1 ? make_float4(r.y, r.z, r.w, 0.0f) : n == 2 ? make_float4(r.z, r.w, 0.0f, 0.0f) : make_float4(r.w, 0.0f, 0.0f, 0.0f);
    }
};
template <> struct Elem<uint16_t> {   // bf16 bit patterns
    typedef uint2 raw;
    typedef uint32_t raw_any __attribute__((ext_vector_type(2), aligned(2)));
    static __device__ __forceinline__ raw zero() { return make_uint2(0u, 0u); }
    static __device__ __forceinline__ raw of(raw_any r) { return make_uint2(r.x, r.y); }
    static __device__ __forceinline__ float4 widen(raw u)
    {
        return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xFFFF0000u), __uint_as_float(u.y << 16),
                           __uint_as_float(u.y & 0xFFFF0000u));
    }
    static __device__ __forceinline__ raw scale(raw u, float f)      // f a power of two: eight significant bits stay eight
    {
        const float4 w = widen(u);
        return make_uint2((__float_as_uint(w.x * f) >> 16) | (__float_as_uint(w.y * f) & 0xFFFF0000u),
                          (__float_as_uint(w.z * f) >> 16) | (__float_as_uint(w.w * f) & 0xFFFF0000u));
    }
    static __device__ __forceinline__ float load1(const uint16_t *p) { return bf16_bits_to_f32(*p); }
    static __device__ __forceinline__ raw drop(raw r, int n)
    {
        const uint64_t w = (((uint64_t)r.y << 32) | r.x) >> (16 * n);
        return make_uint2((uint32_t)w, (uint32_t)(w >> 32));
    }
};

struct ActArgs {
    const void *X;
    int64_t ldx;
    const int32_t *perm;
    int8_t *Xq;
    int64_t ldxq;
    float *s_x;
    float static_scale;
    int32_t M, K, K_o, n_off, kp;
    int32_t is_static;     // 1: static_scale for every row, no absmax
    int32_t store_wt;      // 1: Xq leaves through write-through stores (see store_q)
    int32_t stream;        // 1: X is loaded with the non-temporal hint where that form is built
};

// Loads of X with the non-temporal hint: X does not displace what the last-level cache (256 MB) holds, and memory delivers more (a plain
// loop over 168 MB in, 42 MB out: 6.3 TB/s instead of 5.4).  But a second linear on the same X then finds none of it in the cache.  So the line
// lies where it would not find it anyway: X and its codes, and where a GEMM follows in the same call its weights and output, are more than
// the cache holds.  us behind the kernel that wrote X, plain -> non-temporal, for one, two and three linears on it:
//   total below the line, plain:     fp32 168 MB, 8960 -> 1536 (239 in all) 150 -> 144 | 232 -> 238 | 320 -> 332
//                                    fp32 168 MB, 5120 -> 1536 (243)        161 -> 152 | 237 -> 245 | 323 -> 338
//   above it, non-temporal:          fp32 192 MB, 8960 -> 1536 (270)        221 -> 208 | 335 -> 332 | 455 -> 455
//                                    fp32 168 MB, 5120 -> 5120 (319)        286 -> 273 | 502 -> 474 | 718 -> 681
//                                    fp32 192 MB, 1536 -> 1536 (338)        192 -> 175 | 313 -> 286 | 434 -> 397
//                                    bf16 146 MB, 5120 -> 5120 (391)        406 -> 385 | 760 -> 719 | 1109 -> 1046
// and quantized one, two and three times in a row with nothing between:
//   below:  fp32 192 MB (240 with its codes) 42 -> 35 | 76 -> 80 | 117 -> 122      bf16 146 MB (219) 43 -> 48 | 90 -> 98 | 135 -> 145
//   above:  fp32 216 MB (270)                52 -> 39 | 93 -> 90 | 137 -> 138      bf16 192 MB (288) 63 -> 58 | 122 -> 119 | 183 -> 177
// An X of up to 144 MB is level at best (129 MB behind its producer 41.9 and 42.3).
constexpr size_t STREAM_X_BYTES = (size_t)144 << 20, STREAM_CALL_BYTES = (size_t)265 << 20;

// Stores of the quantized rows.  A kernel ends with a write-back of what its XCDs' L2s still hold, and the
// consumer (the GEMM, on any XCD) reads Xq from memory either way; for an Xq of a few MB that write-back is
// 1-2 us at the end of a 9 us kernel.  Write-through stores (sc0 sc1) send the bytes on while the kernel still
// computes.  Used when the whole Xq is at most 40 MB (beyond that the extra traffic during the kernel costs
// more than the tail); `off` is the byte offset from a.Xq (the host checked that it fits 31 bits).
__device__ __forceinline__ void store_q(const ActArgs &a, size_t off, uint32_t w)
{
#if defined(__HIP_DEVICE_COMPILE__)
    if (a.store_wt) {
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(a.Xq, 0, 0x7fffffff, 0x00020000);
        __builtin_amdgcn_raw_buffer_store_b32(w, r, (int)off, 0, 17);
        return;
    }
#endif
    *reinterpret_cast<uint32_t *>(a.Xq + off) = w;
}

// Workgroup-wide max of a non-negative value; `red` holds one float per wave.
__device__ __forceinline__ float block_max(float v, float *red)
{
    v = wave_max_all(v);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) red[wave] = v;
    __syncthreads();
    return fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

// One row with IEEE divisions and channels gathered from memory: rows with infinities, and the rows of the general kernel below.
template <typename T>
__device__ __forceinline__ void quant_row_far(const ActArgs &a, const T *x, int8_t *out, float s, int t, int nt)
{
    for (int pp = t; pp < a.kp; pp += nt) {
        int p = -1;                                    // logical packed index, -1 = padding
        if (pp < a.K_o) p = pp;
        else if (pp >= a.n_off && pp - a.n_off < a.K - a.K_o) p = a.K_o + (pp - a.n_off);
        int8_t q = 0;
        if (p >= 0) {
            const int k = a.perm ? a.perm[p] : p;
            if ((unsigned)k < (unsigned)a.K) q = (int8_t)quantize_i8(Elem<T>::load1(x + k), s);
        }
        out[pp] = q;
    }
}

// How the packed row is put together.
enum Order {
    NATURAL,       // no permutation: the codes go straight from registers to memory and no LDS image exists
    WHOLE_WORDS,   // four entries of perm at a time are four neighbours of the packed row: no pads before the end, perm 16-byte aligned
    ANY_ORDER,     // pads anywhere (an outlier block that is no multiple of 32), perm at any address
};

// Register-resident rows.  NT threads own a token row at a time, CH chunks of 4 channels per thread (K <= 4 CH NT); NT = 64: four
// independent rows per workgroup, no barrier.  X may have any width from 4 on, any stride and any alignment: a chunk is one load at
// its element's address.  TAIL: K is no multiple of 4; a row's last chunk is loaded from its last four channels and moved down
// when it is used, so that the loads stay free of branches that would wait for them.
//
// Bound by memory at large M (4680 x 8960 fp32, 210 MB from and to memory: 48 -> 42 us, the rate of a device copy; bf16
// 57 -> 30), by latency at small M (256 x 1536: 5.6 -> 3.6 us; 4680 x 1536 bf16 11.0 -> 7.5): perm and the first row are
// requested together and perm is used as it arrives, and the next row of a wave is requested before the current one is worked
// on (NATURAL: once its maximum is known; with eight waves on a SIMD the other rows cover the wait, and that order needs
// fewer registers: 4680 x 5120 bf16 24.4 -> 18.2 us).  (Before: codes scattered byte by byte through a channel -> position table built in LDS by every workgroup, a
// branch to an IEEE division beside every quotient.  Fetching the four bytes with one v_perm_b32 under a selector
// per dword instead of four byte reads costs more setting up than it saves: 15.5 us for the last case.)
// Waves on a SIMD that the registers have to leave room for: as many as run without spilling more than a few.
template <typename T, int CH, int NT, Order ORD> constexpr int waves_per_simd()
{
    return ORD != NATURAL || CH * NT > 4096 ? (CH > 6 ? 3 : 4) : sizeof(T) == 2 || CH <= 3 ? 8 : 6;
}
template <typename T, int CH, int NT, Order ORD, bool TAIL, bool STREAM>
__global__ __launch_bounds__(NT == 64 ? 256 : NT, (waves_per_simd<T, CH, NT, ORD>())) void quant_act_kernel(ActArgs a)
{
    typedef typename Elem<T>::raw raw;
    constexpr bool PERM = ORD != NATURAL;
    constexpr int RW = NT == 64 ? 4 : 1, NWAVE = NT / 64;
    constexpr int CP = ORD == ANY_ORDER ? CH + 1 : CH;       // chunks of the packed row: up to 31 + 127 pads
    constexpr int ZERO = 4 * CH * NT;                        // (ANY_ORDER) image address of a zero, for the pads
    constexpr float MAGIC = 12582912.0f;       // 1.5 * 2^23: the sum rounds half-to-even, the code is its low byte
    __shared__ __align__(16) uint32_t image[PERM ? (NT == 64 ? 4 : 2) : 1][PERM ? CH * NT + (ORD == ANY_ORDER ? 4 : 0) : 1];      // natural order
    __shared__ float red[2][NWAVE];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t = NT == 64 ? (int)(threadIdx.x & 63) : (int)threadIdx.x;
    const int K = a.K, kp = a.kp;
    const int stride = (int)gridDim.x * RW;
    int m = blockIdx.x * RW + (NT == 64 ? wave : 0);

    const T *X = reinterpret_cast<const T *>(a.X);
    auto load_row = [&](int row, raw (&v)[CH]) {
        const T *x = X + (size_t)row * a.ldx;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int k = 4 * (t + c * NT);
            if (k < K) {
                const typename Elem<T>::raw_any *p = reinterpret_cast<const typename Elem<T>::raw_any *>(
                    reinterpret_cast<const char *>(x) + (uint32_t)(TAIL ? min(k, K - 4) : k) * (uint32_t)sizeof(T));
                if constexpr (STREAM) v[c] = Elem<T>::of(__builtin_nontemporal_load(p));
                else v[c] = Elem<T>::of(*p);
            }
        }
    };

    // Channels of the four packed positions of this thread's dword t + c NT, which are their byte addresses in the image.  (An entry
    // of perm outside [0, K), which makes the bytes undefined, is moved inside.)
    int4 ch[PERM ? CP : 1];
    raw v[CH], vn[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) v[c] = vn[c] = Elem<T>::zero();
    typedef int entries __attribute__((ext_vector_type(4), aligned(4)));
    // (ANY_ORDER) index in perm of a dword's first position; its block (n_off is a multiple of 32) ends at index `end`
    auto first_entry = [&](int p) { return p < a.n_off ? p : a.K_o + (p - a.n_off); };
    if constexpr (PERM) {
#pragma unroll
        for (int c = 0; c < CP; ++c) {
            const int p = 4 * (t + c * NT);
            if constexpr (ORD == WHOLE_WORDS) {
                ch[c] = make_int4(0, 0, 0, 0);
                if (p < K) ch[c] = *reinterpret_cast<const int4 *>(a.perm + p);
            } else {                               // four neighbours of perm, from the last four on where they would pass its end
                const entries e = *reinterpret_cast<const entries *>(a.perm + min(first_entry(p), K - 4));
                ch[c] = make_int4(e.x, e.y, e.z, e.w);
            }
        }
    }
    if (m < a.M) load_row(m, v);
    if constexpr (PERM) {
        auto inside = [&](int k) { return (int)min((unsigned)k, (unsigned)(K - 1)); };
#pragma unroll
        for (int c = 0; c < CP; ++c) {
            if constexpr (ORD == ANY_ORDER) {
                const int p = 4 * (t + c * NT), i = first_entry(p), end = p < a.n_off ? a.K_o : K;
                const int by = i - (K - 4);        // > 0: the entries lie that much later in what was loaded
                int4 e = ch[c];
                if (by > 0) e = by == 1 ? make_int4(e.y, e.z, e.w, 0) : by == 2 ? make_int4(e.z, e.w, 0, 0) : make_int4(e.w, 0, 0, 0);
                ch[c] = make_int4(i < end ? inside(e.x) : ZERO, i + 1 < end ? inside(e.y) : ZERO, i + 2 < end ? inside(e.z) : ZERO,
                                  i + 3 < end ? inside(e.w) : ZERO);
            } else {
                ch[c] = make_int4(inside(ch[c].x), inside(ch[c].y), inside(ch[c].z), inside(ch[c].w));
            }
        }
        // (read behind a barrier, or by the wave itself)
        if (ORD == ANY_ORDER && t < (NT == 64 ? 1 : 2)) image[NT == 64 ? wave : t][CH * NT] = 0u;
    }

    for (int buf = 0; m < a.M; m += stride, buf ^= 1) {
        auto request_next = [&]() {                            // flies under this row's work
            if (m + stride < a.M) load_row(m + stride, vn);
        };
        if constexpr (PERM) request_next();
        if constexpr (TAIL) {
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const int k = 4 * (t + c * NT);
                if (k < K && k > K - 4) v[c] = Elem<T>::drop(v[c], k - (K - 4));
            }
        }
        float s = a.static_scale, amax = 0.0f;
        if (!a.is_static) {
#pragma unroll
            for (int c = 0; c < CH; ++c) {                     // (zeros past the end of the row)
                const float4 f = Elem<T>::widen(v[c]);
                amax = fmaxf(amax, fmaxf(fmaxf(fabsf(f.x), fabsf(f.y)), fmaxf(fabsf(f.z), fabsf(f.w))));
            }
        }
        if constexpr (!PERM) request_next();
        if (!a.is_static) {
            amax = wave_max_all(amax);
            if constexpr (NT > 64) {
                if ((threadIdx.x & 63) == 0) red[buf][wave] = amax;
                __syncthreads();
#pragma unroll
                for (int w = 0; w < NWAVE; ++w) amax = fmaxf(amax, red[buf][w]);
            }
            s = amax / 127.0f;
            if (t == 0) a.s_x[m] = s;
        }
        const size_t out = (size_t)m * a.ldxq;         // byte offset of the row in Xq
        ExactQuotient q(s, 127.0f);
        bool far = false;
        if (!q.exact()) {                              // (uniform over the row)
            // Row and scale times the same power of two: no quotient changes.  Up: exact, or infinite and clipped as before.  Down
            // (s > 1e30): values that lose bits lie below 1e-9 and have the code 0 either way.
            const float f = s < 1.0f ? 0x1p96f : 0x1p-96f;
            far = !(s < __builtin_inff());             // an infinity in the row
#pragma unroll
            for (int c = 0; c < CH; ++c) v[c] = Elem<T>::scale(v[c], f);
            q = ExactQuotient(s * f, 127.0f);
        }
        if (far) {
            quant_row_far<T>(a, X + (size_t)m * a.ldx, a.Xq + out, s, t, NT);
            if constexpr (PERM && NT > 64) __syncthreads();        // as many barriers as the other path
        } else {
            auto codes = [&](const raw &r) {
                const float4 f = Elem<T>::widen(r);
                const float b[4] = {q.clamped(f.x) + MAGIC, q.clamped(f.y) + MAGIC, q.clamped(f.z) + MAGIC, q.clamped(f.w) + MAGIC};
                const uint32_t lo = __builtin_amdgcn_perm(__float_as_uint(b[1]), __float_as_uint(b[0]), 0x0c0c0400u);
                const uint32_t hi = __builtin_amdgcn_perm(__float_as_uint(b[3]), __float_as_uint(b[2]), 0x0c0c0400u);
                return (uint32_t)__builtin_amdgcn_perm(hi, lo, 0x05040100u);
            };
            if constexpr (!PERM) {
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                    const int k = 4 * (t + c * NT);
                    if (k < kp) store_q(a, out + k, k < K ? codes(v[c]) : 0u);     // beyond K: zero padding (v is zero there)
                }
            } else {
                uint32_t *img = image[NT == 64 ? wave : buf];
#pragma unroll
                for (int c = 0; c < CH; ++c) img[t + c * NT] = codes(v[c]);
                if constexpr (NT > 64) __syncthreads();            // (one wave's LDS accesses complete in order)
                const uint8_t *bytes = reinterpret_cast<const uint8_t *>(img);
#pragma unroll
                for (int c = 0; c < CP; ++c) {
                    const int p = 4 * (t + c * NT);
                    if (p >= kp) continue;
                    const uint32_t w = (uint32_t)bytes[ch[c].x] | ((uint32_t)bytes[ch[c].y] << 8) | ((uint32_t)bytes[ch[c].z] << 16) |
                                 ((uint32_t)bytes[ch[c].w] << 24);
                    store_q(a, out + p, ORD == ANY_ORDER || p < K ? w : 0u);       // (whole dwords of padding)
                }
            }
        }
#pragma unroll
        for (int c = 0; c < CH; ++c) v[c] = vn[c];
    }
}

// Rows of more than 20480 channels or packed bytes, or of less than one chunk: one workgroup per row, two passes over it (the
// second is served by the cache), gather through perm from global memory.
template <typename T>
__global__ __launch_bounds__(TPB) void quant_act_generic_kernel(ActArgs a)
{
    __shared__ float red[4];
    const int tid = threadIdx.x;
    const T *X = reinterpret_cast<const T *>(a.X);
    for (int m = blockIdx.x; m < a.M; m += gridDim.x) {
        const T *x = X + (size_t)m * a.ldx;
        float s;
        if (a.is_static) {
            s = a.static_scale;
        } else {
            float amax = 0.0f;
            for (int k = tid; k < a.K; k += TPB) amax = fmaxf(amax, fabsf(Elem<T>::load1(x + k)));
            amax = block_max(amax, red);
            s = amax / 127.0f;
            if (tid == 0) a.s_x[m] = s;
            __syncthreads();   // red is reused by the next row
        }
        quant_row_far<T>(a, x, a.Xq + (size_t)m * a.ldxq, s, tid, TPB);
    }
}

int num_cu()
{
    int cus = 0;
    return (qarvd_current_device(nullptr, &cus) == QARVD_OK && cus > 0) ? cus : 256;
}

// Workgroups of a kernel that one CU holds, asked for once per kernel and device (registers decide it here).
template <auto kern> int blocks_per_cu(int threads)
{
    static int held[64] = {0};                 // one array per kernel; the same value from any thread
    int dev = 0;
    if (qarvd_current_device(&dev, nullptr) != QARVD_OK || dev < 0 || dev >= 64) return 1;
    int n = __atomic_load_n(&held[dev], __ATOMIC_RELAXED);
    if (n == 0) {
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, reinterpret_cast<const void *>(kern), threads, 0) != hipSuccess || n < 1) {
            (void)hipGetLastError();
            n = 1;
        }
        __atomic_store_n(&held[dev], n, __ATOMIC_RELAXED);
    }
    return n;
}

template <typename T, int CH, int NT, Order ORD, bool TAIL, bool STREAM>
qarvd_status launch_rows_as(const ActArgs &a, hipStream_t st)
{
    constexpr int RW = NT == 64 ? 4 : 1, TH = NT == 64 ? 256 : NT;
    // as many workgroups as the chip holds, trimmed so that all of them walk the same number of rows
    // (4680 rows on 1024 slots: 936 workgroups of exactly 5 rows instead of 1024 of 4 or 5)
    const int slots = num_cu() * blocks_per_cu<quant_act_kernel<T, CH, NT, ORD, TAIL, STREAM>>(TH);
    const int groups = (a.M + RW - 1) / RW;
    const int rounds = (groups + slots - 1) / slots;
    hipLaunchKernelGGL((quant_act_kernel<T, CH, NT, ORD, TAIL, STREAM>), dim3((groups + rounds - 1) / rounds), dim3(TH), 0, st, a);
    return qarvd_launch_status();
}

// The streaming form is built where a model's widths lead: whole dwords on either side.  (Chosen at run time inside one kernel it cost
// the other inputs 5 to 12 %.)
template <typename T, int CH, int NT, Order ORD, bool TAIL>
qarvd_status launch_rows(const ActArgs &a, hipStream_t st)
{
    if constexpr (!TAIL && ORD != ANY_ORDER)
        if (a.stream) return launch_rows_as<T, CH, NT, ORD, TAIL, true>(a, st);
    return launch_rows_as<T, CH, NT, ORD, TAIL, false>(a, st);
}

// Threads and chunks for a row of `width` channels (ANY_ORDER) or packed bytes; no launch beyond the last width.  A row that
// fits one wave runs without barriers, and work on chunks that hold no channel costs as much as on those that do, so the steps are
// the narrowest of those that pay: time for 4680 rows of 256, fp32, against six chunks for all rows of one wave 6.4 -> 4.1 us
// (NATURAL 5.9 -> 4.2), bf16 13824 wide on 7 x 512 or 4 x 1024 against 9 x 512 45.8 -> 42.2 (NATURAL 45.2 -> 40.0), 20000 wide
// against two passes over the row 237 -> 62.  From inputs that no cache holds, WHOLE_WORDS: bf16 2048 wide on 2 x 256 against
// 3 x 256 10.6 -> 9.4, 4096 wide on 4 x 256 against 5 x 256 16.8 -> 15.4 (fp32 20.2 -> 19.6).  NATURAL takes more threads a row:
// nothing is set up per thread there.
template <typename T, Order ORD, bool TAIL>
bool launch_by_width(const ActArgs &a, int width, hipStream_t st, qarvd_status *out)
{
    auto go = [&](qarvd_status s) {
        *out = s;
        return true;
    };
    if (width <= 1 * 256) return go(launch_rows<T, 1, 64, ORD, TAIL>(a, st));
    if (width <= 2 * 256) return go(launch_rows<T, 2, 64, ORD, TAIL>(a, st));
    if constexpr (ORD == NATURAL) {
        if (width <= 2 * 512) return go(launch_rows<T, 2, 128, ORD, TAIL>(a, st));
        if (width <= 2 * 1024) return go(launch_rows<T, 2, 256, ORD, TAIL>(a, st));
        if (width <= 3 * 1024) return go(launch_rows<T, 3, 256, ORD, TAIL>(a, st));
        if (width <= 3 * 2048) return go(launch_rows<T, 3, 512, ORD, TAIL>(a, st));
        if constexpr (sizeof(T) == 4) {
            if (width <= 3 * 4096) return go(launch_rows<T, 3, 1024, ORD, TAIL>(a, st));
        } else {
            if (width <= 5 * 2048) return go(launch_rows<T, 5, 512, ORD, TAIL>(a, st));
        }
    } else {
        if (width <= 4 * 256) return go(launch_rows<T, 4, 64, ORD, TAIL>(a, st));
        if (width <= 6 * 256) return go(launch_rows<T, 6, 64, ORD, TAIL>(a, st));
        if constexpr (sizeof(T) == 2) {
            if (width <= 2 * 1024) return go(launch_rows<T, 2, 256, ORD, TAIL>(a, st));
        }
        if (width <= 3 * 1024) return go(launch_rows<T, 3, 256, ORD, TAIL>(a, st));
        if (width <= 4 * 1024) return go(launch_rows<T, 4, 256, ORD, TAIL>(a, st));
        if (width <= 5 * 1024) return go(launch_rows<T, 5, 256, ORD, TAIL>(a, st));
        if (width <= 6 * 1024) return go(launch_rows<T, 6, 256, ORD, TAIL>(a, st));
        if (width <= 5 * 2048) return go(launch_rows<T, 5, 512, ORD, TAIL>(a, st));
        if (width <= 7 * 2048) return go(launch_rows<T, 7, 512, ORD, TAIL>(a, st));
    }
    if (width <= 4 * 4096) return go(launch_rows<T, 4, 1024, ORD, TAIL>(a, st));
    if constexpr (ORD != NATURAL && sizeof(T) == 2) {
        if (width <= 9 * 2048) return go(launch_rows<T, 9, 512, ORD, TAIL>(a, st));
    }
    if (width <= 5 * 4096) return go(launch_rows<T, 5, 1024, ORD, TAIL>(a, st));
    return false;
}

template <typename T>
qarvd_status dispatch(const ActArgs &a, bool whole_words, hipStream_t st)
{
    qarvd_status s = QARVD_OK;
    const bool tail = a.K % 4 != 0;
    if (a.K >= 4) {
        if (!a.perm) {
            if (tail ? launch_by_width<T, NATURAL, true>(a, a.kp, st, &s) : launch_by_width<T, NATURAL, false>(a, a.kp, st, &s)) return s;
        } else if (whole_words) {
            if (launch_by_width<T, WHOLE_WORDS, false>(a, a.kp, st, &s)) return s;
        } else {
            if (tail ? launch_by_width<T, ANY_ORDER, true>(a, a.K, st, &s) : launch_by_width<T, ANY_ORDER, false>(a, a.K, st, &s)) return s;
        }
    }
    int grid = a.M < num_cu() * 8 ? a.M : num_cu() * 8;
    hipLaunchKernelGGL((quant_act_generic_kernel<T>), dim3(grid), dim3(TPB), 0, st, a);
    return qarvd_launch_status();
}

qarvd_status quant_act_common(const void *X, qarvd_dtype xdt, int32_t M, int32_t K, int64_t ldx,
                              const int32_t *perm, int32_t K_o, int8_t *Xq, int64_t ldxq, float *s_x,
                              bool is_static, float scale, size_t gemm_bytes, void *stream)
{
    if (!X || !Xq || (!is_static && !s_x)) return QARVD_ERR_INVALID_ARG;
    if (M <= 0 || K <= 0 || K > QARVD_MAX_K || K_o < 0 || K_o > K || ldx < K) return QARVD_ERR_INVALID_ARG;
    if (!perm && K_o != 0) return QARVD_ERR_INVALID_ARG;
    if (is_static && !(scale >= 0.0f)) return QARVD_ERR_INVALID_ARG;
    const PackedK g = qarvd_packed(K, K_o);
    if (ldxq < g.kp) return QARVD_ERR_INVALID_ARG;
    if (xdt != QARVD_F32 && xdt != QARVD_BF16) return QARVD_ERR_UNSUPPORTED;
    if (!qarvd_aligned16(Xq) || (ldxq % 16) != 0) return QARVD_ERR_UNSUPPORTED;
    const size_t esz = xdt == QARVD_F32 ? 4 : 2;
    if (reinterpret_cast<uintptr_t>(X) % esz) return QARVD_ERR_UNSUPPORTED;
    ActArgs a;
    a.X = X; a.ldx = ldx; a.perm = perm; a.Xq = Xq; a.ldxq = ldxq; a.s_x = s_x; a.static_scale = scale;
    a.M = M; a.K = K; a.K_o = K_o; a.n_off = g.n_off; a.kp = g.kp;
    a.store_wt = ((size_t)M * (size_t)g.kp <= ((size_t)40 << 20) && (size_t)M * (size_t)ldxq < ((size_t)1 << 31)) ? 1 : 0;
    a.is_static = is_static ? 1 : 0;
    const size_t x_bytes = (size_t)M * (size_t)K * esz;
    a.stream = x_bytes > STREAM_X_BYTES && x_bytes + (size_t)M * (size_t)g.kp + gemm_bytes > STREAM_CALL_BYTES ? 1 : 0;
    const bool whole_words = K % 4 == 0 && g.n_off == K_o && qarvd_aligned16(perm);
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    return xdt == QARVD_F32 ? dispatch<float>(a, whole_words, st) : dispatch<uint16_t>(a, whole_words, st);
}

}  // namespace

qarvd_status qarvd_quant_act_before_gemm(const void *X, qarvd_dtype xdt, int32_t M, int32_t K, int64_t ldx, const int32_t *perm, int32_t K_o,
                                         int8_t *Xq, int64_t ldxq, float *s_x, size_t gemm_bytes, void *stream)
{
    return quant_act_common(X, xdt, M, K, ldx, perm, K_o, Xq, ldxq, s_x, false, 0.0f, gemm_bytes, stream);
}

extern "C" qarvd_status qarvd_quant_act(const void *X, qarvd_dtype xdt, int32_t M, int32_t K, int64_t ldx,
                                        const int32_t *perm, int32_t K_o, int8_t *Xq, int64_t ldxq,
                                        float *s_x, void *stream)
{
    return quant_act_common(X, xdt, M, K, ldx, perm, K_o, Xq, ldxq, s_x, false, 0.0f, 0, stream);
}

extern "C" qarvd_status qarvd_quant_act_static(const void *X, qarvd_dtype xdt, int32_t M, int32_t K,
                                               int64_t ldx, const int32_t *perm, int32_t K_o, float scale,
                                               int8_t *Xq, int64_t ldxq, void *stream)
{
    return quant_act_common(X, xdt, M, K, ldx, perm, K_o, Xq, ldxq, nullptr, true, scale, 0, stream);
}
