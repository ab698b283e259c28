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

// Four consecutive elements of X as loaded, and widened (exactly) to fp32.
template <typename T> struct Elem;
template <> struct Elem<float> {
    typedef float4 raw;
    static __device__ __forceinline__ raw zero() { return make_float4(0.0f, 0.0f, 0.0f, 0.0f); }
    static __device__ __forceinline__ float4 widen(raw r) { return r; }
    static __device__ __forceinline__ float load1(const float *p) { return *p; }
    static __device__ __forceinline__ raw pack(float a, float b, float c, float d) { return make_float4(a, b, c, d); }
};
template <> struct Elem<uint16_t> {   // bf16 bit patterns
    typedef uint2 raw;
    static __device__ __forceinline__ raw zero() { return make_uint2(0u, 0u); }
    static __device__ __forceinline__ float4 widen(raw u)
    {
        return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xFFFF0000u), __uint_as_float(u.y << 16),
                           __uint_as_float(u.y & 0xFFFF0000u));
    }
    static __device__ __forceinline__ float load1(const uint16_t *p) { return bf16_bits_to_f32(*p); }
    static __device__ __forceinline__ raw pack(float a, float b, float c, float d)
    {
        return make_uint2((__float_as_uint(a) >> 16) | __float_as_uint(b), (__float_as_uint(c) >> 16) | __float_as_uint(d));
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
    int32_t vec;           // 1: four elements of X and of perm at a time (see quant_act_kernel)
    int32_t store_wt;      // 1: Xq leaves through write-through stores (see store_q)
};

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

// One row with IEEE divisions and channels gathered from memory: scales outside the range of the exact quotient (rows of
// magnitudes around 1e-28 and below, or with infinities), and the rows of the general kernel below.
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

// Register-resident rows.  NT threads own a token row at a time, CH chunks of 4 channels per thread (K <= CH * NT * 4);
// NT = 64: four independent rows per workgroup, no barrier.  PERM = false: the codes go straight from registers to
// memory and no LDS image exists.  VEC: rows of X can be read four channels at a time and, where there is a permutation, perm
// four entries at a time in packed order (no pads inside); else element by element.
//
// Bound by memory at large M (4680 x 8960 fp32, 210 MB from and to memory: 48 -> 42 us, the rate of a device copy; bf16
// 57 -> 30), by latency at small M (256 x 1536: 5.6 -> 3.6 us; 4680 x 1536 bf16 11.0 -> 7.5): perm and the first row are
// requested together and perm is used as it arrives, and the next row of a wave is requested before the current one is worked
// on.  (Before: codes scattered byte by byte through a channel -> position table built in LDS by every workgroup, a
// branch to an IEEE division beside every quotient.  Fetching the four bytes with one v_perm_b32 under a selector
// per dword instead of four byte reads costs more setting up than it saves: 15.5 us for the last case.)
template <typename T, int CH, int NT, bool PERM, bool VEC>
__global__ __launch_bounds__(NT == 64 ? 256 : NT, CH > 6 ? 3 : 4) void quant_act_kernel(ActArgs a)
{
    typedef typename Elem<T>::raw raw;
    constexpr int RW = NT == 64 ? 4 : 1, NWAVE = NT / 64;
    constexpr float MAGIC = 12582912.0f;       // 1.5 * 2^23: the sum rounds half-to-even, the code is its low byte
    __shared__ __align__(16) uint32_t image[PERM ? (NT == 64 ? 4 : 2) : 1][PERM ? CH * NT : 1];
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
                if constexpr (VEC) {
                    v[c] = *reinterpret_cast<const raw *>(reinterpret_cast<const char *>(x) + (uint32_t)k * (uint32_t)sizeof(T));
                } else {
                    v[c] = Elem<T>::pack(Elem<T>::load1(x + k), k + 1 < K ? Elem<T>::load1(x + k + 1) : 0.0f,
                                         k + 2 < K ? Elem<T>::load1(x + k + 2) : 0.0f, k + 3 < K ? Elem<T>::load1(x + k + 3) : 0.0f);
                }
            }
        }
    };

    // Channels of the four packed positions of this thread's dword t + c NT.  (An entry of perm outside [0, K), which makes the
    // bytes undefined, is moved inside.)
    int4 ch[PERM ? CH : 1];
    raw v[CH], vn[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) v[c] = vn[c] = Elem<T>::zero();
    auto logical = [&](int p) {                    // packed position -> index into perm, -1 at pads
        if (p < a.n_off) return p < a.K_o ? p : -1;
        const int q = a.K_o + (p - a.n_off);
        return q < K ? q : -1;
    };
    if constexpr (PERM) {
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int p = 4 * (t + c * NT);
            if constexpr (VEC) {
                ch[c] = make_int4(0, 0, 0, 0);
                if (p < K) ch[c] = *reinterpret_cast<const int4 *>(a.perm + p);
            } else {
                ch[c] = make_int4(a.perm[max(logical(p), 0)], a.perm[max(logical(p + 1), 0)], a.perm[max(logical(p + 2), 0)],
                                  a.perm[max(logical(p + 3), 0)]);
            }
        }
    }
    if (m < a.M) load_row(m, v);
    if constexpr (PERM) {
        auto inside = [&](int k) { return (int)min((unsigned)k, (unsigned)(K - 1)); };
#pragma unroll
        for (int c = 0; c < CH; ++c) ch[c] = make_int4(inside(ch[c].x), inside(ch[c].y), inside(ch[c].z), inside(ch[c].w));
    }

    for (int buf = 0; m < a.M; m += stride, buf ^= 1) {
        if (m + stride < a.M) load_row(m + stride, vn);        // flies under this row's work
        float s;
        if (a.is_static) {
            s = a.static_scale;
        } else {
            float amax = 0.0f;
#pragma unroll
            for (int c = 0; c < CH; ++c) {                     // (zeros past the end of the row)
                const float4 f = Elem<T>::widen(v[c]);
                amax = fmaxf(amax, fmaxf(fmaxf(fabsf(f.x), fabsf(f.y)), fmaxf(fabsf(f.z), fabsf(f.w))));
            }
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
        const ExactQuotient q(s, 127.0f);
        if (!q.exact()) {                              // (uniform over the row)
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
                for (int c = 0; c < CH; ++c) {
                    const int p = 4 * (t + c * NT);
                    if (p >= kp) continue;
                    uint32_t w = (uint32_t)bytes[ch[c].x] | ((uint32_t)bytes[ch[c].y] << 8) | ((uint32_t)bytes[ch[c].z] << 16) |
                                 ((uint32_t)bytes[ch[c].w] << 24);
                    if constexpr (VEC) {
                        w = p < K ? w : 0u;                        // (whole dwords of padding)
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (logical(p + e) < 0) w &= ~(0xFFu << (8 * e));
                    }
                    store_q(a, out + p, w);
                }
            }
        }
#pragma unroll
        for (int c = 0; c < CH; ++c) v[c] = vn[c];
    }
}

// Rows of more than 16384 channels: one workgroup per row, two passes over it (the second is served by the cache), gather
// through perm from global memory.
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

template <typename T, int CH, int NT, bool PERM, bool VEC>
qarvd_status launch_rows(const ActArgs &a, hipStream_t st)
{
    constexpr int RW = NT == 64 ? 4 : 1, TH = NT == 64 ? 256 : NT;
    // as many workgroups as the chip holds, trimmed so that all of them walk the same number of rows
    // (4680 rows on 1024 slots: 936 workgroups of exactly 5 rows instead of 1024 of 4 or 5)
    const int slots = num_cu() * blocks_per_cu<quant_act_kernel<T, CH, NT, PERM, VEC>>(TH);
    const int groups = (a.M + RW - 1) / RW;
    const int rounds = (groups + slots - 1) / slots;
    hipLaunchKernelGGL((quant_act_kernel<T, CH, NT, PERM, VEC>), dim3((groups + rounds - 1) / rounds), dim3(TH), 0, st, a);
    return qarvd_launch_status();
}

template <typename T>
qarvd_status dispatch(const ActArgs &a, hipStream_t st)
{
    const int ext = a.kp;      // (without outliers up to 127 more than K: the threads of a row write its padding too)
    if (a.perm && a.vec) {
        // one wave per row while a row fits its registers, then the least threads that hold it at about 24 values each
        if (ext <= 6 * 256) return launch_rows<T, 6, 64, true, true>(a, st);
        if (ext <= 6 * 512) return launch_rows<T, 6, 128, true, true>(a, st);
        if (ext <= 6 * 1024) return launch_rows<T, 6, 256, true, true>(a, st);
        if (ext <= 5 * 2048) return launch_rows<T, 5, 512, true, true>(a, st);
        if (ext <= 9 * 2048) return launch_rows<T, 9, 512, true, true>(a, st);
    } else {
        // no image to share, or element-wise loads that take many threads to keep in flight: twice the threads for a row
        if (ext <= 3 * 512) return a.perm ? launch_rows<T, 3, 128, true, false>(a, st) : a.vec ? launch_rows<T, 3, 128, false, true>(a, st) : launch_rows<T, 3, 128, false, false>(a, st);
        if (ext <= 3 * 1024) return a.perm ? launch_rows<T, 3, 256, true, false>(a, st) : a.vec ? launch_rows<T, 3, 256, false, true>(a, st) : launch_rows<T, 3, 256, false, false>(a, st);
        if (ext <= 3 * 2048) return a.perm ? launch_rows<T, 3, 512, true, false>(a, st) : a.vec ? launch_rows<T, 3, 512, false, true>(a, st) : launch_rows<T, 3, 512, false, false>(a, st);
        if (ext <= 5 * 2048) return a.perm ? launch_rows<T, 5, 512, true, false>(a, st) : a.vec ? launch_rows<T, 5, 512, false, true>(a, st) : launch_rows<T, 5, 512, false, false>(a, st);
        if (ext <= 9 * 2048) return a.perm ? launch_rows<T, 9, 512, true, false>(a, st) : a.vec ? launch_rows<T, 9, 512, false, true>(a, st) : launch_rows<T, 9, 512, false, false>(a, st);
    }
    int grid = a.M < num_cu() * 8 ? a.M : num_cu() * 8;
    hipLaunchKernelGGL((quant_act_generic_kernel<T>), dim3(grid), dim3(TPB), 0, st, a);
    return qarvd_launch_status();
}

qarvd_status quant_act_common(const void *X, qarvd_dtype xdt, int32_t M, int32_t K, int64_t ldx,
                              const int32_t *perm, int32_t K_o, int8_t *Xq, int64_t ldxq, float *s_x,
                              bool is_static, float scale, void *stream)
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
    a.vec = (K % 4 == 0) && (ldx % 4 == 0) && (reinterpret_cast<uintptr_t>(X) % (4 * esz)) == 0 &&
            (!perm || (g.n_off == K_o && qarvd_aligned16(perm))) ? 1 : 0;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    return xdt == QARVD_F32 ? dispatch<float>(a, st) : dispatch<uint16_t>(a, st);
}

}  // namespace

extern "C" qarvd_status qarvd_quant_act(const void *X, qarvd_dtype xdt, int32_t M, int32_t K, int64_t ldx,
                                        const int32_t *perm, int32_t K_o, int8_t *Xq, int64_t ldxq,
                                        float *s_x, void *stream)
{
    return quant_act_common(X, xdt, M, K, ldx, perm, K_o, Xq, ldxq, s_x, false, 0.0f, stream);
}

extern "C" qarvd_status qarvd_quant_act_static(const void *X, qarvd_dtype xdt, int32_t M, int32_t K,
                                               int64_t ldx, const int32_t *perm, int32_t K_o, float scale,
                                               int8_t *Xq, int64_t ldxq, void *stream)
{
    return quant_act_common(X, xdt, M, K, ldx, perm, K_o, Xq, ldxq, nullptr, true, scale, stream);
}
