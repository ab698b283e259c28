// Shared host/device helpers of the gfx950 library (not used by the CPU oracle).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/qarvd.h"

#define QARVD_HIP_TRY(expr)                      \
    do {                                         \
        hipError_t e__ = (expr);                 \
        if (e__ != hipSuccess) {                 \
            (void)hipGetLastError();             \
            return QARVD_ERR_HIP;                \
        }                                        \
    } while (0)

// qarvd_quant_act with a GEMM right behind it that moves `gemm_bytes` of weights and output (quant_act.hip).
__attribute__((visibility("hidden")))
qarvd_status qarvd_quant_act_before_gemm(const void *X, qarvd_dtype xdt, int32_t M, int32_t K, int64_t ldx, const int32_t *perm, int32_t K_o,
                                         int8_t *Xq, int64_t ldxq, float *s_x, size_t gemm_bytes, void *stream);

static inline qarvd_status qarvd_launch_status()
{
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? QARVD_OK : QARVD_ERR_HIP;
}

// Compute-unit count of the current device.  Device attributes are read once per device and kept for the life
// of the process (the only state the library holds besides which kernels already had their LDS limit raised).
static inline qarvd_status qarvd_current_device(int *dev_out, int *cus_out)
{
    static int cu_count[64] = {0};              // filled on first use; the same value from any thread
    int dev = 0;
    QARVD_HIP_TRY(hipGetDevice(&dev));
    int cus = (dev >= 0 && dev < 64) ? cu_count[dev] : 0;
    if (cus <= 0) {
        QARVD_HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
        if (dev >= 0 && dev < 64) cu_count[dev] = cus;
    }
    if (dev_out) *dev_out = dev;
    if (cus_out) *cus_out = cus;
    return QARVD_OK;
}

// Raises a kernel's dynamic-LDS limit the first time it is launched on a device instead of on every launch
// (the call costs microseconds of host time, as much as a short kernel).  `done` is one bit per device,
// a static of the calling launcher, so there is one mask per kernel symbol; the attribute only ever grows.
template <typename Kernel>
static inline qarvd_status qarvd_raise_lds_limit_once(Kernel kernel, int bytes, unsigned long long &done)
{
    int dev = 0;
    QARVD_HIP_TRY(hipGetDevice(&dev));
    const unsigned long long bit = (dev >= 0 && dev < 64) ? (1ull << dev) : 0ull;
    if (bit && (__atomic_load_n(&done, __ATOMIC_ACQUIRE) & bit)) return QARVD_OK;
    QARVD_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
    if (bit) __atomic_fetch_or(&done, bit, __ATOMIC_RELEASE);
    return QARVD_OK;
}

static inline bool qarvd_aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

static inline int32_t qarvd_round_up(int32_t x, int32_t m) { return (x + m - 1) / m * m; }

// Packed-row geometry (see the layout comment in qarvd.h).
struct PackedK {
    int32_t K, K_o;
    int32_t n_off;   // start of the normal block
    int32_t kp;      // packed extent, multiple of 128
};
static inline PackedK qarvd_packed(int32_t K, int32_t K_o)
{
    PackedK g;
    g.K = K;
    g.K_o = K_o;
    g.n_off = qarvd_round_up(K_o, 32);
    g.kp = qarvd_round_up(g.n_off + (K - K_o), 128);
    return g;
}

// Eq. (quantization), symmetric, z = 0, clip to [-127,127], round-half-even; s == 0 -> 0.
// The division is the IEEE-correct fp32 division hipcc emits by default.
__device__ __forceinline__ int quantize_i8(float x, float s)
{
    if (s == 0.0f) return 0;
    float r = rintf(x / s);
    r = fminf(fmaxf(r, -127.0f), 127.0f);
    return (int)r;
}

// The same quantizer with the symmetric range of another bit-width: q in [-qmax, qmax], qmax = 2^(b-1) - 1.
__device__ __forceinline__ int quantize_sym(float x, float s, float qmax)
{
    if (s == 0.0f) return 0;
    float r = rintf(x / s);
    r = fminf(fmaxf(r, -qmax), qmax);
    return (int)r;
}

// ExactQuotients x / s for one scale.  RN(1 / s) times x, corrected twice with fused multiply-adds, IS the correctly rounded
// quotient for 1e-30 <= s <= 1e30 and |x| <= 127.5 s (Markstein's theorem; the argument stands at quantize4_static in
// gemm_dma_common.h): five instructions and no branch, where a product with a redo of the IEEE division near rounding
// boundaries takes as many and 500 bytes of code per value (8960 x 1536: 21 -> 19 us).  s == 0 (a block of zeros, or none): every quotient is 0.
struct ExactQuotient {
    float s, rs, bound;      // bound = RN(qmax s): beyond it the code is +-qmax whatever the quotient
    __device__ __forceinline__ ExactQuotient(float scale, float qmax) : s(scale), rs(scale == 0.0f ? 0.0f : 1.0f / scale), bound(qmax * scale) {}
    __device__ __forceinline__ bool exact() const { return s == 0.0f || (s >= 1e-30f && s <= 1e30f); }
    __device__ __forceinline__ float clamped(float x) const        // quotient of x clamped to [-bound, bound]
    {
        x = __builtin_amdgcn_fmed3f(x, -bound, bound);
        const float q0 = x * rs;
        const float q1 = fmaf(fmaf(-q0, s, x), rs, q0);
        return fmaf(fmaf(-q1, s, x), rs, q1);
    }
};

__device__ __forceinline__ float bf16_bits_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// fp32 -> bf16 bits, round-to-nearest-even (finite inputs).
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return u >> 16;
}

// Reductions over a wave by data-parallel-primitive moves: the values pass between lanes inside vector-ALU
// instructions (sixteen lanes of a row, then the last lane of a row to the next), a few cycles a step, where a shuffle
// goes through the LDS crossbar at its latency, six times in a row.  The result is in lane 63 and is read
// from there, so every lane gets it in a scalar register.  `idle` is what a lane without a source receives.
template <int CTRL> __device__ __forceinline__ int dpp_move(int idle, int v)
{
    return __builtin_amdgcn_update_dpp(idle, v, CTRL, 0xF, 0xF, false);
}
template <typename Step> __device__ __forceinline__ int wave_reduce_bits(int v, Step step)      // step(v, moved copy of v)
{
    v = step(v, [](int idle, int x) { return dpp_move<0x111>(idle, x); });      // row_shr:1, 2, 4, 8
    v = step(v, [](int idle, int x) { return dpp_move<0x112>(idle, x); });
    v = step(v, [](int idle, int x) { return dpp_move<0x114>(idle, x); });
    v = step(v, [](int idle, int x) { return dpp_move<0x118>(idle, x); });
    v = step(v, [](int idle, int x) { return dpp_move<0x142>(idle, x); });      // row_bcast:15, 31
    v = step(v, [](int idle, int x) { return dpp_move<0x143>(idle, x); });
    return __builtin_amdgcn_readlane(v, 63);
}
__device__ __forceinline__ int wave_sum_all(int v)
{
    return wave_reduce_bits(v, [](int x, auto move) { return x + move(0, x); });
}
// Inclusive running sum over the lanes, by the same moves (the row_bcast steps add to the rows behind their source only).
__device__ __forceinline__ int wave_scan(int v)
{
    v += dpp_move<0x111>(0, v);
    v += dpp_move<0x112>(0, v);
    v += dpp_move<0x114>(0, v);
    v += dpp_move<0x118>(0, v);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);
    return v;
}
__device__ __forceinline__ unsigned wave_min_all(unsigned v)
{
    return (unsigned)wave_reduce_bits((int)v, [](int x, auto move) { return (int)min((unsigned)x, (unsigned)move(x, x)); });
}
__device__ __forceinline__ float wave_max_all(float v)
{
    return __int_as_float(wave_reduce_bits(__float_as_int(v), [](int x, auto move) {
        return __float_as_int(fmaxf(__int_as_float(x), __int_as_float(move(x, x))));
    }));
}
__device__ __forceinline__ double wave_sum_all(double v)
{
    auto add = [](double x, auto move) {
        const long long b = __double_as_longlong(x);
        const unsigned lo = (unsigned)move(0, (int)b), hi = (unsigned)move(0, (int)(b >> 32));
        return x + __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
    };
    v = add(v, [](int idle, int x) { return dpp_move<0x111>(idle, x); });
    v = add(v, [](int idle, int x) { return dpp_move<0x112>(idle, x); });
    v = add(v, [](int idle, int x) { return dpp_move<0x114>(idle, x); });
    v = add(v, [](int idle, int x) { return dpp_move<0x118>(idle, x); });
    v = add(v, [](int idle, int x) { return dpp_move<0x142>(idle, x); });
    v = add(v, [](int idle, int x) { return dpp_move<0x143>(idle, x); });
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)b, 63), hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), 63);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
