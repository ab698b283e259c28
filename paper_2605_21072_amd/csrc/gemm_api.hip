// C entry points of the dual-scale W8A8 GEMM: argument validation, variant table and heuristic.
#include "gemm_common.h"

using namespace qarvd_gemm;

namespace {

// Kernels that a call can ask for by number.  pick_variant chooses among 27 to 41, with 1 to 4 for strides beyond 2^22; the
// others stay selectable for comparison.
const Variant kVariants[] = {
    // name, BM, BN, widest outlier block (packed bytes), needs vector output, operand strides up to 2^22, launcher
    {"staged 256x128 dual", 256, 128, 1 << 30, false, false, launch_staged<256, 128, 2, 2, true>},
    {"staged 128x128 dual", 128, 128, 1 << 30, false, false, launch_staged<128, 128, 2, 2, true>},
    {"staged 256x128 single", 256, 128, 0, false, false, launch_staged<256, 128, 2, 2, false>},
    {"staged 128x128 single", 128, 128, 0, false, false, launch_staged<128, 128, 2, 2, false>},
    {"lds-direct 256x128 (4 waves, 3 stages) dual", 256, 128, 128, true, true, launch_dma<256, 128, 2, 2, 3, true>},
    {"lds-direct 256x128 (4 waves, 3 stages) single", 256, 128, 0, true, true, launch_dma<256, 128, 2, 2, 3, false>},
    {"lds-direct 192x128 (4 waves, 3 stages) dual", 192, 128, 128, true, true, launch_dma<192, 128, 2, 2, 3, true>},
    {"lds-direct 192x128 (4 waves, 3 stages) single", 192, 128, 0, true, true, launch_dma<192, 128, 2, 2, 3, false>},
    {"lds-direct 128x128 (4 waves, 4 stages) dual", 128, 128, 128, true, true, launch_dma<128, 128, 2, 2, 4, true>},
    {"lds-direct 128x128 (4 waves, 4 stages) single", 128, 128, 0, true, true, launch_dma<128, 128, 2, 2, 4, false>},
    {"lds-direct 256x256 (8 waves, 4 stages) dual", 256, 256, 128, true, true, launch_dma<256, 256, 2, 4, 4, true>},
    {"lds-direct 256x256 (8 waves, 4 stages) single", 256, 256, 0, true, true, launch_dma<256, 256, 2, 4, 4, false>},
    {"lds-direct 256x128 (8 waves, 4 stages) dual", 256, 128, 128, true, true, launch_dma<256, 128, 4, 2, 4, true>},
    {"lds-direct 256x128 (8 waves, 4 stages) single", 256, 128, 0, true, true, launch_dma<256, 128, 4, 2, 4, false>},
    {"lds-direct 128x256 (8 waves, 4 stages) dual", 128, 256, 128, true, true, launch_dma<128, 256, 2, 4, 4, true>},
    {"lds-direct 128x256 (8 waves, 4 stages) single", 128, 256, 0, true, true, launch_dma<128, 256, 2, 4, 4, false>},
    {"16x16x64 256x224 (8 waves, 4 stages) dual", 256, 224, 128, true, true, launch_mfma16<256, 224, 4, 2, 4, true>},
    {"16x16x64 256x224 (8 waves, 4 stages) single", 256, 224, 0, true, true, launch_mfma16<256, 224, 4, 2, 4, false>},
    {"lds-direct 64x128 (4 waves, 5 stages) dual", 64, 128, 128, true, true, launch_dma<64, 128, 2, 2, 5, true>},
    {"lds-direct 64x128 (4 waves, 5 stages) single", 64, 128, 0, true, true, launch_dma<64, 128, 2, 2, 5, false>},
    {"lds-direct 64x64 (4 waves, 6 stages) dual", 64, 64, 128, true, true, launch_dma<64, 64, 2, 2, 6, true>},
    {"lds-direct 64x64 (4 waves, 6 stages) single", 64, 64, 0, true, true, launch_dma<64, 64, 2, 2, 6, false>},
    {"lds-direct 256x128 (8 waves, 6 stages) dual", 256, 128, 128, true, true, launch_dma<256, 128, 4, 2, 6, true>},
    {"lds-direct 256x128 (8 waves, 6 stages) single", 256, 128, 0, true, true, launch_dma<256, 128, 4, 2, 6, false>},
    {"lds-direct 256x128 (8 waves, 5 stages) dual", 256, 128, 128, true, true, launch_dma<256, 128, 4, 2, 5, true>},
    {"lds-direct 256x128 (8 waves, 5 stages) single", 256, 128, 0, true, true, launch_dma<256, 128, 4, 2, 5, false>},
    {"128-byte stages 256x256 (8 waves, 2 stages) dual", 256, 256, 128, true, true, launch_dma128<256, 256, 2, 4, 2, true>},
    {"128-byte stages 256x256 (8 waves, 2 stages) single", 256, 256, 0, true, true, launch_dma128<256, 256, 2, 4, 2, false>},
    {"128-byte stages 256x128 (8 waves, 3 stages) dual", 256, 128, 128, true, true, launch_dma128<256, 128, 4, 2, 3, true>},
    {"128-byte stages 256x128 (8 waves, 3 stages) single", 256, 128, 0, true, true, launch_dma128<256, 128, 4, 2, 3, false>},
    {"128-byte stages 128x256 (8 waves, 3 stages) dual", 128, 256, 128, true, true, launch_dma128<128, 256, 2, 4, 3, true>},
    {"128-byte stages 128x256 (8 waves, 3 stages) single", 128, 256, 0, true, true, launch_dma128<128, 256, 2, 4, 3, false>},
    {"128-byte stages 128x128 (8 waves, 3 stages) dual", 128, 128, 128, true, true, launch_dma128<128, 128, 2, 4, 3, true>},
    {"128-byte stages 128x128 (8 waves, 3 stages) single", 128, 128, 0, true, true, launch_dma128<128, 128, 2, 4, 3, false>},
    {"128-byte stages 64x64 (4 waves, 4 stages) dual", 64, 64, 128, true, true, launch_dma128<64, 64, 2, 2, 4, true>},
    {"128-byte stages 64x64 (4 waves, 4 stages) single", 64, 64, 0, true, true, launch_dma128<64, 64, 2, 2, 4, false>},
    {"128-byte stages 128x128 (8 waves, 3 stages) any width", 128, 128, 1 << 30, false, true, launch_dma128<128, 128, 2, 4, 3, true, true>},
    {"128-byte stages 64x64 (4 waves, 4 stages) any width", 64, 64, 1 << 30, false, true, launch_dma128<64, 64, 2, 2, 4, true, true>},
    {"128-byte stages 64x128 (8 waves, 4 stages) dual", 64, 128, 128, true, true, launch_dma128<64, 128, 2, 4, 4, true>},
    {"128-byte stages 64x128 (8 waves, 4 stages) single", 64, 128, 0, true, true, launch_dma128<64, 128, 2, 4, 4, false>},
    {"128-byte stages 64x128 (8 waves, 4 stages) any width", 64, 128, 1 << 30, false, true, launch_dma128<64, 128, 2, 4, 4, true, true>},
};
constexpr int kNumVariants = sizeof(kVariants) / sizeof(kVariants[0]);

bool short_rows_ok(const GemmArgs &g) { return g.ldxq <= (1 << 22) && g.ldwq <= (1 << 22); }

bool vector_out_ok(const GemmArgs &g, qarvd_dtype ydt)
{
    const size_t esz = ydt == QARVD_F32 ? 4 : 2;
    // the LDS-direct kernels also address a tile's rows with 32-bit byte offsets: 256 rows x stride x 4 < 2^31
    return (g.N % 8) == 0 && qarvd_aligned16(g.Y) && ((g.ldy * esz) % 16) == 0 && qarvd_aligned16(g.s_n) &&
           qarvd_aligned16(g.s_o) && qarvd_aligned16(g.bias) && short_rows_ok(g) && g.ldy <= (1 << 20);
}

bool variant_fits(const Variant &v, const GemmArgs &g, qarvd_dtype ydt)
{
    if (g.n_off > v.max_n_off) return false;
    if (v.needs_vector_out && !vector_out_ok(g, ydt)) return false;
    if (v.short_rows && !short_rows_ok(g)) return false;
    return true;
}

// Heuristic: a three-constant cost model per candidate, fitted to timings on MI355X (all tiles in turn, operands at the padded
// strides of qarvd_packed_ld, M = 16..4680, N and K = 256..13824, fixed and drawn):
//     time ~ c + ceil(tiles / CUs) * (a + b * T),     T = packed K / 64          (constants in microseconds)
// c is launch plus the first tile's lead-in, a a tile's epilogue and hand-over, b one 64-byte K step of a tile
// that has its CU to itself (two workgroups sharing a CU each run at half speed, which the ceil over
// the CUs already accounts for).  All tiles run on 128-byte-deep stages (gemm_dma128.hip):
// 256x256 has the cheapest K step per MAC and wins when N is wide; the half tiles fill the chip when N = 1536
// (4680 x 8960 -> 1536: 54 us against 79 us for 256x256) and on M of a few hundred rows with N = 8960; 128x128
// when those leave CUs empty (1560 x 8960 -> 1536: 29 us against 45, 1560 x 1536 -> 1536 9.4 against 13.0); 64x128 between that and
// 64x64 (256 x 5120 -> 5120: 15.5 against 18.8 and 17.7), 64x64 when even those would leave most without a tile (520 x 8960 ->
// 1536: 17.0 against 22.6).  The smallest tiles' 64-byte-stage forms, which were the better ones on 32x32x32, are slower than these at
// every size now (256 x 1536 -> 1536 6.7 against 5.9 us, 64 x 8960 -> 1536 19.2 against 15.3, 38 x 296 -> 1008 4.3 against 3.9).
// Depth of the rings: 128x128 on three stages (4 and 3: 1560 x 1536 -> 1536 9.8 and 9.4, 4680 x 5120 -> 5120 even), 64x64 on four
// (3 and 4: 256 x 8960 -> 1536 19.6 and 16.0; INT4 weights on three, 22.8 and 21.9 on four and three; eight: 22.7).
// What needs the general kernels (outlier block over 128 bytes, N % 8 != 0, unaligned outputs) picks by the same model
// from the three tiles built for it; operand strides beyond 2^22 go to the register-staged kernel.
int device_cus()
{
    int cus = 0;
    return (qarvd_current_device(nullptr, &cus) == QARVD_OK && cus > 0) ? cus : 256;
}

struct Cand { int variant, bm, bn; double c, a, b; };

int cheapest(const Cand *cand, int n, const GemmArgs &g)
{
    const int cus = device_cus();      // rounds are counted over the CUs of the device the call runs on
    const double T = g.kp / 64;
    const long tiles128 = (long)((g.M + 127) / 128) * ((g.N + 127) / 128);
    int best = cand[0].variant;
    double best_cost = 1e300;
    for (int i = 0; i < n; ++i) {
        const Cand &c = cand[i];
        if (c.bm == 64 && tiles128 > cus * c.bn / 64) continue;     // the small tiles only pay while 128x128 tiles leave CUs empty, or fill them badly
        const long tiles = (long)((g.M + c.bm - 1) / c.bm) * ((g.N + c.bn - 1) / c.bn);
        const double cost = c.c + (double)((tiles + cus - 1) / cus) * (c.a + c.b * T);
        if (cost < best_cost) {
            best_cost = cost;
            best = c.variant;
        }
    }
    return best;
}

int pick_variant(const GemmArgs &g, qarvd_dtype ydt)
{
    const bool dual = g.n_off > 0;
    if (g.n_off <= 128 && vector_out_ok(g, ydt)) {
        const Cand cand[6] = {{dual ? 27 : 28, 256, 256, 0.50, 7.85, 0.539},
                              {dual ? 29 : 30, 256, 128, 0.60, 5.81, 0.314},
                              {dual ? 31 : 32, 128, 256, 0.55, 5.40, 0.333},
                              {dual ? 33 : 34, 128, 128, 1.30, 3.60, 0.183},
                              {dual ? 39 : 40, 64, 128, 1.91, 2.35, 0.157},
                              {dual ? 35 : 36, 64, 64, 2.40, 0.77, 0.083}};
        return cheapest(cand, 6, g);
    }
    if (short_rows_ok(g)) {
        const Cand cand[3] = {{37, 128, 128, 1.69, 4.01, 0.181}, {41, 64, 128, 1.62, 2.97, 0.131}, {38, 64, 64, 3.13, 0.98, 0.088}};
        return cheapest(cand, 3, g);
    }
    const int cus = device_cus();
    const long tiles_big = (long)((g.M + 255) / 256) * ((g.N + 127) / 128);
    if (dual) return tiles_big >= cus ? 1 : 2;
    return tiles_big >= cus ? 3 : 4;
}

// Host-only checks of a GEMM call's arguments (all but the variant number), and the kernel arguments they give.  Wq: bits = 8 one
// byte per code, bits = 4 two codes per byte.
qarvd_status check_and_fill(int bits, const int8_t *Xq, int64_t ldxq, const float *s_x, const void *Wq, int64_t ldwq, const float *s_normal,
                            const float *s_outlier, const float *bias, int32_t M, int32_t N, int32_t K, int32_t K_o, void *Y,
                            qarvd_dtype ydt, int64_t ldy, int32_t *dbg_acc_normal, int32_t *dbg_acc_outlier, GemmArgs *out)
{
    if (!Xq || !Wq || !s_x || !s_normal || !s_outlier || !Y) return QARVD_ERR_INVALID_ARG;
    if (M <= 0 || N <= 0 || K <= 0 || K > QARVD_MAX_K || K_o < 0 || K_o > K) return QARVD_ERR_INVALID_ARG;
    const PackedK pk = qarvd_packed(K, K_o);
    if (ldxq < pk.kp || ldwq < pk.kp * bits / 8 || ldy < N) return QARVD_ERR_INVALID_ARG;
    if (ydt != QARVD_F32 && ydt != QARVD_BF16) return QARVD_ERR_UNSUPPORTED;
    if (!qarvd_aligned16(Xq) || !qarvd_aligned16(Wq) || (ldxq % 16) || (ldwq % 16)) return QARVD_ERR_UNSUPPORTED;
    const size_t esz = ydt == QARVD_F32 ? 4 : 2;
    if (reinterpret_cast<uintptr_t>(Y) % esz) return QARVD_ERR_UNSUPPORTED;
    if ((reinterpret_cast<uintptr_t>(s_x) | reinterpret_cast<uintptr_t>(s_normal) | reinterpret_cast<uintptr_t>(s_outlier) |
         reinterpret_cast<uintptr_t>(bias) | reinterpret_cast<uintptr_t>(dbg_acc_normal) |
         reinterpret_cast<uintptr_t>(dbg_acc_outlier)) & 3u)
        return QARVD_ERR_UNSUPPORTED;
    GemmArgs g;
    g.Xq = Xq; g.Wq = reinterpret_cast<const int8_t *>(Wq); g.s_x = s_x; g.s_n = s_normal; g.s_o = s_outlier; g.bias = bias;
    g.Y = Y; g.dbg_n = dbg_acc_normal; g.dbg_o = dbg_acc_outlier;
    g.ldxq = ldxq; g.ldwq = ldwq; g.ldy = ldy; g.M = M; g.N = N; g.n_off = pk.n_off; g.kp = pk.kp;
    g.tiles_m = g.tiles_n = 0; g.act = 0; g.out_scale = 0.0f; g.store_wt = 0;
    g.vec_out = vector_out_ok(g, ydt);
    *out = g;
    return QARVD_OK;
}

}  // namespace

extern "C" int32_t qarvd_gemm_num_variants(void) { return kNumVariants; }

extern "C" const char *qarvd_gemm_variant_name(int32_t variant)
{
    if (variant < 1 || variant > kNumVariants) return "";
    return kVariants[variant - 1].name;
}

extern "C" qarvd_status qarvd_w8a8_dual_gemm_variant(int32_t variant, const int8_t *Xq, int64_t ldxq,
                                                     const float *s_x, const int8_t *Wq, int64_t ldwq,
                                                     const float *s_normal, const float *s_outlier,
                                                     const float *bias, int32_t M, int32_t N, int32_t K,
                                                     int32_t K_o, void *Y, qarvd_dtype ydt, int64_t ldy,
                                                     int32_t *dbg_acc_normal, int32_t *dbg_acc_outlier,
                                                     void *stream)
{
    if (variant < 0 || variant > kNumVariants) return QARVD_ERR_INVALID_ARG;
    GemmArgs g;
    if (qarvd_status s_c = check_and_fill(8, Xq, ldxq, s_x, Wq, ldwq, s_normal, s_outlier, bias, M, N, K, K_o, Y, ydt, ldy, dbg_acc_normal,
                                          dbg_acc_outlier, &g);
        s_c != QARVD_OK)
        return s_c;
    if (variant == 0) variant = pick_variant(g, ydt);
    const Variant &v = kVariants[variant - 1];
    if (!variant_fits(v, g, ydt)) return QARVD_ERR_UNSUPPORTED;
    return v.launch(g, ydt, reinterpret_cast<hipStream_t>(stream));
}

extern "C" qarvd_status qarvd_w8a8_dual_gemm(const int8_t *Xq, int64_t ldxq, const float *s_x,
                                             const int8_t *Wq, int64_t ldwq, const float *s_normal,
                                             const float *s_outlier, const float *bias, int32_t M, int32_t N,
                                             int32_t K, int32_t K_o, void *Y, qarvd_dtype ydt, int64_t ldy,
                                             int32_t *dbg_acc_normal, int32_t *dbg_acc_outlier, void *stream)
{
    return qarvd_w8a8_dual_gemm_variant(0, Xq, ldxq, s_x, Wq, ldwq, s_normal, s_outlier, bias, M, N, K, K_o, Y, ydt,
                                        ldy, dbg_acc_normal, dbg_acc_outlier, stream);
}

// ---- W4A8: packed INT4 weights, the same kernels with the W operand widened in registers ----
namespace {
using namespace qarvd_gemm;
struct W4Variant {
    int BM, BN;
    int form;     // 0: N % 8 == 0, aligned outputs, outlier block up to 128 bytes; 1: any of these, strides up to 2^22; 2: any
    qarvd_status (*dual)(const GemmArgs &, qarvd_dtype, hipStream_t);
    qarvd_status (*single)(const GemmArgs &, qarvd_dtype, hipStream_t);
};
const W4Variant kW4Variants[] = {
    // 64-byte stages; the first is chosen by number only
    {256, 256, 0, launch_dma<256, 256, 2, 4, 4, true, true>, launch_dma<256, 256, 2, 4, 4, false, true>},
    {128, 128, 0, launch_dma<128, 128, 2, 2, 4, true, true>, launch_dma<128, 128, 2, 2, 4, false, true>},
    // register-staged: any N, any outlier-block width, any output alignment, any stride
    {128, 128, 2, launch_staged<128, 128, 2, 2, true, true>, launch_staged<128, 128, 2, 2, false, true>},
    // 128-byte stages; one build serves layers with and without outliers
    {256, 256, 0, launch_dma128<256, 256, 2, 4, 3, true, false, true>, launch_dma128<256, 256, 2, 4, 3, true, false, true>},
    {256, 128, 0, launch_dma128<256, 128, 4, 2, 3, true, false, true>, launch_dma128<256, 128, 4, 2, 3, true, false, true>},
    {128, 256, 0, launch_dma128<128, 256, 2, 4, 3, true, false, true>, launch_dma128<128, 256, 2, 4, 3, true, false, true>},
    {128, 128, 1, launch_dma128<128, 128, 2, 4, 3, true, true, true>, launch_dma128<128, 128, 2, 4, 3, true, true, true>},
    {64, 64, 1, launch_dma128<64, 64, 2, 2, 3, true, true, true>, launch_dma128<64, 64, 2, 2, 3, true, true, true>},
};
constexpr int kNumW4Variants = sizeof(kW4Variants) / sizeof(kW4Variants[0]);
}  // namespace

extern "C" int32_t qarvd_w4_gemm_num_variants(void) { return kNumW4Variants; }

extern "C" qarvd_status qarvd_w4a8_dual_gemm(const int8_t *Xq, int64_t ldxq, const float *s_x, const uint8_t *Wq4,
                                             int64_t ldwq4, const float *s_normal, const float *s_outlier,
                                             const float *bias, int32_t M, int32_t N, int32_t K, int32_t K_o, void *Y,
                                             qarvd_dtype ydt, int64_t ldy, int32_t *dbg_acc_normal,
                                             int32_t *dbg_acc_outlier, int32_t variant, void *stream)
{
    if (variant < 0 || variant > kNumW4Variants) return QARVD_ERR_INVALID_ARG;
    GemmArgs g;
    if (qarvd_status s_c = check_and_fill(4, Xq, ldxq, s_x, Wq4, ldwq4, s_normal, s_outlier, bias, M, N, K, K_o, Y, ydt, ldy, dbg_acc_normal,
                                          dbg_acc_outlier, &g);
        s_c != QARVD_OK)
        return s_c;
    const bool fast_ok = g.n_off <= 128 && g.vec_out;
    if (variant == 0) {
        // The cost model of the INT8 path, with constants of its own.  An INT4 weight stage is half as wide, so 256x256 has room for
        // three stages and less LDS traffic a K step: 4680 x 5120 -> 13824 280 us (64-byte stages 309), 4680 x 1536 -> 1536 15.7
        // (19.3), 520 x 8960 -> 1536 22.5 (41.7), 64 x 5120 -> 5120 14.4 (24.6); 2251 x 2360 -> 2252 with 150 outliers 27.0 against
        // 65.6 register-staged, which keeps strides beyond 2^22.  (The 64-byte-stage 128x128 tile is no candidate any more: level at
        // best, 2609 x 277 -> 1400 7.9 both, elsewhere 84 x 732 -> 4008 8.1 against 5.5.)
        const Cand cand[5] = {{7, 128, 128, 2.74, 3.47, 0.196}, {8, 64, 64, 3.60, 1.00, 0.101},
                              {4, 256, 256, 2.80, 8.00, 0.517}, {5, 256, 128, 1.59, 4.44, 0.366}, {6, 128, 256, 1.29, 4.79, 0.357}};
        variant = !short_rows_ok(g) ? 3 : cheapest(cand, fast_ok ? 5 : 2, g);
    }
    const int form = kW4Variants[variant - 1].form;
    if ((form == 0 && !fast_ok) || (form == 1 && !short_rows_ok(g))) return QARVD_ERR_UNSUPPORTED;     // a tile asked for by name
    const W4Variant &v = kW4Variants[variant - 1];
    return (g.n_off > 0 ? v.dual : v.single)(g, ydt, reinterpret_cast<hipStream_t>(stream));
}

// ---- chained layers: INT8 output quantized in the epilogue ----------------------------------------------
namespace {
struct Q8Variant {
    int BM, BN;
    double c, a, b;     // cost model of pick_variant
    qarvd_status (*dual)(const GemmArgs &, hipStream_t);
    qarvd_status (*single)(const GemmArgs &, hipStream_t);
};
const Q8Variant kQ8Variants[] = {
    // 64-byte stages: chosen by number only (128x128: 256 x 5120 -> 5120 28 us against 20 for the last one)
    {256, 256, 0, 0, 0, launch_dma_q8<256, 256, 2, 4, 4, true>, launch_dma_q8<256, 256, 2, 4, 4, false>},
    {128, 256, 0, 0, 0, launch_dma_q8<128, 256, 2, 4, 4, true>, launch_dma_q8<128, 256, 2, 4, 4, false>},
    {128, 128, 0, 0, 0, launch_dma_q8<128, 128, 2, 2, 4, true>, launch_dma_q8<128, 128, 2, 2, 4, false>},
    {256, 256, 1.48, 11.37, 0.489, launch_dma128_q8<256, 256, 2, 4, 2, true>, launch_dma128_q8<256, 256, 2, 4, 2, false>},
    {256, 128, 1.53, 6.29, 0.319, launch_dma128_q8<256, 128, 4, 2, 3, true>, launch_dma128_q8<256, 128, 4, 2, 3, false>},
    {128, 256, 1.38, 6.22, 0.326, launch_dma128_q8<128, 256, 2, 4, 3, true>, launch_dma128_q8<128, 256, 2, 4, 3, false>},
    {128, 128, 1.49, 3.83, 0.159, launch_dma128_q8<128, 128, 4, 2, 3, true>, launch_dma128_q8<128, 128, 4, 2, 3, false>},
};
constexpr int kNumQ8Variants = sizeof(kQ8Variants) / sizeof(kQ8Variants[0]);
}  // namespace

extern "C" int32_t qarvd_q8_gemm_num_variants(void) { return kNumQ8Variants; }

extern "C" qarvd_status qarvd_w8a8_dual_gemm_q8(const int8_t *Xq, int64_t ldxq, const float *s_x, const int8_t *Wq,
                                                int64_t ldwq, const float *s_normal, const float *s_outlier,
                                                const float *bias, int32_t M, int32_t N, int32_t K, int32_t K_o,
                                                qarvd_act act, float out_scale, int8_t *Y8, int64_t ldy8,
                                                int32_t variant, void *stream)
{
    if (!Xq || !Wq || !s_x || !s_normal || !s_outlier || !Y8) return QARVD_ERR_INVALID_ARG;
    if (M <= 0 || N <= 0 || K <= 0 || K > QARVD_MAX_K || K_o < 0 || K_o > K) return QARVD_ERR_INVALID_ARG;
    if (act != QARVD_ACT_NONE && act != QARVD_ACT_GELU_TANH) return QARVD_ERR_INVALID_ARG;
    if (!(out_scale >= 1.0e-30f) || out_scale > 1.0e30f) return QARVD_ERR_INVALID_ARG;     // NaN, zero, negative, inf; 1 / s must be normal
    if (variant < 0 || variant > kNumQ8Variants) return QARVD_ERR_INVALID_ARG;
    const PackedK pk = qarvd_packed(K, K_o);
    if (ldxq < pk.kp || ldwq < pk.kp || ldy8 < N) return QARVD_ERR_INVALID_ARG;
    if (!qarvd_aligned16(Xq) || !qarvd_aligned16(Wq) || (ldxq % 16) || (ldwq % 16)) return QARVD_ERR_UNSUPPORTED;
    if ((reinterpret_cast<uintptr_t>(s_x) & 3u) || !qarvd_aligned16(s_normal) || !qarvd_aligned16(s_outlier) ||
        !qarvd_aligned16(bias))
        return QARVD_ERR_UNSUPPORTED;
    // 16 codes per store; 32-bit byte offsets inside a tile
    if ((N % 16) || !qarvd_aligned16(Y8) || (ldy8 % 16) || ldxq > (1 << 22) || ldwq > (1 << 22) || ldy8 > (1 << 22))
        return QARVD_ERR_UNSUPPORTED;
    GemmArgs g;
    g.Xq = Xq; g.Wq = Wq; g.s_x = s_x; g.s_n = s_normal; g.s_o = s_outlier; g.bias = bias;
    g.Y = Y8; g.dbg_n = nullptr; g.dbg_o = nullptr;
    g.ldxq = ldxq; g.ldwq = ldwq; g.ldy = ldy8; g.M = M; g.N = N; g.n_off = pk.n_off; g.kp = pk.kp;
    g.tiles_m = g.tiles_n = 0; g.act = (int32_t)act; g.out_scale = out_scale; g.vec_out = 1; g.store_wt = 0;
    if (g.n_off > 128) return QARVD_ERR_UNSUPPORTED;
    if (variant == 0) {
        const double T = g.kp / 64;
        double best_cost = 1e300;
        const int cus = device_cus();
        for (int i = 0; i < kNumQ8Variants; ++i) {
            const Q8Variant &c = kQ8Variants[i];
            if (c.a == 0) continue;
            const long tiles = (long)((M + c.BM - 1) / c.BM) * ((N + c.BN - 1) / c.BN);
            const double cost = c.c + (double)((tiles + cus - 1) / cus) * (c.a + c.b * T);
            if (cost < best_cost) { best_cost = cost; variant = i + 1; }
        }
    }
    const Q8Variant &v = kQ8Variants[variant - 1];
    return (g.n_off > 0 ? v.dual : v.single)(g, reinterpret_cast<hipStream_t>(stream));
}

// ---- the online pair in one call ------------------------------------------------------------------------------
// Workspace: Xq [M, packed_ld] | s_x [M]; packed_ld is a multiple of 128, so both are aligned.
extern "C" size_t qarvd_linear_workspace(int32_t M, int32_t K, int32_t K_o)
{
    const int32_t ld = K_o < 0 ? 0 : qarvd_packed_ld(K, K_o);
    return M > 0 && ld > 0 ? (size_t)M * (size_t)ld + (size_t)M * sizeof(float) : 0;
}

extern "C" qarvd_status qarvd_linear(const void *X, qarvd_dtype xdt, int64_t ldx, const int32_t *perm, int32_t w_bits,
                                     const void *Wq, int64_t ldwq, const float *s_normal, const float *s_outlier,
                                     const float *bias, int32_t M, int32_t N, int32_t K, int32_t K_o, void *Y,
                                     qarvd_dtype ydt, int64_t ldy, void *workspace, size_t workspace_bytes, void *stream)
{
    const size_t need = qarvd_linear_workspace(M, K, K_o);
    if (need == 0 || (w_bits != 8 && w_bits != 4)) return QARVD_ERR_INVALID_ARG;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 127u) || workspace_bytes < need) return QARVD_ERR_WORKSPACE;
    const int64_t ld = qarvd_packed_ld(K, K_o);
    int8_t *const Xq = reinterpret_cast<int8_t *>(workspace);
    float *const s_x = reinterpret_cast<float *>(Xq + (size_t)M * (size_t)ld);
    // Both halves' arguments are checked before the first of them is launched: the GEMM's here, quant_act's by itself.
    GemmArgs g;
    if (qarvd_status s_c = check_and_fill(w_bits, Xq, ld, s_x, Wq, ldwq, s_normal, s_outlier, bias, M, N, K, K_o, Y, ydt, ldy, nullptr,
                                          nullptr, &g);
        s_c != QARVD_OK)
        return s_c;
    const size_t gemm_bytes = (size_t)N * ((size_t)g.kp * w_bits / 8 + (size_t)M * (ydt == QARVD_F32 ? 4 : 2));
    if (qarvd_status st = qarvd_quant_act_before_gemm(X, xdt, M, K, ldx, K_o > 0 ? perm : nullptr, K_o, Xq, ld, s_x, gemm_bytes, stream); st != QARVD_OK)
        return st;
    if (w_bits == 4)
        return qarvd_w4a8_dual_gemm(Xq, ld, s_x, reinterpret_cast<const uint8_t *>(Wq), ldwq, s_normal, s_outlier, bias, M, N, K, K_o,
                                    Y, ydt, ldy, nullptr, nullptr, 0, stream);
    return qarvd_w8a8_dual_gemm_variant(0, Xq, ld, s_x, reinterpret_cast<const int8_t *>(Wq), ldwq, s_normal, s_outlier, bias, M, N, K,
                                        K_o, Y, ydt, ldy, nullptr, nullptr, stream);
}
