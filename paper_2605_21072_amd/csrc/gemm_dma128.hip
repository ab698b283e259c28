// LDS-direct dual-scale W8A8 GEMM for gfx950 with 128-byte-deep K stages (appendix "Quantization Kernels",
// kernel (ii); Eq. (dual_scale)): INT8 x INT8 -> INT32 on v_mfma_i32_16x16x64_i8, fp32 dequant epilogue.
//
// Same design as the 64-byte-stage kernel (persistent workgroups, a ring of LDS stages filled by
// buffer_load ... lds, the outlier head tile visited last and re-multiplied from LDS in the epilogue, scales
// double-buffered in LDS, swizzled output patches), with two differences that matter on MI355X.
//
// A stage row is a whole 128-byte cache line.  One LDS-direct load moves 8 rows x 128 bytes, so every line that leaves the L2
// is used completely by the instruction that asked for it; with 64-byte rows each line is requested twice, one
// iteration apart, and under load (all CUs streaming) the vector L1 fill path then delivers half as many useful
// bytes (measured with a K-loop skeleton on 256 CUs: 2500 against 1220 cycles per 256 x 256 x 64 step).
//
// The instruction is 16x16x64.  The chip is power-limited on real data, and a MAC costs less energy there than in 32x32x32 (half
// the accumulator traffic per MAC): a 256 x 256 K loop without epilogue runs at 3.08 POPS with 16x16x64 and at 2.69 with
// 32x32x32 on Gaussian codes, although it takes more cycles (zeros as operands, where the clock stays up: 3.6 and 4.1).  Same
// tiles on 32x32x32 against now, us: 4680 x 8960 -> 1536 62.2 -> 58.3, 4680 x 5120 -> 13824 302 -> 290 (128 x 256: 308 -> 284),
// 4680 x 1536 -> 8960 76.9 -> 75.0, 4680 x 1536 -> 1536 15.8 -> 15.0, 520 x 8960 -> 1536 on 64 x 64 21.1 -> 17.0 (two k-steps a
// stage instead of four, each with twice the MFMAs to hide its reads behind).
// Consequences:
//   * two MFMA k-steps of 64 bytes per stage, all fragments of the next in flight under this one's MFMAs, one barrier per stage;
//   * the outlier range (at most 128 packed bytes, in units of 32) is exactly the first K tile: one head tile, H <= 1.  Where it
//     ends in the middle of a k-step, that step is multiplied twice, with the other half's lanes zeroed;
//   * a lane owns 4 consecutive columns of every 16x16 block and the same columns in every row block, so the epilogue reads
//     its scales and biases once a tile, and an output patch is whole 128-byte lines (whole 64-byte sectors for bf16 outputs of
//     tiles up to 128 x 128 and for INT8 outputs);
//   * a stage is refilled by the iteration that consumed it (its last fragments are in registers before the
//     iteration's barrier, and each wave waits for its own LDS reads before arriving), so all NSTAGE stages are
//     in use and a load has NSTAGE - 1 iterations to land; 256 x 256 tiles run with two 64 KB stages;
//   * where the LDS has room (256 x 256) the output patches get their own 16 KB behind the stages, so a whole
//     stage is free for the next tile's first K tile during the epilogue; otherwise they sit in a free stage;
//   * 256 x 256 tiles need all 256 registers of a wave: no second copy of the K loop (rows below the matrix are multiplied as the
//     zeros they load as, which costs issue slots but hardly power), and the accumulators are cleared, not started from an inline
//     zero in a first iteration of its own (which the compiler no longer keeps in place: 140 registers spilled).
//
// GEN = true is the general form: an outlier block of any width, any N, any output alignment.  Tiles of at most 64
// accumulator registers a wave have room for a second set, so the K loop runs in natural order and the sums move to
// the outlier set where the range ends; nothing is kept in LDS or multiplied again.  Outputs that are not whole
// 16-byte chunks leave through unaligned 16-byte stores, the last partial chunk of a row element by element.
// Against the register-staged kernel that took these shapes before: 2251 x 2360 x 2252, 150 outliers, fp32 out
// 64.1 -> 26 us; 4680 x 5120 x 13825, 200 outliers 1213 -> 369; 20 x 13824 x 700 126 -> 29; 1001 x 1003 x 1005
// 21.1 -> 6.6.  256 x 128 tiles (two full sets leave too few registers: 60 spilled) were 27 us on the first
// and 352 on the second and are not built.
#include <algorithm>
#include <type_traits>

#include "gemm_dma_common.h"

namespace qarvd_gemm {

namespace {

constexpr int BK2 = 128;                  // K bytes per stage row
constexpr int KS2 = BK2 / 64;             // MFMA k-steps per stage
constexpr int PATCH2_BYTES = 2048;        // output patch of a wave: 16 rows of 128 bytes, or 32 of 64

// Swizzle for 128-byte LDS rows (eight 16-byte slots).  A row covers half of the 64 banks, so rows of equal
// parity share their banks.  A fragment read (ds_read_b128, lane l -> row l & 15, chunk l >> 4 of a k-step's four)
// must spread over all banks both when the hardware groups lanes {8p..8p+7, 32+8p..32+8p+7} (eight consecutive
// rows times the chunks c and c ^ 2) and when it groups sixteen consecutive lanes (sixteen consecutive rows, one
// chunk): rows r, r+2, r+4, r+6 take slots that differ in bits 0 and 2, rows r and r+8 in bit 1.
__device__ __forceinline__ int swz128(int r) { return ((r >> 1) & 1) | (((r >> 3) & 1) << 1) | (((r >> 2) & 1) << 2); }

// 64-byte rows of packed INT4 (four chunks, two a k-step, an 8-byte read per lane): four rows cover the banks once, so rows r,
// r + 4, r + 8, r + 12 put a chunk into different slots.
__device__ __forceinline__ int swz_w4(int r) { return (r >> 2) & 3; }

// W4: the W operand is packed INT4, 64 bytes per row and stage.
template <int BM, int BN, int WM, int WN, int NSTAGE, bool W4>
struct Geo2 {
    static constexpr int NW = WM * WN;
    static constexpr int THREADS = 64 * NW;
    static constexpr int WTM = BM / WM, WTN = BN / WN;
    static constexpr int TM = WTM / 16, TN = WTN / 16;
    static constexpr int WROW = W4 ? 64 : BK2;                     // bytes of a W row in a stage
    static constexpr int WGRP = W4 ? 16 : 8;                       // W rows an LDS-direct load (1 KB) covers
    static constexpr int NA = BM / 8 / NW, NB = BN / WGRP / NW;    // LDS-direct loads per wave per stage
    static constexpr int NLOAD = NA + NB;
    static constexpr int STG = BM * BK2 + BN * WROW;
    static constexpr int PATCHES = NW * PATCH2_BYTES;
    static constexpr int NSCALE = BM + 3 * BN;
    static constexpr int SCALE_BYTES = 2 * NSCALE * (int)sizeof(float);
    static constexpr bool PATCH_EXTRA = NSTAGE * STG + PATCHES + SCALE_BYTES <= 160 * 1024;   // patches behind the stages
    static constexpr int PATCH_OFF = NSTAGE * STG;
    static constexpr int SCALES_OFF = NSTAGE * STG + (PATCH_EXTRA ? PATCHES : 0);
    static constexpr int LDS_BYTES = SCALES_OFF + SCALE_BYTES;
    static constexpr int SPT = (NSCALE + THREADS - 1) / THREADS;
    static_assert(BM % (8 * NW) == 0 && BN % (WGRP * NW) == 0, "row groups must divide over the waves");
    static_assert(NW % 2 == 0, "the load swizzle takes bit 3 of a row from the wave number");
    static_assert(WTM % 32 == 0 && WTN % 32 == 0, "wave tile is TM x TN blocks of 16 x 16, stored in pairs");
    static constexpr int WG_PER_CU = NW >= 8 || 2 * LDS_BYTES > 160 * 1024 ? 1 : 8 / NW;     // bounded by LDS, two waves per SIMD
    static constexpr int WAVES_PER_SIMD = WG_PER_CU * NW >= 8 ? 2 : 1;
    static_assert(TM * TN * 4 <= 256 / WAVES_PER_SIMD, "accumulators: half of the registers a wave can have");
    static_assert(PATCHES <= STG, "the output patches fit into one stage");
    static_assert(PATCH_EXTRA ? NSTAGE >= 2 : NSTAGE >= 3, "a head tile, the patches and one stage for the next tile");
    static_assert(LDS_BYTES <= 160 * 1024, "LDS per workgroup");
    static_assert((NSTAGE - 1) * NLOAD < 64, "vmcnt is a 6-bit counter");
};

typedef v4i v4i_unaligned __attribute__((aligned(2)));   // 16 bytes at an address that is aligned to an output element only

// WT: output stores write through the L2 (see output_writes_through).
template <int BM, int BN, int WM, int WN, int NSTAGE, bool DUAL, bool DBG, typename OutT, bool GEN, bool W4, bool WT>
__global__ __launch_bounds__(64 * WM * WN, (Geo2<BM, BN, WM, WN, NSTAGE, W4>::WAVES_PER_SIMD)) void gemm_dma128_kernel(GemmArgs g)
{
    using G = Geo2<BM, BN, WM, WN, NSTAGE, W4>;
    constexpr int TM = G::TM, TN = G::TN, NA = G::NA, NB = G::NB, NW = G::NW, STG = G::STG, NL = G::NLOAD;
    extern __shared__ __align__(16) unsigned char smem[];
    float *const sc_both = reinterpret_cast<float *>(smem + G::SCALES_OFF);   // 2 x { s_x[BM] | s_n[BN] | s_o[BN] | bias[BN] }

    const long long p_ts = QARVD_PROF ? clock64() : 0;
    const long long p_rs = QARVD_PROF ? wall_clock64() : 0;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int ntiles = g.tiles_m * g.tiles_n;
    int tile = blockIdx.x;
    int m0, n0;                                    // tile being computed

    // ---- LDS-direct load addressing: load i of this wave fills rows (NW*i + wave)*8 .. +8 of the operand tile;
    // lane l fills slot (l & 7) of row (l >> 3) of those with global chunk (l & 7) ^ swz128(row in the tile).  Tile base in the
    // descriptor, one byte offset per lane and operand, the load's rows and the K position as scalar offset.  The descriptor
    // covers the rows of the tile that exist, so rows past the matrix read as zeros and cost no traffic (their products land
    // in rows / columns that are never stored).
    const int drow = lane >> 3;
    const int dchunk = ((lane & 7) ^ swz128(8 * (wave & 1) + drow)) << 4;      // (NW is even: row bit 3 = wave bit 0)
    const int ldx = (int)g.ldxq, ldw = (int)g.ldwq;
    const int va = (wave * 8 + drow) * ldx + dchunk;
    const int vb = W4 ? (wave * 16 + (lane >> 2)) * ldw + (((lane & 3) ^ swz_w4(lane >> 2)) << 4)      // 16 rows x 64 bytes per load
                      : (wave * 8 + drow) * ldw + dchunk;
    const int8_t *base_a, *base_b;
    int bytes_a, bytes_b;
    int lm0, ln0;                                  // tile the load addressing points at
    auto aim_loads = [&](int t) {
        int tm, tn;
        tile_coords(t, g.tiles_m, g.tiles_n, tm, tn);
        lm0 = tm * BM;
        ln0 = tn * BN;
        base_a = g.Xq + (size_t)lm0 * g.ldxq;
        base_b = g.Wq + (size_t)ln0 * g.ldwq;
        bytes_a = (min(BM, g.M - lm0) - 1) * ldx + g.kp;
        bytes_b = (min(BN, g.N - ln0) - 1) * ldw + (W4 ? g.kp / 2 : g.kp);
    };
    auto issue = [&](int ktile, int stage) {
        unsigned char *sb = smem + stage * STG;
        const int koff = ktile * BK2;
#pragma unroll
        for (int i = 0; i < NA; ++i)
            buffer_load_lds16(base_a, bytes_a, va, koff + i * NW * 8 * ldx, sb + (NW * i + wave) * 1024);
#pragma unroll
        for (int i = 0; i < NB; ++i)
            buffer_load_lds16(base_b, bytes_b, vb, (W4 ? koff / 2 : koff) + i * NW * G::WGRP * ldw, sb + BM * BK2 + (NW * i + wave) * 1024);
    };

    // ---- scales and bias: registers during the previous tile's K loop, then the other LDS buffer ----
    float r_s[G::SPT];
    auto fetch_scales = [&](int sm0, int sn0) {
#pragma unroll
        for (int u = 0; u < G::SPT; ++u) {
            const int e = tid + u * G::THREADS;
            float v = 0.f;
            if (e < BM) v = g.s_x[min(sm0 + e, g.M - 1)];
            else if (e < BM + BN) v = g.s_n[min(sn0 + e - BM, g.N - 1)] * (W4 ? 0.0625f : 1.0f);             // INT4 codes enter the
            else if (e < BM + 2 * BN) v = g.s_o[min(sn0 + e - BM - BN, g.N - 1)] * (W4 ? 0.0625f : 1.0f);    // MFMA times 16 (exact)
            else if (e < BM + 3 * BN && g.bias) v = g.bias[min(sn0 + e - BM - 2 * BN, g.N - 1)];
            r_s[u] = v;
        }
    };
    auto park_scales = [&](int buf) {
        float *dst = sc_both + buf * G::NSCALE;
#pragma unroll
        for (int u = 0; u < G::SPT; ++u) {
            const int e = tid + u * G::THREADS;
            if (e < G::NSCALE) dst[e] = r_s[u];
        }
    };
    // fetched and parked on every pass, for the last tile too (it re-reads its own), so that each fetch is
    // followed by its use on every path and the compiler never drains the stage loads to protect these registers
    auto fetch_next_scales = [&](int t) {
        int tm, tn;
        tile_coords(min(t, ntiles - 1), g.tiles_m, g.tiles_n, tm, tn);
        fetch_scales(tm * BM, tn * BN);
    };

    // ---- fragment addressing: lane l reads row (l & 15), chunk 4*ks + (l >> 4) of a k-step ----
    const int frow = lane & 15, fq = lane >> 4, fsw = swz128(frow);
    const int x_base = (wm * G::WTM + frow) * BK2;               // X rows: MFMA B operand
    const int w_base = BM * BK2 + (wn * G::WTN + frow) * G::WROW + (W4 ? 8 * (fq & 1) : 0);    // W rows: MFMA A operand
    int coff[KS2], wcoff[KS2];
#pragma unroll
    for (int ks = 0; ks < KS2; ++ks) {
        coff[ks] = (((4 * ks) | fq) ^ fsw) << 4;
        wcoff[ks] = W4 ? (((2 * ks) | (fq >> 1)) ^ swz_w4(frow)) << 4 : coff[ks];     // packed INT4: k-step ks is two chunks, 8 bytes a lane
    }
    auto read_w = [&](const unsigned char *sb, int j, int c) -> v4i {   // W fragment of block j, k-step offset c
        if constexpr (W4) return unpack_w4(*reinterpret_cast<const v2i *>(sb + w_base + j * 16 * G::WROW + c));
        else return *reinterpret_cast<const v4i *>(sb + w_base + j * 16 * BK2 + c);
    };
    auto read_x = [&](const unsigned char *sb, int i, int c) -> v4i {
        return *reinterpret_cast<const v4i *>(sb + x_base + i * 16 * BK2 + c);
    };

    v4i acc[TM][TN];
    v4i acc_o[GEN ? TM : 1][GEN ? TN : 1];      // (GEN) the outlier sum, moved here when the K loop passes its end
    static_assert(!GEN || TM * TN <= 16, "two accumulator sets");
    v4i xf[KS2][TM], wf[KS2][TN];
    const v4i zero4 = {0, 0, 0, 0};
    auto load_frags = [&](const unsigned char *sb, int ks) {
#pragma unroll
        for (int j = 0; j < TN; ++j) wf[ks][j] = read_w(sb, j, wcoff[ks]);
#pragma unroll
        for (int i = 0; i < TM; ++i) xf[ks][i] = read_x(sb, i, coff[ks]);
    };
    auto mma_to = [&](auto &sums, int ks, int keep) {      // keep: -1, or 0 in lanes whose part of the k-step is left out
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                sums[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wf[ks][j] & keep, xf[ks][i], sums[i][j], 0, 0, 0);
    };
    auto mma = [&](int ks) { mma_to(acc, ks, -1); };
    auto clear = [&](auto &sums) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) sums[i][j] = zero4;
    };
    auto mask_w = [&](int ks, bool keep) {         // lanes that do not keep their bytes multiply by zero
#pragma unroll
        for (int j = 0; j < TN; ++j) wf[ks][j] = keep ? wf[ks][j] : zero4;
    };
    // Instruction-order hints (masks: 0x008 MFMA, 0x100 LDS read, 0x020 VMEM read).  The fragment reads of the next k-step go
    // out behind the first MFMAs of this one, one each, the refill's loads behind every second one after them: the reads then
    // have the rest of the k-step to land (256 x 256: spread evenly over the k-step 3.08, so 3.16 POPS in a K loop without epilogue).
    auto interleave = [&](auto loads_tag) {
        constexpr int S = TM * TN, R = TM + TN, L = decltype(loads_tag)::value ? NL : 0;
        constexpr int FREE = S > R ? S - R : 1;    // MFMAs without a read behind them
        int loads = 0;
#pragma unroll
        for (int m = 0; m < S; ++m) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            if (m < R) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            while (loads < L && loads * FREE < (m + 1 - R) * L) {
                __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
                ++loads;
            }
        }
    };
    auto interleave_reads = [&]() { interleave(std::false_type{}); };
    auto interleave_reads_and_loads = [&]() { interleave(std::true_type{}); };

    // ---- K tiles: T >= 1 of 128 bytes.  Tile 0 holds the outlier range (when there is one) and is visited last:
    // order H, .., T-1, 0.  Iteration `it` reads stage (base + it) % NSTAGE and, once read, refills it.
    const int T = g.kp / BK2;
    const int o_steps = DUAL ? g.n_off / 32 : 0;      // the outlier range in units of half a k-step, 32 bytes (!GEN: <= 4)
    const int H = !GEN && o_steps > 0 ? 1 : 0;
    const int Tn = T - H;
    auto seq = [&](int it) { return it < Tn ? it + H : it - Tn; };
    const int NPRO = min(NSTAGE, T);                  // stages filled before a tile's K loop starts
    const int PF = min(NSTAGE - H - (G::PATCH_EXTRA ? 0 : 1), NPRO);   // of those, under the previous epilogue (>= 1)

    int base = 0, sbuf = 0;
    bool first_stage_landed = false, rest_pending = false;
    aim_loads(tile);
    fetch_scales(lm0, ln0);
    issue(seq(0), 0);   // a fixed number of loads, so the wait the compiler puts before the scale writes covers
    park_scales(0);     // exactly the scale fetch and leaves the stage loads in flight
#pragma unroll
    for (int p = 1; p < NSTAGE; ++p)
        if (p < T) issue(seq(p), p);
    long long p_vm = 0, p_bar = 0, p_loop = 0, p_epi = 0, p_pro = 0, p_mark = p_ts;
    int p_tiles = 0;

    for (;;) {
    m0 = lm0;
    n0 = ln0;
    const int next_tile = tile + (int)gridDim.x;
    const bool more = next_tile < ntiles;
    // The wait counts assume only stage loads are outstanding; the previous tile's output stores may still be,
    // but they are older than every load issued after them, so the waits only get stricter.  A tile whose first
    // stage was prefetched under the previous epilogue waits for nothing here: that epilogue waited for the
    // prefetch before its first store.
    if (!first_stage_landed) wait_stages_in_flight<NSTAGE - 1, NL>(NPRO - 1);
    __builtin_amdgcn_s_barrier();   // first stage visible; everyone has left the previous tile's epilogue
    fetch_next_scales(next_tile);   // (before the stage loads: the waits count those from the youngest)
    if (rest_pending) {
        for (int p = PF; p < NPRO; ++p) issue(seq(p), (base + p) % NSTAGE);
    }
    load_frags(smem + base * STG, 0);
    int stage = base;
    [[maybe_unused]] const long long p_t0 = QARVD_PROF ? clock64() : 0;

    // iteration it:  MFMA F0 | read F1 under it;  wait, barrier;  MFMA F1 | read F0(it+1), refill this stage with K tile it+NSTAGE
    // Before the barrier a wave waits for its own loads of stage it+1 and for its own LDS reads (the last
    // fragments of this stage), so after the barrier stage it+1 is complete and stage `it` is dead.
    auto next_of = [&](int st) { return st + 1 == NSTAGE ? 0 : st + 1; };
    auto first_half = [&]() {
        load_frags(smem + stage * STG, 1);
        mma(0);
        interleave_reads();
        __builtin_amdgcn_sched_barrier(0);       // the waits must not float up into the MFMAs
    };
    auto refill_half = [&](int ktile) {
#if QARVD_PROF
        const long long q1 = clock64();
#endif
        wait_vmcnt<(NSTAGE - 2) * NL>();
        wait_lgkmcnt0();
        __builtin_amdgcn_s_barrier();
#if QARVD_PROF
        p_bar += clock64() - q1;
#endif
        load_frags(smem + next_of(stage) * STG, 0);
        issue(ktile, stage);
        mma(1);
        interleave_reads_and_loads();
        __builtin_amdgcn_sched_barrier(0);
        stage = next_of(stage);
    };
    if constexpr (GEN) {
        // Natural K order.  The tiles up to the one in which the outlier range ends go through an unscheduled loop, that one is
        // multiplied twice, each time with the lanes of the other range zeroed, and the rest runs through the scheduled iteration
        // with nothing in it that knows of the split (a test between the k-steps of one loop for all cost 40 % of its rate).
        const int o_tile = o_steps >> 2, o_sub = o_steps & 3;
        auto other_half = [&](int it, auto mma1) {
            if (it + 1 < T) {
                wait_stages_in_flight<NSTAGE - 2, NL>(T - 2 - it);
                wait_lgkmcnt0();
                __builtin_amdgcn_s_barrier();
            }
            mma1();
            __builtin_amdgcn_sched_barrier(0);
            if (it + 1 < T) load_frags(smem + next_of(stage) * STG, 0);
            if (it + NSTAGE < T) issue(it + NSTAGE, stage);
            stage = next_of(stage);
        };
        clear(acc_o);
        int it = 0;
#pragma unroll 1
        for (; it < o_tile && it < T; ++it) {
            load_frags(smem + stage * STG, 1);
            mma_to(acc_o, 0, -1);
            other_half(it, [&]() { mma_to(acc_o, 1, -1); });
        }
        clear(acc);
        if (o_sub > 0 && it < T) {
            const int in0 = o_sub > (fq >> 1) ? -1 : 0, in1 = o_sub > 2 + (fq >> 1) ? -1 : 0;       // this lane's half k-steps of the range
            load_frags(smem + stage * STG, 1);
            mma_to(acc_o, 0, in0);
            mma_to(acc, 0, ~in0);
            other_half(it, [&]() {
                mma_to(acc_o, 1, in1);
                mma_to(acc, 1, ~in1);
            });
            ++it;
        }
        for (; it < T - NSTAGE; ++it) {
            first_half();
            refill_half(it + NSTAGE);
        }
#pragma unroll 1
        for (; it < T; ++it) {
            first_half();
            if (it + 1 < T) {
                wait_stages_in_flight<NSTAGE - 2, NL>(T - 2 - it);
                wait_lgkmcnt0();
                __builtin_amdgcn_s_barrier();
                load_frags(smem + next_of(stage) * STG, 0);
            }
            mma(1);
            stage = next_of(stage);
        }
    } else {
        clear(acc);
        int it = 0;
        for (; it < T - NSTAGE; ++it) {          // steady state: every tile here is a normal tile
            first_half();
            refill_half(seq(it + NSTAGE));
        }
        // the last tiles, nothing left to issue
#pragma unroll 1
        for (; it < T - 1; ++it) {
            first_half();
            wait_stages_in_flight<NSTAGE - 2, NL>(T - 2 - it);       // stage it + 1 has landed
            wait_lgkmcnt0();
            __builtin_amdgcn_s_barrier();
            load_frags(smem + next_of(stage) * STG, 0);
            mma(1);
            interleave_reads();
            __builtin_amdgcn_sched_barrier(0);
            stage = next_of(stage);
        }
        // the very last one is the head tile, if there is one: only its normal part, what lies past the outlier range (which may
        // end in the middle of a k-step), is summed here
        load_frags(smem + stage * STG, 1);
        if (o_steps == 1) mask_w(0, fq >= 2);
        if (o_steps < 2) mma(0);
        if (o_steps == 3) mask_w(1, fq >= 2);
        if (o_steps < 4) mma(1);
    }
    [[maybe_unused]] const long long p_t1 = QARVD_PROF ? clock64() : 0;
    wait_lgkmcnt0();                // this wave's scale writes and fragment reads have landed ...
    __builtin_amdgcn_s_barrier();   // ... and everyone is done with every stage but the head tile's

    // ---- epilogue -------------------------------------------------------------------------
    // the head tile sits in stage (base + Tn) % NSTAGE; the patches behind the stages, or in the stage read just
    // before the head; the rest of the ring takes the next tile's first PF stages
    // (the lane number is taken anew: what the epilogue derives from it would otherwise be kept, or spilled, through the K loop)
    int el = lane;
    asm volatile("" : "+v"(el));
    const int er = el & 15, eq = el >> 4;
    const int hstage0 = (base + Tn) % NSTAGE;
    const int pstage = (base + Tn - 1 + 2 * NSTAGE) % NSTAGE;
    const int nbase = (base + T) % NSTAGE;
    park_scales(sbuf ^ 1);          // free since the previous tile's epilogue; nothing else is in flight here
    if (more) {
        aim_loads(next_tile);
        for (int p = 0; p < PF; ++p) issue(seq(p), (nbase + p) % NSTAGE);
    }
    const float *sc_lds = sc_both + sbuf * G::NSCALE;
    const float *sx_lds = sc_lds, *sn_lds = sc_lds + BM, *so_lds = sc_lds + BM + BN, *bs_lds = sc_lds + BM + 2 * BN;
    unsigned char *const patch = (G::PATCH_EXTRA ? smem + G::PATCH_OFF : smem + pstage * STG) + wave * PATCH2_BYTES;
    OutT *Y = reinterpret_cast<OutT *>(g.Y);
    constexpr int ESZ = (int)sizeof(OutT), EPC = 16 / ESZ;     // output elements per 16-byte chunk
    // A patch is 16 rows of 128 bytes, whole lines of the output, or 32 rows of 64 where a wave's row is that short.  Block (i, j)
    // puts this lane's four outputs, columns 16 j + 4 eq .., into row 16 i + er.  Read back, lane l takes chunk l % chunks of a
    // row; the rows go to the lanes so that the sixteen lanes a pass serves, 8p .. 8p+7 and 32+8p .. 32+8p+7, cover the banks.
    constexpr int PRS = G::WTN * ESZ >= 128 ? 128 : 64, PROWS = PATCH2_BYTES / PRS, PCH = PRS / 16;
    constexpr int PCB = PRS / ESZ / 16, PRB = PROWS / 16;      // blocks of a patch: columns, rows
    static_assert(G::WTN * ESZ % PRS == 0 && (PRB == 1 || PCB == TN), "patches are whole rows of the wave tile, or parts of one row block");
    auto pswz = [](int row) { return PRS == 128 ? swz128(row) : (row >> 2) & 3; };
    const int prow = PRS == 128 ? 2 * ((el >> 3) & 3) + (el >> 5) : 4 * ((el >> 3) & 3) + 2 * (el >> 5) + ((el >> 2) & 1);
    const int pch = el & (PCH - 1);
    const int pw_addr = er * PRS + ((((4 * eq * ESZ) >> 4) ^ pswz(er)) << 4) + ((4 * eq * ESZ) & 15);     // column block 0 of a patch
    unsigned char *const y_tile = reinterpret_cast<unsigned char *>(Y + (size_t)m0 * g.ldy);
    const int ldy_b = (int)g.ldy * ESZ;
    const int y_bytes = (min(BM, g.M - m0) - 1) * ldy_b + g.N * ESZ;
    const int y_lane = (wm * G::WTM + prow) * ldy_b + (n0 + wn * G::WTN + pch * EPC) * ESZ;
    const int n_left = g.N - n0 - wn * G::WTN - pch * EPC;            // columns from this lane's chunk to the matrix edge
    const StaticQuant sq = make_static_quant(sizeof(OutT) == 1 ? g.out_scale : 1.0f);

    // Software pipeline over the 16 x 16 blocks, row blocks outermost: a patch is read back as soon as it is complete and
    // stored after the next block's arithmetic; the outlier MFMAs of a row of blocks start before its arithmetic.  A lane
    // serves the same 4 TN columns in every row block, so their scales and biases are read once a tile, and so are the W fragments
    // of the outlier range's first 64 bytes.
    auto epilogue = [&](auto steps_tag) {
        constexpr int OSTEPS = decltype(steps_tag)::value;      // k-steps of the outlier range (GEN: 1 if there is one)
        constexpr bool HASO = OSTEPS > 0;
        v4i pend[2];
        int pend_voff = 0, pend_soff = 0, pend_row = 0, pend_col = 0;
        bool pending = false, stored = false;       // compile-time after unrolling
        auto store_unaligned = [&]() {              // (GEN) rows that are not whole, 16-byte aligned chunks
            const int left = n_left - pend_col;     // columns of the matrix from this lane's chunk on
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int ml = wm * G::WTM + pend_row + p * (PROWS / 2) + prow;
                if (m0 + ml >= g.M) continue;
                OutT *const y = Y + (size_t)(m0 + ml) * g.ldy + (g.N - left);
                if (left >= EPC) {
                    *reinterpret_cast<v4i_unaligned *>(y) = pend[p];
                } else if (left > 0) {              // the last, partial chunk of a row
                    using bits_t = std::conditional_t<ESZ == 4, uint32_t, uint16_t>;
#pragma unroll
                    for (int k = 0; k < EPC - 1; ++k)
                        if (k < left) reinterpret_cast<bits_t *>(y)[k] = (bits_t)((unsigned)pend[p][k * ESZ / 4] >> (8 * (k * ESZ % 4)));
                }
            }
        };
        auto flush_commit = [&]() {                 // patch (already in registers) -> global
            if (!pending) return;
            if (!stored) {
                // the next tile's first stages were issued when this epilogue began; waiting for them before the
                // first output store means no later stage wait has an output store ahead of it in the counter
                __builtin_amdgcn_sched_barrier(0);
#if QARVD_PROF == 2
                const long long q0 = clock64();
#endif
                wait_vmcnt<0>();
#if QARVD_PROF == 2
                p_vm += clock64() - q0;      // (diagnostic build 2: o[1] = ticks spent in this wait, summed over the tiles)
#endif
                __builtin_amdgcn_sched_barrier(0);
                stored = true;
            }
            if constexpr (GEN) {
                if (!g.vec_out) store_unaligned();
            }
            if (!GEN || g.vec_out) {
#pragma unroll
                for (int p = 0; p < 2; ++p) buffer_store16(y_tile, y_bytes, pend_voff, pend_soff + p * (PROWS / 2) * ldy_b, pend[p], WT);
            }
            pending = false;
        };
        auto flush = [&](int row0, int col0) {      // first row and column of the patch inside the wave tile
            flush_commit();
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int row = p * (PROWS / 2) + prow;
                pend[p] = *reinterpret_cast<const v4i *>(patch + row * PRS + ((pch ^ pswz(row)) << 4));
            }
            pend_voff = col0 + EPC <= n_left ? y_lane : 0x7ffffff0;
            pend_soff = row0 * ldy_b + col0 * ESZ;
            pend_row = row0;
            pend_col = col0;
            pending = true;
        };

        v4f sn[TN], so[TN], bs[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int nt = wn * G::WTN + j * 16 + 4 * eq;             // column inside the workgroup tile
            sn[j] = *reinterpret_cast<const v4f *>(sn_lds + nt);
            if constexpr (HASO) so[j] = *reinterpret_cast<const v4f *>(so_lds + nt);
            bs[j] = *reinterpret_cast<const v4f *>(bs_lds + nt);
        }
        // The outlier sum of a block is multiplied while the block before it is worked on, from fragments read a row of blocks
        // ahead.  Half k-steps past the end of the outlier range multiply by zero in the X fragment.
        constexpr bool HEAD = HASO && !GEN;
        const unsigned char *hb = smem + hstage0 * STG;
        const int keep0 = o_steps > (eq >> 1) ? -1 : 0, keep1 = o_steps > 2 + (eq >> 1) ? -1 : 0;
        constexpr bool HOLD = HEAD && OSTEPS == 1;      // the W fragments stay in registers, where there is room for them
        v4i wh[HOLD ? TN : 1], xo0, xo1, xn0 = zero4, xn1 = zero4, ao_next = zero4;
        auto read_head = [&](int i) {
            if constexpr (HEAD) xn0 = read_x(hb, i, coff[0]) & keep0;
            if constexpr (HEAD && OSTEPS > 1) xn1 = read_x(hb, i, coff[1]) & keep1;
        };
        auto head_mma = [&](int j) {
            if constexpr (HEAD) ao_next = __builtin_amdgcn_mfma_i32_16x16x64_i8(HOLD ? wh[HOLD ? j : 0] : read_w(hb, j, wcoff[0]), xo0, zero4, 0, 0, 0);
            if constexpr (HEAD && OSTEPS > 1) ao_next = __builtin_amdgcn_mfma_i32_16x16x64_i8(read_w(hb, j, wcoff[1]), xo1, ao_next, 0, 0, 0);
        };
        if constexpr (HOLD) {
#pragma unroll
            for (int j = 0; j < TN; ++j) wh[j] = read_w(hb, j, wcoff[0]);
        }
        read_head(0);
        xo0 = xn0;
        xo1 = xn1;
        head_mma(0);
        float sx_next = sx_lds[wm * G::WTM + er];
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const float sx = sx_next;
            if (i + 1 < TM) {
                sx_next = sx_lds[wm * G::WTM + (i + 1) * 16 + er];
                read_head(i + 1);
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                v4i ao;
                if constexpr (HASO && GEN) {
                    ao = acc_o[i][j];
                } else {
                    ao = ao_next;
                    if (j == TN - 1) {
                        xo0 = xn0;
                        xo1 = xn1;
                    }
                    if (i + 1 < TM || j + 1 < TN) head_mma((j + 1) % TN);
                }
                float y[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float v;
                    if constexpr (HASO) {
                        v = (float)ao[e] * so[j][e];
                        v = fmaf((float)acc[i][j][e], sn[j][e], v);
                    } else {
                        // acc_o == 0: (float)0 * s_o is +0 and the first fma reduces to this one
                        v = fmaf((float)acc[i][j][e], sn[j][e], 0.0f);
                    }
                    y[e] = fmaf(v, sx, bs[j][e]);
                }
                if constexpr (DBG) {
                    const int m = m0 + wm * G::WTM + i * 16 + er, n = n0 + wn * G::WTN + j * 16 + 4 * eq;
                    if (m < g.M) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            if (n + e >= g.N) continue;
                            if (g.dbg_n) g.dbg_n[(size_t)m * g.N + n + e] = acc[i][j][e] >> (W4 ? 4 : 0);
                            if (g.dbg_o) {
                                int aov = 0;
                                if constexpr (HASO) aov = ao[e] >> (W4 ? 4 : 0);
                                g.dbg_o[(size_t)m * g.N + n + e] = aov;
                            }
                        }
                    }
                }
                unsigned char *const pw = patch + (i % PRB) * 16 * PRS + (pw_addr ^ ((j % PCB) * 16 * ESZ));
                if constexpr (sizeof(OutT) == 1) {
                    // chained layer: activation, then the next layer's static scale (Eq. (quantization))
                    *reinterpret_cast<unsigned *>(pw) = quantize4_static<out_is_gelu<OutT>::value>(y, sq);
                } else if constexpr (sizeof(OutT) == 2) {
                    v2u pk;
                    pk.x = cvt_pk_bf16(y[0], y[1]);
                    pk.y = cvt_pk_bf16(y[2], y[3]);
                    *reinterpret_cast<v2u *>(pw) = pk;
                } else {
                    *reinterpret_cast<v4f *>(pw) = v4f{y[0], y[1], y[2], y[3]};
                }
                if (i % PRB == PRB - 1 && j % PCB == PCB - 1) flush(i / PRB * PROWS, j / PCB * PCB * 16);
            }
        }
        flush_commit();
    };
    if (!DUAL || o_steps == 0) epilogue(std::integral_constant<int, 0>{});
    else if (GEN || o_steps <= 2) epilogue(std::integral_constant<int, DUAL ? 1 : 0>{});
    else epilogue(std::integral_constant<int, DUAL && !GEN ? 2 : 0>{});
#if QARVD_PROF
    {
        const long long p_t2 = clock64();
        if (p_tiles == 0) { if (QARVD_PROF != 2) p_vm = p_t0 - p_mark; } else p_pro += p_t0 - p_mark;
        p_loop += p_t1 - p_t0; p_epi += p_t2 - p_t1; p_mark = p_t2; ++p_tiles;
    }
#endif
    if (!more) break;
    first_stage_landed = true;      // PF >= 1
    rest_pending = true;
    base = nbase;
    sbuf ^= 1;
    tile = next_tile;
    }
#if QARVD_PROF
    if (lane == 0) {   // per wave: sums over its tiles of loop, lead-in, barrier-wait, epilogue, hand-over ticks
        OutT *Yp = reinterpret_cast<OutT *>(g.Y);
        int *o = (DBG && g.dbg_o) ? g.dbg_o + ((size_t)blockIdx.x * NW + wave) * 8
                                  : reinterpret_cast<int *>(Yp + (size_t)g.M * g.ldy) + ((size_t)blockIdx.x * NW + wave) * 8;
        o[0] = (int)p_loop; o[1] = (int)p_vm; o[2] = (int)p_bar; o[3] = (int)p_epi; o[4] = (int)(wall_clock64() - p_rs);
        o[5] = p_tiles; o[6] = (int)(clock64() - p_ts); o[7] = (int)p_pro;
    }
#else
    (void)p_vm; (void)p_bar; (void)p_loop; (void)p_epi; (void)p_pro; (void)p_mark; (void)p_tiles; (void)p_rs;
#endif
}

// Output stores write through the L2 where they are whole 64-byte sectors: nothing is left to write back when the kernel ends, and the
// L2s keep the operands.  Against plain stores of more than 40 MB, us, GEMM alone: 4680 x 1536 -> 8960 bf16 69.6 -> 65.2, INT8
// out 76.1 -> 73.4; 4680 x 5120 -> 13824 INT8 out 285 -> 276 (with a kernel that reads the output next 93.6 -> 90.6, 89.6 -> 88.1, 306
// -> 297).  Rows that begin inside a sector share theirs with the next tile's stores, in another XCD's L2: there it costs more than it
// saves beyond 40 MB, for outputs up to that size it is level (1536 -> 4616 bf16, 41 MB: 41.4 plain, 42.5 written through).
// Plain and written through: 1536 -> 8968 bf16 65.3 and 77.3 (with a reader 91.2 and 109), 1536 -> 8976 64.8 and 70.5, 1536 -> 8968 fp32 84.4
// and 125, 5120 -> 13832 bf16 270 and 305, general tile with 200 outliers 1536 -> 8968 bf16 85.8 and 99.7; rows at 64 bytes,
// 1536 -> 8992 bf16, 67.8 and 65.1; INT8 outputs, whose rows are whole 16-byte chunks, level (1536 -> 13840 125 both, with a reader 146.5
// and 149.5).  The choice is a kernel's, not a branch's: at every store it cost 2 to 4 % of the GEMM.
bool output_writes_through(const GemmArgs &g, size_t elem)
{
    return (size_t)g.M * (size_t)g.N * elem <= ((size_t)40 << 20) || ((g.ldy * (int64_t)elem | (int64_t)reinterpret_cast<uintptr_t>(g.Y)) & 63) == 0;
}

template <int BM, int BN, int WM, int WN, int NSTAGE, bool DUAL, bool DBG, typename OutT, bool GEN, bool W4, bool WT = true>
qarvd_status launch128_one(const GemmArgs &g, hipStream_t st)
{
    using G = Geo2<BM, BN, WM, WN, NSTAGE, W4>;
    // (the smaller tiles are not chosen for outputs that large, and a dump of the accumulators is not timed)
    if constexpr (WT && BM >= 128 && !DBG && sizeof(OutT) > 1)
        if (!output_writes_through(g, sizeof(OutT))) return launch128_one<BM, BN, WM, WN, NSTAGE, DUAL, DBG, OutT, GEN, W4, false>(g, st);
    auto k = gemm_dma128_kernel<BM, BN, WM, WN, NSTAGE, DUAL, DBG, OutT, GEN, W4, WT>;
    static unsigned long long lds_limit_raised = 0;      // one mask per instantiation, i.e. per kernel symbol
    if (qarvd_status st_a = qarvd_raise_lds_limit_once(k, G::LDS_BYTES, lds_limit_raised); st_a != QARVD_OK) return st_a;
    int grid = 0;
    if (qarvd_status st_g = persistent_grid(g.tiles_m * g.tiles_n, G::WG_PER_CU, &grid); st_g != QARVD_OK) return st_g;
    hipLaunchKernelGGL(k, dim3(grid), dim3(G::THREADS), G::LDS_BYTES, st, g);
    return qarvd_launch_status();
}

}  // namespace

template <int BM, int BN, int WM, int WN, int NSTAGE, bool DUAL, bool GEN, bool W4>
qarvd_status launch_dma128(const GemmArgs &g0, qarvd_dtype ydt, hipStream_t st)
{
    GemmArgs g = g0;
    g.tiles_m = (g.M + BM - 1) / BM;
    g.tiles_n = (g.N + BN - 1) / BN;
    const bool dbg = g.dbg_n != nullptr || g.dbg_o != nullptr;   // raw-accumulator dumps: separate, slower build
    if (ydt == QARVD_BF16)
        return !dbg ? launch128_one<BM, BN, WM, WN, NSTAGE, DUAL, false, uint16_t, GEN, W4>(g, st)
                    : launch128_one<BM, BN, WM, WN, NSTAGE, DUAL, true, uint16_t, GEN, W4>(g, st);
    return !dbg ? launch128_one<BM, BN, WM, WN, NSTAGE, DUAL, false, float, GEN, W4>(g, st)
                : launch128_one<BM, BN, WM, WN, NSTAGE, DUAL, true, float, GEN, W4>(g, st);
}

template <int BM, int BN, int WM, int WN, int NSTAGE, bool DUAL>
qarvd_status launch_dma128_q8(const GemmArgs &g0, hipStream_t st)
{
    GemmArgs g = g0;
    g.tiles_m = (g.M + BM - 1) / BM;
    g.tiles_n = (g.N + BN - 1) / BN;
    return g.act == 1 ? launch128_one<BM, BN, WM, WN, NSTAGE, DUAL, false, Int8GeluOut, false, false>(g, st)
                      : launch128_one<BM, BN, WM, WN, NSTAGE, DUAL, false, Int8Out, false, false>(g, st);
}

#define QARVD_INST128_Q8(BM, BN, WM, WN, NS)                                                         \
    template qarvd_status launch_dma128_q8<BM, BN, WM, WN, NS, true>(const GemmArgs &, hipStream_t); \
    template qarvd_status launch_dma128_q8<BM, BN, WM, WN, NS, false>(const GemmArgs &, hipStream_t);
QARVD_INST128_Q8(256, 256, 2, 4, 2)
QARVD_INST128_Q8(256, 128, 4, 2, 3)
QARVD_INST128_Q8(128, 256, 2, 4, 3)
QARVD_INST128_Q8(128, 128, 4, 2, 3)

#define QARVD_INST128(BM, BN, WM, WN, NS)                                                                        \
    template qarvd_status launch_dma128<BM, BN, WM, WN, NS, true, false, false>(const GemmArgs &, qarvd_dtype, hipStream_t);   \
    template qarvd_status launch_dma128<BM, BN, WM, WN, NS, false, false, false>(const GemmArgs &, qarvd_dtype, hipStream_t);
QARVD_INST128(256, 256, 2, 4, 2)
QARVD_INST128(256, 128, 4, 2, 3)
QARVD_INST128(128, 256, 2, 4, 3)
QARVD_INST128(128, 128, 2, 4, 3)
QARVD_INST128(64, 128, 2, 4, 4)
QARVD_INST128(64, 64, 2, 2, 4)

#define QARVD_INST128_GEN(BM, BN, WM, WN, NS)                                                                    \
    template qarvd_status launch_dma128<BM, BN, WM, WN, NS, true, true, false>(const GemmArgs &, qarvd_dtype, hipStream_t);
QARVD_INST128_GEN(128, 128, 2, 4, 3)
QARVD_INST128_GEN(64, 128, 2, 4, 4)
QARVD_INST128_GEN(64, 64, 2, 2, 4)

#define QARVD_INST128_W4(BM, BN, WM, WN, NS, GEN)                                                                    \
    template qarvd_status launch_dma128<BM, BN, WM, WN, NS, true, GEN, true>(const GemmArgs &, qarvd_dtype, hipStream_t);
QARVD_INST128_W4(256, 256, 2, 4, 3, false)
QARVD_INST128_W4(256, 128, 4, 2, 3, false)
QARVD_INST128_W4(128, 256, 2, 4, 3, false)
QARVD_INST128_W4(128, 128, 2, 4, 3, true)
QARVD_INST128_W4(64, 64, 2, 2, 3, true)

}  // namespace qarvd_gemm
