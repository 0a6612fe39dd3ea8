// bf16 matrix multiply C = A B (fp32 accumulation) for gfx950 (MI355X): the GEMM of the paper's
// appendix as a second workload, and the reference point for what a kernel made of MFMAs and LDS
// traffic alone sustains on this chip.
//
// One workgroup computes a TM x TN tile of C with WM x WN waves, each wave a (TM/WM) x (TN/WN) part of
// it in 16 x 16 accumulator blocks.  A and B are streamed in steps of 64 along K through a ring of
// kStages LDS stages filled by direct global->LDS loads:
//
//   A stage  TM rows x 64 k     (128-byte rows; 16-byte chunks XOR-swizzled for 16-row same-chunk b128 reads)
//   B stage  64 k x TN columns, as panels of 64 columns (128-byte rows; swizzled for the transposing reads
//            that turn k-major rows into "8 consecutive k per lane")
//
// The products are issued as D^T: v_mfma_f32_16x16x32_bf16(B fragment, A fragment), so that a lane owns one
// ROW of C and stores 4 consecutive columns at a time.  The fragments of one half step (32 k) are read from
// LDS while the MFMAs of the half step before it run; the barrier that frees a stage sits in the middle of a
// step, and the loads that refill it follow one at a time between the MFMAs of the second half.
//
// KS > 1: KS groups of WM x WN waves in one workgroup share the K range, group g taking the steps g, g + KS, ...
// with a ring of its own; the partial sums meet in LDS at the end, always in the same order.
#include "tk_common.h"
#include "tk_launch.h"

#include <type_traits>

namespace tk {

// sixteen zero bytes: the source of the chunks of A and the rows of B that lie beyond K
__device__ __attribute__((aligned(16))) const bf16 g_gemm_zero[8] = {};

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// A: 16 lanes read the same chunk of 16 consecutive rows; 128-byte rows alternate between the two halves of the banks
__device__ __forceinline__ int gemm_swz_a(int row) { return (row >> 1) & 7; }
// B: 32 lanes read 32 bytes of the rows r..r+3 and r+8..r+11 (one transposing read)
__device__ __forceinline__ int gemm_swz_b(int row) { return (((row >> 1) & 1) | (((row >> 3) & 1) << 1)) << 1; }

template <int TM, int TN, int WM, int WN, int KS, int STAGES>
struct GemmTile {
    static constexpr int kTileM = TM, kTileN = TN, kTileK = 64;
    static constexpr int kGroupThreads = 64 * WM * WN, kThreads = kGroupThreads * KS;
    static constexpr int kStages = STAGES;
    static constexpr int kPartM = TM / WM, kPartN = TN / WN;            // of one wave
    static constexpr int kBlocksM = kPartM / 16, kBlocksN = kPartN / 16;
    static constexpr int kABytes = TM * 128, kStageBytes = kABytes + TN * 128;
    static constexpr int kALoads = TM * 8 / kGroupThreads, kBLoads = TN * 8 / kGroupThreads;    // per thread and step
    static constexpr int kLoads = kALoads + kBLoads;
    static constexpr int kLdsBytes = KS * STAGES * kStageBytes;
    static_assert(TM * 8 % kGroupThreads == 0 && TN * 8 % kGroupThreads == 0 && TN % 64 == 0, "whole loads per thread");
    static_assert((KS - 1) * TM * TN * 4 <= kLdsBytes && kLdsBytes <= 160 * 1024, "LDS");
};

// Any M >= 1, N and K multiples of 8 (so that every row starts on a 16-byte boundary).  The kernel works on
// whole tiles: rows of A past M fetch row M-1 and columns of B past N fetch the last 8 columns (their results
// are never stored), and in the step that runs past K the chunks of A and the rows of B beyond it are fetched
// from a block of zeros.  The offsets are clamped once, ahead of the loop; a step that lies within K runs the
// same instructions whatever the shape.
//
// WIDE: lane offsets in 64 bits, for matrices whose rows within one tile lie 4 GiB or more apart (gemm_fits_32_bits).
// Otherwise an offset is a 32-bit register next to a scalar base, which saves a 64-bit vector addition per load.
template <class S, int WM, int WN, int KS, int WAVES_PER_SIMD, bool WIDE>
__global__ __launch_bounds__(S::kThreads, WAVES_PER_SIMD)
void gemm_kernel(const bf16* __restrict__ A, const bf16* __restrict__ B, bf16* __restrict__ C,
                 int M, int N, int K, int tiles_m, int tiles_n, int super_m)
{
    constexpr int MB = S::kBlocksM, NB = S::kBlocksN;
    __shared__ __attribute__((aligned(1024))) char lds[S::kLdsBytes];

    const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kg = KS == 1 ? 0 : wave_all / (WM * WN);              // this wave's share of K
    const int wave = KS == 1 ? wave_all : wave_all % (WM * WN);
    const int tid = threadIdx.x - kg * S::kGroupThreads;
    const int lane = threadIdx.x & 63;
    const int l16 = lane & 15;
    const int quad = lane >> 4;
    const int wm = wave / WN, wn = wave % WN;
    char* const ring = lds + kg * (S::kStages * S::kStageBytes);

    // tile order: XCD-contiguous ids, then groups of super_m tile rows walked column by column, so
    // the workgroups resident on one XCD share a few A and B panels in its L2 (Section 3.3 of the
    // paper makes the same point about block order for its GEMM)
    const int total = tiles_m * tiles_n;
    const int logical = xcd_remap(blockIdx.x, total);
    const int super_rows = (tiles_m / super_m) * super_m;
    int tm, tn;
    if (logical < super_rows * tiles_n) {
        const int grp = logical / (super_m * tiles_n), in = logical % (super_m * tiles_n);
        tm = grp * super_m + in % super_m;
        tn = in / super_m;
    } else {
        const int rest = tiles_m - super_rows, in = logical - super_rows * tiles_n;
        tm = super_rows + in % rest;
        tn = in / rest;
    }
    const int m0 = tm * S::kTileM, n0 = tn * S::kTileN;

    // ---- per-thread source offsets (bytes from the tile's first row / column) of the direct-to-LDS loads of one stage
    // A: LDS position s = it * threads + tid holds (row = s / 8, physical chunk = s % 8)
    // B: position s holds (panel = s / 512, k row = s / 8 % 64, physical chunk = s % 8)
    const bf16* const a_tile = A + (size_t)m0 * K;
    const bf16* const b_tile = B + n0;
    using Offset = std::conditional_t<WIDE, uint64_t, uint32_t>;
    Offset a_src[S::kALoads], b_src[S::kBLoads];
#pragma unroll
    for (int it = 0; it < S::kALoads; it++) {
        const int s = it * S::kGroupThreads + tid, pc = s & 7;
        int row = s >> 3;
        const int chunk = pc ^ gemm_swz_a(row);
        if (row > M - 1 - m0) row = M - 1 - m0;
        a_src[it] = ((Offset)row * (Offset)K + chunk * 8) * 2;
    }
#pragma unroll
    for (int it = 0; it < S::kBLoads; it++) {
        const int s = it * S::kGroupThreads + tid, row = (s >> 3) & 63, pc = s & 7;
        int col = (s >> 9) * 64 + ((pc ^ gemm_swz_b(row)) << 3);
        if (col > N - 8 - n0) col = N - 8 - n0;
        b_src[it] = ((Offset)row * (Offset)N + col) * 2;
    }
    auto load = [&](const bf16* base, Offset off, char* dst) {
        if constexpr (WIDE) load_global_to_lds16_untracked((const char*)base + off, dst);
        else load_global_to_lds16_sbase_untracked(base, off, dst);
    };
    auto issue_stage = [&](int step, int stage_off) {
        char* base = ring + stage_off + wave * 1024;
        const int k0 = step * S::kTileK;
        if (__builtin_expect(k0 <= K - S::kTileK, 1)) {
            const bf16* a = a_tile + k0;
            const bf16* b = b_tile + (size_t)k0 * N;
#pragma unroll
            for (int it = 0; it < S::kALoads; it++)
                load(a, a_src[it], base + it * (S::kGroupThreads * 16));
#pragma unroll
            for (int it = 0; it < S::kBLoads; it++)
                load(b, b_src[it], base + S::kABytes + it * (S::kGroupThreads * 16));
        } else {
            const int left = K - k0;            // <= 0: a step of a K share that the others have and this one has not
            const int at = left > 0 ? k0 : 0;   // (no address past the matrices is formed)
            const char* a = (const char*)(a_tile + at);
            const char* b = (const char*)(b_tile + (size_t)at * N);
#pragma unroll
            for (int it = 0; it < S::kALoads; it++) {
                const int s = it * S::kGroupThreads + tid;
                const int k = ((s & 7) ^ gemm_swz_a(s >> 3)) << 3;
                load_global_to_lds16_untracked(k < left ? a + a_src[it] : (const char*)g_gemm_zero, base + it * (S::kGroupThreads * 16));
            }
#pragma unroll
            for (int it = 0; it < S::kBLoads; it++) {
                const int row = ((it * S::kGroupThreads + tid) >> 3) & 63;
                load_global_to_lds16_untracked(row < left ? b + b_src[it] : (const char*)g_gemm_zero,
                                               base + S::kABytes + it * (S::kGroupThreads * 16));
            }
        }
    };

    // ---- per-lane LDS read offsets
    // A fragment (second MFMA operand: lane <-> row of A, k = 8 * quad ..+7): row 16a + l16, logical chunk 4 * half + quad
    const int a_lane = (wm * S::kPartM + l16) * 128 + ((quad ^ gemm_swz_a(l16)) << 4);
    // B fragment (first MFMA operand: lane <-> column of B, same k) through transposing reads: lane j of a
    // quad addresses k row 8 * quad + j / 4 (second read: +4), columns 4 * (j % 4) of a 16-column block
    const int b_row = 8 * quad + (l16 >> 2);
    const int b_lane = S::kABytes + b_row * 128 + ((((l16 & 3) >> 1) ^ gemm_swz_b(b_row)) << 4) + ((l16 & 1) << 3);

    f32x4 acc[NB][MB];
#pragma unroll
    for (int b = 0; b < NB; b++)
#pragma unroll
        for (int a = 0; a < MB; a++) acc[b][a] = f32x4{0.f, 0.f, 0.f, 0.f};

    bf16x8 af[2][MB], bfr[2][NB];       // two sets of fragments: one being multiplied, one being read
    auto read_a = [&](int set, const char* stage, int half, int a) __attribute__((always_inline)) {
        af[set][a] = lds_read_b128(stage, (a_lane ^ (half << 6)) + a * 16 * 128);
    };
    auto read_b = [&](int set, const char* stage, int half, int b) __attribute__((always_inline)) {
        const int block = wn * NB + b;          // 16-column block of the tile
        const int off = (block >> 2) * 8192 + half * 32 * 128, x = b_lane ^ ((block & 3) << 5);
        bfr[set][b] = concat(lds_read_tr16(stage, x + off), lds_read_tr16(stage, x + off + 4 * 128));
    };
    // One half step: the products of a set of fragments, and between them the reads of the other set and the loads of a whole
    // stage.  Issued in one go behind the barrier, the loads of all waves (64 KB a step with 256x256 tiles, of which a compute
    // unit takes 64 bytes a cycle) held every wave up until they were through, and its MFMAs with it.  Spread over the half, us before
    // and after (random data, the same tile): 8192^3 789, 760; M1000 N6144 K2048 28.7, 26.4; 2048^2 K8192 68.3, 60.5; M64 N512 K8192 in
    // 64x128 tiles 47.3, 34.4.  The reads are done by the middle, ahead of the wait for them at the barrier (192x256 tiles, M3564 N2344
    // K8696: 145, spread over the whole half 161).  Half steps of 32 MFMAs, whose two stages leave the loads
    // less than a step to arrive, have theirs issued in the first three quarters (8192^3 776, 760; shorter ones lose by it).
    auto half_step = [&](auto loads, auto set_, const char* stage, int half, const bf16* a_from, const bf16* b_from, char* to) __attribute__((always_inline)) {
        constexpr int set = decltype(set_)::value;
        constexpr int kMfmas = MB * NB, kReads = MB + NB, kLoads = decltype(loads)::value ? S::kLoads : 0;
        constexpr int kLoadSpan = kMfmas >= 32 ? kMfmas * 3 / 4 : kMfmas;
        int r = 0, l = 0;
#pragma unroll
        for (int m = 0; m < kMfmas; m++) {
#pragma unroll
            for (; l * kLoadSpan < (m + 1) * kLoads && l < kLoads; l++) {
                if (l < S::kALoads) load(a_from, a_src[l], to + l * (S::kGroupThreads * 16));
                else load(b_from, b_src[l - S::kALoads], to + S::kABytes + (l - S::kALoads) * (S::kGroupThreads * 16));
            }
#pragma unroll
            for (; r * kMfmas < 2 * (m + 1) * kReads && r < kReads; r++) {
                if (r < MB) read_a(set ^ 1, stage, half, r); else read_b(set ^ 1, stage, half, r - MB);
            }
            const int b = m / MB, a = m % MB;
            acc[b][a] = mfma16(bfr[set][b], af[set][a], acc[b][a]);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    const int steps_all = (K + S::kTileK - 1) / S::kTileK;
    const int n_steps = (steps_all + KS - 1) / KS;      // of every group (the last one of some may lie past K)
#pragma unroll
    for (int s = 0; s < S::kStages; s++)
        if (s < n_steps) issue_stage(s * KS + kg, s * S::kStageBytes);
    if (n_steps >= S::kStages) wait_vmcnt<(S::kStages - 1) * S::kLoads>(); else wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int a = 0; a < MB; a++) read_a(0, ring, 0, a);
#pragma unroll
    for (int b = 0; b < NB; b++) read_b(0, ring, 0, b);

    int stage = 0;
    auto next_stage = [&]() { return stage + S::kStageBytes == S::kStages * S::kStageBytes ? 0 : stage + S::kStageBytes; };
    // Between the halves of a step: every wave's last reads of its stage have completed, so it can be refilled; the next
    // step's stage (issued kStages - 1 steps ago) must have landed, the newer ones stay in flight.
    int s = 0;
    const int in_range = K / S::kTileK;                 // steps that lie within K
    int n_full = (in_range - kg + KS - 1) / KS - S::kStages;    // steps of this group whose refill lies within K
    if (n_full > n_steps - S::kStages) n_full = n_steps - S::kStages;
#pragma unroll 1
    for (; s < n_full; s++) {
        const int old = stage, next = ((s + S::kStages) * KS + kg) * S::kTileK;
        half_step(std::false_type{}, std::integral_constant<int, 0>{}, ring + stage, 1, nullptr, nullptr, nullptr);
        stage = next_stage();
        wait_vmcnt_lds_done<(S::kStages - 2) * S::kLoads>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        half_step(std::true_type{}, std::integral_constant<int, 1>{}, ring + stage, 0, a_tile + next, b_tile + (size_t)next * N, ring + old + wave * 1024);
    }
#pragma unroll 1
    for (; s < n_steps; s++) {
        const int old = stage;
        half_step(std::false_type{}, std::integral_constant<int, 0>{}, ring + stage, 1, nullptr, nullptr, nullptr);
        stage = next_stage();
        if (s + S::kStages <= n_steps) wait_vmcnt_lds_done<(S::kStages - 2) * S::kLoads>(); else wait_vmcnt_lds_done<0>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if (s + S::kStages < n_steps) issue_stage((s + S::kStages) * KS + kg, old);
        __builtin_amdgcn_sched_barrier(0);
        // (after the last step: fragments of a stage nobody writes, which nobody uses)
        half_step(std::false_type{}, std::integral_constant<int, 1>{}, ring + stage, 0, nullptr, nullptr, nullptr);
    }

    if constexpr (KS > 1) {
        wait_vmcnt_lds_done<0>();
        __builtin_amdgcn_s_barrier();
        // partial sums of the groups 1.. : [group][wave][block][lane] x 16 bytes
        char* part = lds + wave * (NB * MB * 1024) + lane * 16;
        if (kg > 0) {
#pragma unroll
            for (int b = 0; b < NB; b++)
#pragma unroll
                for (int a = 0; a < MB; a++)
                    *(f32x4*)(part + (kg - 1) * (S::kTileM * S::kTileN * 4) + (b * MB + a) * 1024) = acc[b][a];
        }
        __syncthreads();
        if (kg > 0) return;
#pragma unroll
        for (int g = 0; g < KS - 1; g++)
#pragma unroll
            for (int b = 0; b < NB; b++)
#pragma unroll
                for (int a = 0; a < MB; a++)
                    acc[b][a] += *(const f32x4*)(part + g * (S::kTileM * S::kTileN * 4) + (b * MB + a) * 1024);
    }

    // ---- epilogue: lane <-> row of C; registers of block (b, a) <-> columns 16b + 4 * quad ..+3 (N is a multiple of 8)
#pragma unroll
    for (int a = 0; a < MB; a++) {
        const size_t row = (size_t)m0 + wm * S::kPartM + 16 * a + l16;
        if (row >= (size_t)M) continue;
        bf16* crow = C + row * N;
#pragma unroll
        for (int b = 0; b < NB; b++) {
            const size_t col = (size_t)n0 + wn * S::kPartN + 16 * b + 4 * quad;
            if (col >= (size_t)N) continue;
            *(bf16x4*)(crow + col) = __builtin_shufflevector(cvt2(acc[b][a][0], acc[b][a][1]), cvt2(acc[b][a][2], acc[b][a][3]), 0, 1, 2, 3);
        }
    }
}

template <int TM, int TN, int WM, int WN, int KS, int STAGES, int WAVES_PER_SIMD, bool WIDE = false>
static hipError_t launch_tile(const void* a, const void* b, void* c, int M, int N, int K, hipStream_t stream)
{
    using S = GemmTile<TM, TN, WM, WN, KS, STAGES>;
    const int tiles_m = (M + TM - 1) / TM, tiles_n = (N + TN - 1) / TN;
    constexpr int super_m = TM >= 256 ? 4 : TM >= 128 ? 8 : 16;     // tile rows walked together
    hipLaunchKernelGGL((gemm_kernel<S, WM, WN, KS, WAVES_PER_SIMD, WIDE>), dim3(tiles_m * tiles_n), dim3(S::kThreads), 0, stream,
                       (const bf16*)a, (const bf16*)b, (bf16*)c, M, N, K, tiles_m, tiles_n, super_m);
    return hipGetLastError();
}

// The tile shapes, what their steps cost on MI355X, and the choice between them.  Beside a launch, the same for all, a call
// takes about
//   (tiles on the busiest of the compute units) * (steps of a tile / KS) * us per step,
// and the shape with the smallest product is taken.  Us per 64-wide k step of one tile (one tile on a unit / several of them after or
// next to each other), fitted to 900 sizes of up to 10000 a side for which every shape was timed: the choice takes 1.8 % more than the
// best shape, on average over the sizes of 5 us and more.  8192^3 with each:
//   256x256  8 waves   1.40 / 1.485   0.76 ms (1.45 PFLOP/s; least L2 and LDS traffic per flop)
//   192x256  8 waves   1.15 / 1.25    0.91 ms       64x128  4 waves  0.42 / 0.34   1.37 ms
//   128x256  8 waves   0.88 / 0.93    0.87 ms       64x64   4 waves  0.228 / 0.24  2.5 ms (L2 bound: 16 KB per 0.5 MFLOP)
//   256x128  8 waves   0.87 / 0.92    0.86 ms       64x64  K split in 2:  0.446 / 0.53 per two steps
//   128x192  8 waves   0.645 / 0.846  0.99 ms       32x64  K split in 4:  0.60 / 0.75 per four steps
//   128x128  8 waves   0.454 / 0.56   1.15 ms
//   128x128  4 waves, two workgroups per compute unit: 0.68 alone, 1.09 for two   1.00 ms
// (A single 256x256 tile with four waves of 128x128, one per SIMD, took 0.96 ms: nothing filled the gaps of a
// wave.  Two waves per SIMD and 16x16x32 MFMAs, which move half the accumulator bits per flop of the 32x32x16 form, do.
// 32x64 with K split in 2 would be chosen for 65 to 128 k only, where it gains nothing: 3.7 us either way, the launch.)
// The last three have 64-bit lane offsets and are only considered where a shape of the same rows needs them (128x256 with
// four waves: few enough threads for the widest N): M1 N34200008 K72 1.76 ms, M250 N34500008 K64 7.0, M300 N35000000 K128
// 15.1, M32 N8 K69400008 456.  Their figures are those of a loop that issued a stage's loads in one go.  They stay: such calls are
// bound by B and C, and of 14 with N = 34600000 and up to 233 rows none has a shape that takes over 1.2 % less than the chosen one.
struct GemmChoice {
    hipError_t (*launch)(const void*, const void*, void*, int, int, int, hipStream_t);
    int threads, tile_m, tile_n, ks;
    float one, more;        // us per step: the only tile of a compute unit; every tile of several
    bool wide;              // 64-bit lane offsets
};
static const GemmChoice kGemmChoices[] = {
    {launch_tile<256, 256, 2, 4, 1, 2, 2>, 512, 256, 256, 1, 1.40f, 1.485f, false},
    {launch_tile<192, 256, 2, 4, 1, 2, 2>, 512, 192, 256, 1, 1.15f, 1.25f, false},
    {launch_tile<256, 128, 4, 2, 1, 3, 2>, 512, 256, 128, 1, 0.87f, 0.92f, false},
    {launch_tile<128, 256, 2, 4, 1, 3, 2>, 512, 128, 256, 1, 0.88f, 0.93f, false},
    {launch_tile<128, 192, 2, 4, 1, 3, 2>, 512, 128, 192, 1, 0.645f, 0.846f, false},
    {launch_tile<128, 128, 2, 4, 1, 4, 2>, 512, 128, 128, 1, 0.454f, 0.56f, false},
    {launch_tile<128, 128, 2, 2, 1, 2, 2>, 256, 128, 128, 1, 0.68f, 0.547f, false},
    {launch_tile<64, 128, 2, 2, 1, 3, 2>, 256, 64, 128, 1, 0.42f, 0.34f, false},
    {launch_tile<64, 64, 2, 2, 1, 3, 2>, 256, 64, 64, 1, 0.228f, 0.24f, false},
    {launch_tile<64, 64, 2, 2, 2, 3, 2>, 512, 64, 64, 2, 0.446f, 0.53f, false},
    {launch_tile<32, 64, 1, 4, 4, 3, 4>, 1024, 32, 64, 4, 0.60f, 0.75f, false},
    {launch_tile<256, 256, 2, 4, 1, 2, 2, true>, 512, 256, 256, 1, 1.50f, 1.57f, true},
    {launch_tile<128, 256, 2, 2, 1, 3, 1, true>, 256, 128, 256, 1, 1.01f, 1.02f, true},
    {launch_tile<64, 128, 2, 2, 1, 3, 2, true>, 256, 64, 128, 1, 0.42f, 0.34f, true},
};

// Whether every lane offset within a tile of tile_m rows is below 4 GiB: the last row of A that the tile fetches, and the
// last of the up to 64 rows of B in a step.  (A: from K = 8.4 million with 256 rows; B: from N = 34 million with K >= 64.)
static bool gemm_fits_32_bits(int tile_m, int M, int N, int K)
{
    const long long a_rows = tile_m < M ? tile_m : M, b_rows = K < 64 ? K : 64;
    return a_rows * K * 2 <= 0xffffffffLL && b_rows * N * 2 <= 0xffffffffLL;
}

hipError_t launch_gemm(const void* a, const void* b, void* c, int M, int N, int K, hipStream_t stream)
{
    int cus = 0;
    hipError_t e = compute_unit_count(&cus);
    if (e != hipSuccess) return e;
    const GemmChoice* best = nullptr;
    double best_us = 0;
    for (const GemmChoice& g : kGemmChoices) {
        const long long tiles = (((long long)M + g.tile_m - 1) / g.tile_m) * (((long long)N + g.tile_n - 1) / g.tile_n);
        if (tiles * g.threads > 0xffffffffLL) continue;                             // the threads of a launch are counted in 32 bits
        if (g.ks > 1 && K > 0x7fffffff - 64 * g.ks) continue;                       // (the steps of the last share would leave the range of an int)
        if (gemm_fits_32_bits(g.tile_m, M, N, K) == g.wide) continue;               // (wide: only where the offsets need it)
        const long long rounds = (tiles + cus - 1) / cus;
        const int steps = (K + 63) / 64, share = (steps + g.ks - 1) / g.ks;
        const double us = (double)share * (rounds == 1 ? g.one : (double)rounds * g.more);
        if (!best || us < best_us) { best = &g; best_us = us; }
    }
    return best ? best->launch(a, b, c, M, N, K, stream) : hipErrorInvalidValue;
}

}  // namespace tk
