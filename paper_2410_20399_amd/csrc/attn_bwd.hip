// Fused exact softmax attention, backward pass, for gfx950 (MI355X).
//
// The paper reports the backward kernel's speed only (the attention plots of Section 4.1 and the profile table of Section 4.2); the algorithm
// here is the chain rule with P recomputed from the saved log-sum-exp:
//
//   kernel 1  Delta_i = sum_d dO_id O_id          (HBM stream)
//   kernel 2  dK, dV: persistent workgroups walk the 128-key tiles (large launches at D = 128: 256-key tiles, 64 keys a wave); wave w owns keys 32w..32w+31 and keeps
//             their dK^T, dV^T accumulators in registers while it loops over 32-query blocks:
//               S  = Q_i K_j^T            P  = 2^(S*c - LSE_i*log2e)
//               dP = dO_i V_j^T           dS = P (dP - Delta_i)
//               dV_j^T += dO_i^T P        dK_j^T += Q_i^T dS
//   kernel 3  dQ: one workgroup per 128-query tile, wave w owns queries 32w..32w+31 and keeps
//             their dQ^T accumulator in registers while it loops over 64-key tiles:
//               S^T = K_j Q_i^T, dP^T = V_j dO_i^T, dS^T as above, dQ_i^T += K_j^T dS^T
//
// dQ gets a kernel of its own (recomputing S and dP) instead of fp32 atomics from kernel 2: the
// L2 atomic units retire about one fp32 lane per clock per channel (measured ~0.33 T lane-adds/s
// for the whole chip), and a 128-key tile needs N/128 partial sums per dQ element, which made
// the atomics alone as long as all the matrix work.  The split is also deterministic.
//
// With a large workspace (the chip has 288 GB) the recomputation goes away as well: kernel 2 then
// also stores its bf16 dS blocks, 2 bytes per (query, key) pair, exactly as its lanes hold them
// (SPILL), and dQ becomes one product per pair,
//   kernel 4  dQ_i = scale * sum_j dS_ij K_j  from the stored blocks (attn_bwd_dq_from_ds_kernel),
// which is bound by reading dS back from HBM instead of by 6*D flops per pair.  10*D flops per
// pair are executed instead of 14*D; Delta then comes from kernel 1.
//
// In kernel 2, S and dP are produced with the KEY index on lanes and the query index on
// registers, so P and dS in accumulator layout are directly the B operands of the two products
// contracted over queries; their A operands (dO^T, Q^T) come from row-major LDS tiles via
// transposing reads.  Kernel 3 mirrors the forward kernel: QUERY index on lanes, so LSE_i and
// Delta_i are lane scalars and dS^T is directly the B operand of the product contracted over keys.
#include "tk_common.h"
#include "tk_launch.h"

#include <type_traits>

namespace tk {

// ------------------------------------------------------------------------------------------
// kernel 1: Delta
// ------------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256)
void attn_bwd_delta_kernel(const bf16* __restrict__ O, const bf16* __restrict__ dO,
                           float* __restrict__ delta, size_t n_chunks)
{
    constexpr int kLanesPerRow = D / 8;
    const size_t chunk = (size_t)blockIdx.x * 256 + threadIdx.x;   // one 8-element chunk per thread
    if (chunk >= n_chunks) return;                                  // (whole rows: n_chunks is a multiple of D/8)
    bf16x8 a = *(const bf16x8*)(O + chunk * 8);
    bf16x8 b = *(const bf16x8*)(dO + chunk * 8);
    float acc = 0.f;
#pragma unroll
    for (int e = 0; e < 8; e++) acc = __builtin_fmaf((float)a[e], (float)b[e], acc);
#pragma unroll
    for (int off = kLanesPerRow / 2; off >= 1; off >>= 1) acc += __shfl_xor(acc, off);
    if ((threadIdx.x & (kLanesPerRow - 1)) == 0) delta[chunk / kLanesPerRow] = acc;
}

hipError_t launch_attn_bwd_delta(const void* o, const void* d_o, float* delta,
                                 int B, int H, int N, int D, hipStream_t stream)
{
    const size_t n_chunks = (size_t)B * H * N * D / 8;
    const dim3 grid((unsigned)((n_chunks + 255) / 256));
    if (D == 128) hipLaunchKernelGGL((attn_bwd_delta_kernel<128>), grid, dim3(256), 0, stream, (const bf16*)o, (const bf16*)d_o, delta, n_chunks);
    else          hipLaunchKernelGGL((attn_bwd_delta_kernel<64>), grid, dim3(256), 0, stream, (const bf16*)o, (const bf16*)d_o, delta, n_chunks);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// kernel 2: dK, dV
// ------------------------------------------------------------------------------------------
// LSE stand-in for query rows past the end of a sequence: P = 2^(s - inf) = 0 for them.
__device__ float g_lse_pad[1] = {INFINITY};

// The scores are formed as scale * (S - LSE / scale), and LSE / scale has to stay finite: where the scale is smaller than this, K
// is taken 2^64 times smaller and the scale larger.  (What that takes from elements of K below 2^-62 is less than 2^-53 of a
// score: Q is below 2^128, the scale below 2^-119.)
constexpr float kLeastScale = 1e-36f;
__device__ __forceinline__ void shrink_k(bf16x8& k) {
#pragma unroll
    for (int i = 0; i < 8; i++) k[i] = (bf16)((float)k[i] * 0x1p-64f);
}

template <int D>
struct DkdvShape {
    static constexpr int kWaves = 4;
    static constexpr int kThreads = 256;
    static constexpr int kTileKV = 128;                 // keys per workgroup (32 per wave)
    static constexpr int kTileQ = 32;                   // queries per loop iteration
    // LDS ring of query blocks.  D = 64: four stages, filled three blocks ahead.  D = 128 (the pipelined
    // step, see the kernel): seven stages, six of them filled at the start; step n then fetches block n + 6
    // into the stage of block n - 1, which nobody reads any more.
    static constexpr bool kPipe = (D == 128);
    static constexpr int kStages = kPipe ? 7 : 4;
    static constexpr int kAhead = kStages - 1;
    static constexpr int kRowBytes = D * 2;
    static constexpr int kChunksPerRow = D / 8;
    static constexpr int kQTileBytes = kTileQ * kRowBytes;
    static constexpr int kStageBytes = 2 * kQTileBytes + kWaves * 256;     // Q, dO, and for each wave LSE[32], Delta[32]; a multiple of 256
    static constexpr int kQLoads = kTileQ * kChunksPerRow / kThreads;   // per thread, per tensor
    static constexpr int kLoadsPerBlock = 2 * kQLoads;  // per thread, of Q and dO rows (one more load fetches the statistics)
    static constexpr int kEpiPitch = kRowBytes + 8;     // row pitch of the epilogue staging tile: the odd multiple of 8 bytes spreads
                                                        // both the 8-byte column-piece writes and the row reads over the banks
};

// Chunk swizzle of every row-major bf16 tile in the backward kernels (rows of D elements): spreads
// both a 16-row same-chunk read (MFMA operand rows) and a 4-row x 64-byte transposing read over
// the banks.
template <int D> __device__ __forceinline__ int swz(int row) {
    return D == 128 ? (((row & 3) << 2) | ((row >> 2) & 3)) : ((((row >> 1) & 1) << 2) | ((row >> 2) & 3));
}

// At D = 128: one wave per SIMD (the dK^T, dV^T accumulators and the K, V fragments take 192
// registers), so nothing hides LDS latency or fills the vector ALU but the schedule itself: the
// pipelined step described inside the kernel, with the query blocks arriving by direct global->LDS
// loads issued six blocks ahead into a seven-stage ring.
// At D = 64 the registers allow two workgroups per compute unit, i.e. two waves per SIMD that fill
// each other's gaps (the vector work per MFMA is twice that of D = 128 there), and the phases of a
// block run one after the other, every MFMA operand read one phase ahead of its use:
//     phase 1  S, dP MFMAs from row fragments already in registers; meanwhile the transposed
//              fragments (dO^T, Q^T) of THIS block are read from LDS
//     phase 2  P, dS on the vector ALU
//     phase 3  dV^T, dK^T MFMAs from the transposed fragments; meanwhile the row fragments and the
//              statistics of the NEXT block are read from LDS
// with the query blocks issued three blocks ahead into a four-stage ring.
// (The statistics as starting values of the accumulators, S and dP in two sets of vector registers instead of one that is copied
// out of accumulator registers, and no wait for the wave's LDS reads before a step's barrier, us before and after, B16 H16 N4096
// causal: D128 2170, 2030, storing dS 2520, 2385, D64 1135, 1070.)
//
// Nothing hides a workgroup's start-up and wind-down either, so the launch is persistent: the
// resident workgroups (one per compute unit, two at D = 64) walk the key tiles v = blockIdx.x, blockIdx.x + stride, ... and
// the query-block stream never stops: the loads issued during the last blocks of one key tile
// already fetch the first blocks of the next, and the next tile's K, V fragments are requested
// before the current tile's results are stored.
// Nq queries, Nk keys.  TAIL: the general case (Nq != Nk, or a length that is not a multiple of
// 128); the aligned square case compiles without any of the tail code.  Causal: query i sees keys
// j <= i + (Nk - Nq), Nq <= Nk.
//
// SPILL: every 32-key x 32-query block of dS is also written to DS as the wave holds it after the
// conversion to bf16: 2 KB per block, [2 halves][64 lanes][16 bytes], where lane (key k = lane % 32,
// h = lane / 32) holds in half s the queries 16s + 8g + 4h + t (g = 0..1, t = 0..3) of the block, at
// element 4g + t.  Block (query head, key tile kt, query block qb, wave w) sits at
// (((head * num_kv_tiles + kt) * n_qb + qb) * 4 + w) * 2048 bytes.  Masked pairs and padding rows hold 0.
//
// SPLIT (implies TAIL): the queries are dealt to n_splits workgroups - the query heads of a group to
// n_splits / q_splits and, without a mask, the blocks of a head to q_splits - each of which leaves fp32
// sums over its own in Part ([n_splits][2: dK, dV][B * hkv][Nk][D], unscaled) for attn_bwd_dkdv_sum_kernel.
// For launches with fewer units than compute units: a unit's time is the length of its query stream, 1 us a
// block of 32 queries, whether the other compute units are idle or not.
//
// stride: the number of workgroups.  (Asked of gridDim, it lay in a third cache line of the arguments, 0.3 us of every launch.)
template <int D, bool CAUSAL, bool TAIL, bool SPILL, bool SPLIT>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1)
void attn_bwd_dkdv_kernel(const bf16* __restrict__ Q, const bf16* __restrict__ K, const bf16* __restrict__ V,
                          const bf16* __restrict__ dO, const float* __restrict__ LSE, const float* __restrict__ Delta,
                          bf16* __restrict__ dK, bf16* __restrict__ dV,
                          int Nq, int Nk, int num_kv_tiles, int total_units, float scale, int hq, int hkv, int stride,
                          char* __restrict__ DS, int n_qb, int units, int n_splits, int q_splits,
                          float* __restrict__ Part)
{
    using S = DkdvShape<D>;
    __shared__ __attribute__((aligned(1024))) char ring[S::kStages * S::kStageBytes];
    __shared__ __attribute__((aligned(16))) char epi[S::kWaves * 32 * S::kEpiPitch];   // per-wave staging of the dK / dV tile

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int l32 = lane & 31;
    const int h = lane >> 5;
    const int j16 = lane & 15;
    const int ghalf = (lane >> 4) & 1;
    const float score_scale = scale < kLeastScale ? scale * 0x1p64f : scale;     // (see shrink_k)
    const float c = score_scale * kLog2e;

    // Work unit: one key tile, or, when causal, the pair (u, last - u): tile u loops over the
    // query blocks from its diagonal on, so the pairs carry (nearly) the same work and the static
    // schedule is balanced.  (Not paired where every tile can have a workgroup of its own, see pair_tiles().)  A "pass" is
    // one key tile; (vu, half) names the pass `half` of unit vu.  `units` per key/value head come from the host: formed here
    // from a flag, they cost the masked step of the D = 64 kernel a wait in the middle (32 masked blocks 29.1, 31.0 us).
    // Grouped-query attention: a key/value head is shared by `group` consecutive query heads, and a
    // pass streams the query blocks of all of them, one head after the other, into the same dK, dV
    // accumulators.  bh below counts key/value heads.
    const int heads_per_kv = hq / hkv;
    const int group = SPLIT ? heads_per_kv / (n_splits / q_splits) : heads_per_kv;      // query heads of a pass
    auto q_head_row = [&](int bh, int split) {         // first row of the first query head of a pass of key/value head bh
        return (size_t)((bh / hkv) * hq + (bh % hkv) * heads_per_kv + (SPLIT ? split / q_splits * group : 0)) * Nq;
    };
    // The query blocks of a pass: blocks of 32 rows from pass_ibegin(kt) on, per query head of the
    // group; an even count (the loops below take two blocks per trip), of which the first
    // `n_masked` may touch the diagonal.  General case: the first query that sees a key of the tile
    // is j0 - off, rounded down to a block boundary; rows past Nq are padding.
    const int off = TAIL ? Nk - Nq : 0;
    const int q_chunk = SPLIT && !CAUSAL ? dkdv_q_chunk(Nq, q_splits) : 0;      // blocks of a head in one split
    auto pass_ibegin = [&](int kt, int split) {
        if (SPLIT && !CAUSAL) return split % q_splits * q_chunk * S::kTileQ;
        if (!CAUSAL) return 0;
        if (!TAIL) return kt * S::kTileKV;
        const int first = kt * S::kTileKV - off;
        return first > 0 ? first & ~(S::kTileQ - 1) : 0;
    };
    auto pass_nblocks = [&](int ibegin) {
        const int n = TAIL ? 2 * ((Nq - ibegin + 2 * S::kTileQ - 1) / (2 * S::kTileQ)) : (Nq - ibegin) / S::kTileQ;
        return SPLIT && !CAUSAL && n > q_chunk ? q_chunk : n;
    };
    auto pass_tile = [&](int vu, int half, int& bh, int& kt, int& split) {
        const int logical = xcd_remap(vu, total_units);
        bh = logical / units;
        const int unit = logical % units;
        split = 0;
        if (SPLIT) { split = bh % n_splits; bh /= n_splits; }      // (the units of a split, which read the same queries, are neighbours)
        kt = half == 0 ? unit : num_kv_tiles - 1 - unit;
    };
    // the pass after (vu, half) in this workgroup's walk; vu >= total_units means "none"
    auto next_pass = [&](int& vu, int& half) {
        if (CAUSAL && half == 0) {
            const int unit = xcd_remap(vu, total_units) % units;
            if (num_kv_tiles - 1 - unit >= units) { half = 1; return; }   // (not paired, or the middle one of an odd count: no partner)
        }
        vu += stride;
        half = 0;
    };

    // ---- query-block prefetch: Q, dO rows (swizzled), LSE and Delta of 32 queries
    int q_src[S::kQLoads];
#pragma unroll
    for (int it = 0; it < S::kQLoads; it++) {
        int s = it * S::kThreads + tid;
        int row = s / S::kChunksPerRow, pc = s % S::kChunksPerRow;
        q_src[it] = row * D + ((pc ^ swz<D>(row)) * 8);
    }
    // Producer side of the ring: a cursor over the query blocks of this workgroup's passes, in the
    // order the passes consume them.  Every call issues the same number of loads in every wave (the
    // vmcnt waits below count them); once the walk is exhausted it fetches one block again and again
    // into stages nobody reads.
    // The lengths need not be multiples of the tile sizes: the kernel works on padded sequences.
    // Reads of rows past the end are redirected to the last row; a query row >= Nq gets LSE = +inf,
    // so its P and dS are exactly 0; key rows >= Nk are computed like any other and not stored.
    const float* const stat_src = (lane < 32 ? LSE : Delta) + l32;
    int p_vu = blockIdx.x, p_half = 0, p_nblocks = 0, p_g = 0, p_ibegin = 0;
    size_t p_head_row = 0;                  // first row of the group's first query head of the producer's pass
    size_t p_row = 0;                       // first row of the next block to fetch (rows of all heads counted through)
    int p_i0 = 0;                           // ... and its first query within its head
    int p_left = 0;                         // blocks left in the current head's run, this one included
    int p_advance = S::kTileQ;              // rows from one block to the next (0 once the walk is exhausted)
    int p_stage = 0;                        // byte offset of the ring stage the next block goes to
    auto next_stage = [&](int off) { return off + S::kStageBytes == S::kStages * S::kStageBytes ? 0 : off + S::kStageBytes; };
    auto producer_head = [&]() __attribute__((always_inline)) {            // the cursor at the first block of query head p_g of the pass
        p_row = p_head_row + (size_t)p_g * Nq + p_ibegin;
        p_i0 = p_ibegin;
        p_left = p_nblocks;
    };
    auto producer_open = [&]() __attribute__((always_inline)) {            // set the cursor to the first block of pass (p_vu, p_half)
        int bh, kt, split;
        pass_tile(p_vu, p_half, bh, kt, split);
        p_ibegin = pass_ibegin(kt, split);
        p_head_row = q_head_row(bh, split);
        p_nblocks = pass_nblocks(p_ibegin);
        p_g = 0;
        producer_head();
    };
    // the end of a head's run: rare, so that the steady state of prepare() below is straight-line scalar code
    auto producer_turn = [&]() __attribute__((always_inline)) {
        if (++p_g < group) { producer_head(); return; }
        next_pass(p_vu, p_half);
        if (p_vu < total_units) { producer_open(); return; }
        p_row -= p_advance;                 // exhausted: stay on the last block
        p_i0 -= p_advance;
        p_advance = 0;
        p_left = 0x7fffffff;
    };
    // A block's fetch is split into prepare() (the cursor: scalar work, one rare branch) and its loads,
    // emit(0 .. kLoadsPerBlock): the pipelined step spreads the loads over its matrix instructions, because
    // the compute unit's address unit takes one 16-byte-per-lane instruction every ~16 cycles and a wave
    // that issues several in a row stalls on it.
    size_t e_head_row = 0, e_row = 0;       // of the block being fetched: first row of its head; its own first row
    int e_i0 = 0, e_stage = 0;              // its first query within the head; byte offset of its ring stage
    auto prepare = [&]() __attribute__((always_inline)) {
        e_row = p_row;
        e_i0 = p_i0;
        e_head_row = p_row - p_i0;
        e_stage = p_stage;
        p_stage = next_stage(p_stage);
        p_row += p_advance;
        p_i0 += p_advance;
        --p_left;
    };
    // (kept apart from prepare(): the pipelined step calls prepare() in the middle of a long basic block,
    // which this branch would split)
    auto prepare_turn = [&]() __attribute__((always_inline)) {
        if (__builtin_expect(p_left == 0, 0)) producer_turn();
    };
    auto emit = [&](int which) {
        char* base = ring + e_stage;
        if (which < S::kLoadsPerBlock) {        // Q rows, then dO rows
            const int it = which % S::kQLoads;
            const bf16* block = (which < S::kQLoads ? Q : dO) + e_row * D;      // wave-uniform
            char* dst = base + (which < S::kQLoads ? 0 : S::kQTileBytes) + it * (S::kThreads * 16) + wave * 1024;
            if (TAIL) {
                // a block that runs past the last query: rows >= Nq fetch row Nq-1 instead
                const int r = e_i0 + (it * S::kThreads + tid) / S::kChunksPerRow;
                load_global_to_lds16_untracked(block + q_src[it] - (r < Nq ? 0 : r - (Nq - 1)) * D, dst);
            } else {
                load_global_to_lds16_sbase_untracked(block, (uint32_t)q_src[it] * 2, dst);
            }
        } else {
            // The statistics: every wave fetches a copy of its own (a branch on the wave number costs every wave a
            // restart of its instruction stream, and the waits would have to count differently per wave):
            // lanes 0..31 LSE of the block's 32 queries, lanes 32..63 their Delta
            const float* src = stat_src + e_row;
            if (TAIL && e_i0 + l32 >= Nq) src = lane < 32 ? g_lse_pad : Delta + e_head_row + (Nq - 1);
            load_global_to_lds4_untracked(src, base + 2 * S::kQTileBytes + wave * 256);
        }
    };
    auto issue_next = [&]() {
        prepare();
#pragma unroll
        for (int which = 0; which <= S::kLoadsPerBlock; which++) emit(which);
        prepare_turn();
    };

    // A wave turns its copy of a block's statistics, once they are here, into -LSE / scale and -Delta.  The accumulators of S
    // and dP start from these, so that scale * S - LSE takes the vector ALU one multiplication and dP - Delta nothing.
    // (Three instructions a block instead of two more for each of a lane's 16 scores.)
    const float stat_mul = lane < 32 ? -1.0f / score_scale : -1.0f;
    auto wave_stat = [&](int stage) { return (float*)(ring + stage + 2 * S::kQTileBytes + wave * 256); };
    auto scale_stat = [&](int stage) { float* st = wave_stat(stage) + lane; *st = *st * stat_mul; };

    // ---- per-lane LDS offsets
    // row operand (A of S and dP): row l32, logical chunk 2*kb + h
    const int row_lane = l32 * S::kRowBytes + ((h ^ swz<D>(l32)) << 4);
    // transposed operand from a 32-row Q/dO block (A of dV^T, dK^T): rows 16*ks + 4h + j16/4 (+8)
    const int trq_row = 4 * h + (j16 >> 2);
    const int trq_lane = trq_row * S::kRowBytes + (((2 * ghalf + ((j16 & 3) >> 1)) ^ swz<D>(trq_row)) << 4) + ((j16 & 1) << 3);

    constexpr int kSteps = D / 16;          // MFMA steps of S / dP; also 2 * (D/32) steps of dV^T / dK^T
    bf16x8 kf[D / 16], vf[D / 16];          // K, V fragments of this wave's 32 keys (B operands of S = Q K^T and dP = dO V^T)
    auto load_kv = [&](int bh, int kt) {
        const int key = kt * S::kTileKV + wave * 32 + l32;
        const size_t row = (size_t)bh * Nk + ((!TAIL || key < Nk) ? key : Nk - 1);
#pragma unroll
        for (int kb = 0; kb < D / 16; kb++) {
            kf[kb] = *(const bf16x8*)(K + row * D + kb * 16 + h * 8);
            vf[kb] = *(const bf16x8*)(V + row * D + kb * 16 + h * 8);
        }
    };

    int c_vu = blockIdx.x, c_half = 0;      // consumer side: the pass being computed (the grid never exceeds the unit count)
    int c_stage = 0;                        // byte offset of the ring stage of the next block to consume ...
    int c_stage1 = S::kStageBytes, c_stage2 = 2 * S::kStageBytes;      // ... and of the two blocks after it (D = 128)
    bool first_pass = true;
    {
        int bh, kt, split;
        pass_tile(c_vu, c_half, bh, kt, split);
        producer_open();
#pragma unroll
        for (int b = 0; b < S::kAhead; b++) issue_next();
        load_kv(bh, kt);
    }

#pragma unroll 1
    while (c_vu < total_units) {
    int bh, kt, split;
    pass_tile(c_vu, c_half, bh, kt, split);
    const size_t head = (size_t)bh * Nk * D;       // of the key/value head
    const int j0 = kt * S::kTileKV;
    const int jw0 = j0 + wave * 32;                // first key of this wave
    const int my_j = jw0 + l32;
    const int i_begin = pass_ibegin(kt, split);
    const int n_blocks = pass_nblocks(i_begin);           // per query head of the group
    // blocks that may hold a masked (query, key) pair: rows below j0 + 127 - off, i.e. four blocks
    // from i_begin when that is the tile's own first row, up to five when off is not a multiple of 32
    const int n_masked = !CAUSAL ? 0 : !TAIL ? 4 : (n_blocks < 6 ? n_blocks : 6);

    f32x16 dk_acc[D / 32], dv_acc[D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; db++)
#pragma unroll
        for (int r = 0; r < 16; r++) { dk_acc[db][r] = 0.f; dv_acc[db][r] = 0.f; }

    if (__builtin_expect(scale < kLeastScale, 0)) {
#pragma unroll
        for (int kb = 0; kb < D / 16; kb++) shrink_k(kf[kb]);
    }
    // Every global load so far (this pass's K, V fragments, its first blocks, the previous pass's
    // stores) completes here.  The empty asm statements pin the fragment loads above this point (the
    // compiler would otherwise sink them to their first use inside the loop and wait for them there,
    // draining the prefetch every iteration): inside the loop the only waits on the vector memory
    // counter are the explicit ones, which leave the newest prefetches in flight.
#pragma unroll
    for (int kb = 0; kb < D / 16; kb++) {
        // (D = 128: into the accumulator half of the register file, from where the matrix instructions read
        // them just as well; that leaves the other half to the vector ALU's operands, the score blocks among them)
        if (S::kPipe) asm volatile("" : "+a"(kf[kb]), "+a"(vf[kb]));
        else asm volatile("" : "+v"(kf[kb]), "+v"(vf[kb]));
    }
    wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();           // the pass's first blocks landed and visible
    __builtin_amdgcn_sched_barrier(0);
    if (first_pass) {                       // (later passes: done by the steps before them)
        scale_stat(c_stage);
        if (S::kPipe) scale_stat(c_stage1);
        first_pass = false;
    }

    // register r of a score block <-> query i0 + 8*(r/4) + 4h + r%4, lane <-> key my_j
    const bool pad_key = TAIL && SPILL && my_j >= Nk;    // a padding key was computed from the last real row: its dS must not reach dQ
    auto q_head_of = [&](int g) { return (size_t)(bh / hkv) * hq + (size_t)(bh % hkv) * heads_per_kv + (SPLIT ? split / q_splits * group : 0) + g; };

    if constexpr (S::kPipe) {
    // ------------------------------------------------------------------------------------------
    // D = 128: one wave per SIMD.  A wave issues in order, at most one instruction every four cycles,
    // and a matrix instruction holds the matrix pipe for 32: with matrix instructions back to back the
    // wave idles until the pipe frees, and the ~150 vector instructions of a block then run with the
    // pipe idle.  So every matrix instruction here is followed by the handful of other instructions
    // that fit in its shadow, and the work of three consecutive blocks is in flight at once:
    //     step n, first half    S, dP of block n+1 (16 MFMAs)  next to  P, dS of block n (vector ALU) and
    //                           the transposing LDS reads of block n's Q^T, dO^T fragments
    //     step n, second half   dV^T, dK^T of block n (16 MFMAs)  next to  the LDS reads of the row fragments
    //                           and the statistics of block n+2, the dS stores and the prefetch
    // S and dP exist twice, for blocks with an even and an odd number: a step writes one set and reads the other.  The empty asm statements keep each group in program order: the compiler keeps them in
    // order with each other and with the scheduling barriers, and each one names a value that the
    // instructions of its group produce or consume.
    // ------------------------------------------------------------------------------------------
    bf16x8 rq[kSteps], rdo[kSteps];         // row fragments: operands of the next S, dP
    bf16x8 tq[kSteps], tdo[kSteps];         // transposed fragments [ks * (D/32) + db]: operands of the next dV^T, dK^T
    bf16x8 pb[2], dsb[2];                   // bf16 P, dS of the block in hand
    f32x16 s_even, dp_even, s_odd, dp_odd;  // S - LSE / scale, dP - Delta of blocks with an even and an odd number
    auto read_stat = [&](f32x16& acc, const float* stat, int g) {          // four of the values that an accumulator starts from
        const f32x4 x = ((const f32x4*)stat)[2 * g + h];
#pragma unroll
        for (int t = 0; t < 4; t++) acc[4 * g + t] = x[t];
    };

    auto read_rows = [&](const char* qs, int kb) {
        rq[kb] = lds_read_b128(qs, row_lane ^ ((2 * kb) << 4));
        rdo[kb] = lds_read_b128(qs + S::kQTileBytes, row_lane ^ ((2 * kb) << 4));
    };
    auto read_tq = [&](const char* qs, int idx) {
        const int ks = idx / (D / 32), db = idx % (D / 32);
        const int row_off = 16 * ks * S::kRowBytes;
        const int x0 = (4 * db) << 4, x1 = ((4 * db) ^ 2) << 4;
        tq[idx] = concat(lds_read_tr16(qs, (trq_lane ^ x0) + row_off),
                         lds_read_tr16(qs, (trq_lane ^ x1) + row_off + 8 * S::kRowBytes));
    };
    auto read_tdo = [&](const char* qs, int idx) {
        const int ks = idx / (D / 32), db = idx % (D / 32);
        const int row_off = 16 * ks * S::kRowBytes;
        const int x0 = (4 * db) << 4, x1 = ((4 * db) ^ 2) << 4;
        const char* dos = qs + S::kQTileBytes;
        tdo[idx] = concat(lds_read_tr16(dos, (trq_lane ^ x0) + row_off),
                          lds_read_tr16(dos, (trq_lane ^ x1) + row_off + 8 * S::kRowBytes));
    };
    // S, dP of the block whose row fragments are in rq / rdo; `between(kb, which)` runs after each MFMA
    auto scores = [&](f32x16& s_out, f32x16& dp_out, auto between) {
#pragma unroll
        for (int kb = 0; kb < kSteps; kb++) {
            asm volatile("" : "+v"(s_out));
            s_out = mfma32(rq[kb], kf[kb], s_out);
            asm volatile("" : "+v"(s_out));
            between(kb, 0);
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("" : "+v"(dp_out));
            dp_out = mfma32(rdo[kb], vf[kb], dp_out);
            asm volatile("" : "+v"(dp_out));
            between(kb, 1);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // ---- start of the pass: S, dP of its first block; its statistics and the second block's row
    // fragments are read meanwhile.  (The previous pass computed scores for this block too, with its own
    // K and V: they are dropped.)
    {
        const char* q0s = ring + c_stage;
        const char* q1s = ring + c_stage1;
#pragma unroll
        for (int kb = 0; kb < kSteps; kb++) read_rows(q0s, kb);
#pragma unroll
        for (int g = 0; g < 4; g++) { read_stat(s_even, wave_stat(c_stage), g); read_stat(dp_even, wave_stat(c_stage) + 32, g); }
        __builtin_amdgcn_sched_barrier(0);
        scores(s_even, dp_even, [&](int kb, int which) {
            if (kb < 4) {
                if (which == 0) read_stat(s_odd, wave_stat(c_stage1), kb);
                else read_stat(dp_odd, wave_stat(c_stage1) + 32, kb);
            }
        });
#pragma unroll
        for (int kb = 0; kb < kSteps; kb++) read_rows(q1s, kb);
        __builtin_amdgcn_sched_barrier(0);
    }

    // sc, dc: S - LSE / scale, dP - Delta of this block; s_next, dp_next: of the next one
    auto step = [&](auto masked, int blk, char* ds_head, f32x16& sc, f32x16& dc, f32x16& s_next, f32x16& dp_next) __attribute__((always_inline)) {
        const int i0 = i_begin + blk * S::kTileQ;
        const char* q0s = ring + c_stage;           // block n
        const char* q2s = ring + c_stage2;          // block n+2
        const int stage2 = c_stage2;
        c_stage = c_stage1;
        c_stage1 = c_stage2;
        c_stage2 = next_stage(c_stage2);

        // ---- first half.  After each MFMA of the next block's S, dP: one element of P and dS - the
        // exponential of element r is started in one group and used in the next, so that nothing waits
        // for it - and the transposing reads of one operand of the second half.
        float pe[16], de[16];
        float* const stat2 = wave_stat(stage2) + lane;      // statistics of block n+2, to be scaled
        float st = 0.f;
        auto element_start = [&](int r) {
            const int g = r >> 2, t = r & 3;
            float sv = sc[r];
            if (decltype(masked)::value && i0 + 8 * g + 4 * h + t + off < my_j) sv = -INFINITY;
            if (pad_key) sv = -INFINITY;
            pe[r] = __builtin_amdgcn_exp2f(sv * c);
            asm volatile("" : "+v"(pe[r]));
        };
        auto element_finish = [&](int r) {
            de[r] = pe[r] * dc[r];
            asm volatile("" : "+v"(de[r]));
        };
        scores(s_next, dp_next, [&](int kb, int which) {
            const int r = 2 * kb + which;
            element_start(r);
            if (r > 0) element_finish(r - 1);
            if (which == 0) read_tdo(q0s, kb); else read_tq(q0s, kb);
            if (r == 2) st = *stat2;
            if (kb == kSteps / 2 + 1) {          // (elements 0..8 are done)
                if (which == 0) {
                    pb[0] = cvt8(pe[0], pe[1], pe[2], pe[3], pe[4], pe[5], pe[6], pe[7]);
                    asm volatile("" : "+v"(pb[0]));
                } else {
                    dsb[0] = cvt8(de[0], de[1], de[2], de[3], de[4], de[5], de[6], de[7]);
                    asm volatile("" : "+v"(dsb[0]));
                }
            }
            if (r == 14) { st *= stat_mul; asm volatile("" : "+v"(st)); }
        });

        // ---- second half: the products of this block, next to the reads of the next blocks' fragments
        element_finish(15);
#pragma unroll
        for (int idx = 0; idx < kSteps; idx++) {
            const int ks = idx / (D / 32), db = idx % (D / 32);
            if (idx == 0) {                  // the second half of P, dS is not needed before idx = kSteps / 2
                pb[1] = cvt8(pe[8], pe[9], pe[10], pe[11], pe[12], pe[13], pe[14], pe[15]);
                dsb[1] = cvt8(de[8], de[9], de[10], de[11], de[12], de[13], de[14], de[15]);
            }
            dv_acc[db] = mfma32(tdo[idx], pb[ks], dv_acc[db]);
            asm volatile("" : : "v"(dv_acc[db][0]));
            rq[idx] = lds_read_b128(q2s, row_lane ^ ((2 * idx) << 4));
            if (idx == 0) asm volatile("" : "+v"(pb[1]), "+v"(dsb[1]));
            if (idx == 0) prepare();         // block n+6 goes into the stage of block n-1, which every wave has left
            if (idx == 0) *stat2 = st;
            if (idx == S::kLoadsPerBlock + 1) emit(S::kLoadsPerBlock);
            __builtin_amdgcn_sched_barrier(0);
            dk_acc[db] = mfma32(tq[idx], dsb[ks], dk_acc[db]);
            asm volatile("" : : "v"(dk_acc[db][0]));
            rdo[idx] = lds_read_b128(q2s + S::kQTileBytes, row_lane ^ ((2 * idx) << 4));
            if (idx >= 2 && idx < 6) read_stat(sc, wave_stat(stage2), idx - 2);           // (S and dP of block n+2 start from there)
            if (idx >= 4) read_stat(dc, wave_stat(stage2) + 32, idx - 4);
            if (idx >= 1 && idx <= S::kLoadsPerBlock) emit(idx - 1);
            if (SPILL && idx == kSteps / 2 + 2) {       // (both halves of dS exist; every step issues exactly these two stores)
                char* dst = ds_head + ((size_t)(i0 / S::kTileQ) * 4 + wave) * 2048 + lane * 16;
                *(bf16x8*)dst = dsb[0];
                *(bf16x8*)(dst + 1024) = dsb[1];
            }
            __builtin_amdgcn_sched_barrier(0);
        }

        // Block n+3 (issued three steps ago) must have landed before the next step reads it; the newer
        // prefetches stay in flight, and so do the dS stores issued since: the counter retires loads and stores in issue order, and the stores of the last
        // four steps are younger than the loads waited for.  After the barrier the next step's prefetch overwrites the stage of
        // block n: what this wave read from it (dO^T and Q^T above, rows and statistics two steps ago) has returned, since the MFMAs of this
        // step took it; the reads still in flight are of block n+2.
        constexpr int kStores = SPILL ? 8 : 0;
        prepare_turn();
        wait_vmcnt<3 * (S::kLoadsPerBlock + 1) + kStores>();
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };

    // When causal, the first n_masked blocks of every query head are the ones that may touch the
    // diagonal.  The stream runs on across the heads of the group.
#pragma unroll 1
    for (int g = 0; g < group; g++) {
        // dS blocks of (this query head, this key tile); query block 0 = queries 0..31 of the head
        char* ds_head = SPILL ? DS + ((q_head_of(g) * num_kv_tiles + kt) * n_qb) * (size_t)8192 : nullptr;
        int blk = 0;
        auto two_steps = [&](auto masked) __attribute__((always_inline)) {         // (n_blocks and n_masked are even)
            step(masked, blk, ds_head, s_even, dp_even, s_odd, dp_odd);
            step(masked, blk + 1, ds_head, s_odd, dp_odd, s_even, dp_even);
        };
        if (CAUSAL) {
#pragma unroll 1
            for (; blk < n_masked; blk += 2) two_steps(std::true_type{});
        }
#pragma unroll 1
        for (; blk < n_blocks; blk += 2) two_steps(std::false_type{});
    }
    } else {
    // ------------------------------------------------------------------------------------------
    // D = 64: the registers allow two workgroups per compute unit, i.e. two waves per SIMD that fill
    // each other's gaps; the phases of a block run one after the other.
    // ------------------------------------------------------------------------------------------
    bf16x8 rq[kSteps], rdo[kSteps];         // row fragments of the block about to be computed
    bf16x8 tq[kSteps], tdo[kSteps], pb[2], dsb[2];      // transposed fragments [ks * (D/32) + db] and bf16 P / dS of a block
    f32x16 s, dp;                           // S - LSE / scale, dP - Delta; start from the statistics, which the step before reads

    auto read_stat = [&](int stage, int g) {
        const f32x4 l = ((const f32x4*)wave_stat(stage))[2 * g + h], d = ((const f32x4*)wave_stat(stage))[8 + 2 * g + h];
#pragma unroll
        for (int t = 0; t < 4; t++) { s[4 * g + t] = l[t]; dp[4 * g + t] = d[t]; }
    };
    auto read_rows = [&](const char* qs, int kb) {
        rq[kb] = lds_read_b128(qs, row_lane ^ ((2 * kb) << 4));
        rdo[kb] = lds_read_b128(qs + S::kQTileBytes, row_lane ^ ((2 * kb) << 4));
    };
    auto read_transposed = [&](const char* qs, int idx) {
        const int ks = idx / (D / 32), db = idx % (D / 32);
        const int row_off = 16 * ks * S::kRowBytes;
        const int x0 = (4 * db) << 4, x1 = ((4 * db) ^ 2) << 4;
        const char* dos = qs + S::kQTileBytes;
        tdo[idx] = concat(lds_read_tr16(dos, (trq_lane ^ x0) + row_off),
                          lds_read_tr16(dos, (trq_lane ^ x1) + row_off + 8 * S::kRowBytes));
        tq[idx] = concat(lds_read_tr16(qs, (trq_lane ^ x0) + row_off),
                         lds_read_tr16(qs, (trq_lane ^ x1) + row_off + 8 * S::kRowBytes));
    };
#pragma unroll
    for (int kb = 0; kb < kSteps; kb++) { read_rows(ring + c_stage, kb); read_stat(c_stage, kb); }

    auto step = [&](auto masked, int blk, char* ds_head) {
        const int i0 = i_begin + blk * S::kTileQ;
        const char* qs = ring + c_stage;
        c_stage = next_stage(c_stage);
        const char* qs_next = ring + c_stage;
        float* const stat_next = wave_stat(c_stage) + lane;

        issue_next();                       // into the stage of the previous block, which every wave has left
        __builtin_amdgcn_sched_barrier(0);

        // ---- phase 1: S = Q K^T, dP = dO V^T; read this block's transposed fragments and statistics
        const float st = *stat_next * stat_mul;
#pragma unroll
        for (int kb = 0; kb < kSteps; kb++) {
            s = mfma32(rq[kb], kf[kb], s);
            dp = mfma32(rdo[kb], vf[kb], dp);
            read_transposed(qs, kb);
            __builtin_amdgcn_sched_barrier(0);
        }
        *stat_next = st;

        // ---- phase 2: P, dS.  Only the first blocks of a causal tile touch the diagonal: they run as a
        // loop of their own that pushes the masked scores to -inf (P = 2^-inf = 0), so that the main
        // loop carries no compare / select per element.
        if (decltype(masked)::value) {
#pragma unroll
            for (int r = 0; r < 16; r++)
                if (i0 + 8 * (r >> 2) + 4 * h + (r & 3) + off < my_j) s[r] = -INFINITY;
        }
        if (pad_key) {
#pragma unroll
            for (int r = 0; r < 16; r++) s[r] = -INFINITY;
        }
#pragma unroll
        for (int g = 0; g < 4; g++) {
#pragma unroll
            for (int t = 0; t < 4; t++) {
                const int r = 4 * g + t;
                const float p = __builtin_amdgcn_exp2f(s[r] * c);
                s[r] = p;
                dp[r] *= p;
            }
        }
#pragma unroll
        for (int ks = 0; ks < 2; ks++) {
            const int r0 = 8 * ks;
            pb[ks] = cvt8(s[r0], s[r0 + 1], s[r0 + 2], s[r0 + 3], s[r0 + 4], s[r0 + 5], s[r0 + 6], s[r0 + 7]);
            dsb[ks] = cvt8(dp[r0], dp[r0 + 1], dp[r0 + 2], dp[r0 + 3], dp[r0 + 4], dp[r0 + 5], dp[r0 + 6], dp[r0 + 7]);
        }
        // SPILL: every step issues exactly these two stores - the waits below count them
        if (SPILL) {
            char* dst = ds_head + ((size_t)(i0 / S::kTileQ) * 4 + wave) * 2048 + lane * 16;
            *(bf16x8*)dst = dsb[0];
            *(bf16x8*)(dst + 1024) = dsb[1];
        }

        // ---- phase 3: dV^T += dO^T P, dK^T += Q^T dS, and the reads of the next block's row fragments
        // (that block landed before the barrier that ended the previous iteration; the next block in the
        // stream is the next pass's first one after this pass's last)
#pragma unroll
        for (int idx = 0; idx < kSteps; idx++) {
            const int ks = idx / (D / 32), db = idx % (D / 32);
            dv_acc[db] = mfma32(tdo[idx], pb[ks], dv_acc[db]);
            dk_acc[db] = mfma32(tq[idx], dsb[ks], dk_acc[db]);
            read_rows(qs_next, idx);
            read_stat(c_stage, idx);
        }

        // the block two ahead in the stream (issued two iterations ago) must have landed before the
        // next iteration reads its rows; the newer prefetches may stay in flight.  After the barrier the next step's prefetch
        // overwrites the stage of this block: what this wave read from it has returned, since MFMAs of this step and of the one before took
        // it; the reads still in flight are of the next block.
        // (the counter retires loads and stores in issue order: the dS stores of this step and of the
        // previous one were issued after the loads waited for)
        constexpr int kStores = SPILL ? 4 : 0;
        wait_vmcnt<(S::kAhead - 2) * (S::kLoadsPerBlock + 1) + kStores>();
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };

#pragma unroll 1
    for (int g = 0; g < group; g++) {
        char* ds_head = SPILL ? DS + ((q_head_of(g) * num_kv_tiles + kt) * n_qb) * (size_t)8192 : nullptr;
        int blk = 0;
        if (CAUSAL) {
#pragma unroll 1
            for (; blk < n_masked; blk++) step(std::true_type{}, blk, ds_head);
        }
#pragma unroll 1
        for (; blk < n_blocks; blk++) step(std::false_type{}, blk, ds_head);
    }
    }

    // The next pass's K, V fragments are requested now, so that they travel while this pass's last
    // products and its stores run (S and dP are done with the old fragments).
    next_pass(c_vu, c_half);
    if (c_vu < total_units) {
        int nbh, nkt, nsplit;
        pass_tile(c_vu, c_half, nbh, nkt, nsplit);
        load_kv(nbh, nkt);
    }
    if (SPLIT) {            // fp32 sums, 16 bytes per lane straight from the accumulators
        if (my_j < Nk) {
            const size_t kv_floats = (size_t)(total_units / (units * n_splits)) * Nk * D;     // of all key/value heads
            float* dst = Part + (size_t)split * 2 * kv_floats + head + (size_t)my_j * D + 4 * h;
#pragma unroll
            for (int db = 0; db < D / 32; db++)
#pragma unroll
                for (int g = 0; g < 4; g++) {
                    *(f32x4*)(dst + 32 * db + 8 * g) = f32x4{dk_acc[db][4 * g], dk_acc[db][4 * g + 1], dk_acc[db][4 * g + 2], dk_acc[db][4 * g + 3]};
                    *(f32x4*)(dst + kv_floats + 32 * db + 8 * g) = f32x4{dv_acc[db][4 * g], dv_acc[db][4 * g + 1], dv_acc[db][4 * g + 2], dv_acc[db][4 * g + 3]};
                }
        }
        continue;
    }
    // ---- epilogue.  In accumulator layout a lane holds 4 consecutive columns of ONE key row
    // (lane <-> key my_j, register r of block db <-> column 32db + 8*(r/4) + 4h + r%4), so storing
    // from there would touch 32 rows per instruction.  Each wave instead turns its 32 x D tile
    // around in a private LDS buffer and stores whole rows, 16 bytes per lane.
    char* my_epi = epi + wave * (32 * S::kEpiPitch);
    auto store_tile = [&](const f32x16 (&acc)[D / 32], float mul, bf16* dst) {   // dst: first row of this wave's tile
#pragma unroll
        for (int db = 0; db < D / 32; db++)
#pragma unroll
            for (int g = 0; g < 4; g++) {
                bf16x2 a = cvt2(acc[db][4 * g] * mul, acc[db][4 * g + 1] * mul);
                bf16x2 b = cvt2(acc[db][4 * g + 2] * mul, acc[db][4 * g + 3] * mul);
                *(bf16x4*)(my_epi + l32 * S::kEpiPitch + (32 * db + 8 * g + 4 * h) * 2) = __builtin_shufflevector(a, b, 0, 1, 2, 3);
            }
        constexpr int kLanesPerRow = D * 2 / 16;
        constexpr int kRowsPerStore = 64 / kLanesPerRow;
        const int sub_row = lane / kLanesPerRow, col16 = lane % kLanesPerRow;
#pragma unroll
        for (int i = 0; i < 32 / kRowsPerStore; i++) {
            const int row = i * kRowsPerStore + sub_row;
            const char* src = my_epi + row * S::kEpiPitch + col16 * 16;
            const bf16x4 lo = *(const bf16x4*)src, hi = *(const bf16x4*)(src + 8);
            if (!TAIL || jw0 + row < Nk) *(bf16x8*)(dst + (size_t)row * D + col16 * 8) = concat(lo, hi);
        }
    };
    store_tile(dk_acc, scale, dK + head + (size_t)jw0 * D);
    store_tile(dv_acc, 1.0f, dV + head + (size_t)jw0 * D);
    }   // pass
    wait_vmcnt<0>();      // the spare prefetches of the last blocks must not outlive the workgroup's LDS
}

// dK = scale * sum of the n_splits partial sums, dV likewise without the scale; blockIdx.y: 0 dK, 1 dV.  n4: groups of four elements of one tensor.
__global__ __launch_bounds__(256)
void attn_bwd_dkdv_sum_kernel(const float* __restrict__ Part, bf16* __restrict__ dK, bf16* __restrict__ dV, size_t n4, int n_splits, float scale)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n4) return;
    const f32x4* src = (const f32x4*)Part + (size_t)blockIdx.y * n4 + i;
    f32x4 acc = src[0];
#pragma unroll 4
    for (int s = 1; s < n_splits; s++) acc += src[(size_t)s * 2 * n4];
    const float mul = blockIdx.y == 0 ? scale : 1.0f;
    const bf16x2 lo = cvt2(acc[0] * mul, acc[1] * mul), hi = cvt2(acc[2] * mul, acc[3] * mul);
    *(bf16x4*)((blockIdx.y == 0 ? dK : dV) + 4 * i) = __builtin_shufflevector(lo, hi, 0, 1, 2, 3);
}

template <int D, bool CAUSAL, bool TAIL, bool SPILL, bool SPLIT>
static hipError_t launch_dkdv_tt(const void* q, const void* k, const void* v, const void* d_o,
                                 const float* lse, const float* delta, void* dk, void* dv,
                                 int B, int H, int Hkv, int Nq, int Nk, float scale, hipStream_t stream, void* ds,
                                 int resident, bool paired, int n_splits, int q_splits, float* part)
{
    using S = DkdvShape<D>;
    const int num_kv_tiles = (Nk + S::kTileKV - 1) / S::kTileKV;
    const int units = CAUSAL && paired ? (num_kv_tiles + 1) / 2 : num_kv_tiles;
    const int total_units = B * Hkv * n_splits * units;
    const int grid = total_units < resident ? total_units : resident;
    hipLaunchKernelGGL((attn_bwd_dkdv_kernel<D, CAUSAL, TAIL, SPILL, SPLIT>), dim3(grid), dim3(S::kThreads), 0, stream,
                       (const bf16*)q, (const bf16*)k, (const bf16*)v, (const bf16*)d_o, lse, delta,
                       (bf16*)dk, (bf16*)dv, Nq, Nk, num_kv_tiles, total_units, scale, H, Hkv, grid,
                       (char*)ds, ds_query_blocks(Nq), units, n_splits, q_splits, part);
    if (SPLIT) {
        const size_t n4 = (size_t)B * Hkv * Nk * D / 4;
        hipLaunchKernelGGL(attn_bwd_dkdv_sum_kernel, dim3((unsigned)((n4 + 255) / 256), 2), dim3(256), 0, stream,
                           part, (bf16*)dk, (bf16*)dv, n4, n_splits, scale);
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// kernel 2 at D = 128 for large launches: 64 keys a wave
// ------------------------------------------------------------------------------------------
// The same work in the same order (the bits of dK, dV and dS are those of the kernel above, except that a NaN of its masked blocks may
// be a number here), with tiles of 256 keys: every Q, dO
// row that comes from L2, and every fragment that is read from LDS, serves twice the matrix instructions.  One wave per SIMD:
// the dK^T, dV^T accumulators take the whole accumulator half of the register file; K stays in registers, V in LDS.  A step is
//     first half    S, dP of block n (32 MFMAs)  next to  the LDS reads of its rows, the fetch of block n+3, the statistics of
//                   block n+1, the dS stores of block n-1 and the first fragments of the second half
//     second half   dV^T, dK^T of block n-1 (32 MFMAs)  next to  P, dS of block n, one element behind each MFMA, and the first
//                   fragments of the next step
// What bounds it: the second half has 4.6 vector instructions to an MFMA, which a single wave issues in about 40 of the 32
// cycles that the matrix pipe takes; and power (without its loads the kernel takes 13 % less time on normal data, on
// constant data 5 %).  dK/dV alone, us, 128 keys and 256: B16 H16 N4096 without a mask 3680, 3300; causal 2020, 1870; causal and
// storing dS 2385, 2255 (with 22 and 24 registers in scratch memory 1945, 2378).  The matrix pipe is busy in 56 % of its cycles (128-key
// tiles: 47 %).  From beyond L2 it reads more, 4.2 GB there instead of 1.7: the workgroups of an XCD are at four heads at once, 8 MB of Q
// and dO, and not at two.  It stores 0.13 GB of dS more, blocks that the mask takes wholly.  Two waves per SIMD in turns, as in the forward, do not fit: 256 registers a wave.
//
// The accumulators are only touched by inline assembly, which the compiler sees as writing them at once: results are read, and
// copies made in front of a product, behind the waits that the hardware wants (mfma32_acc_wait, and the s_nop behind the last).
__device__ __forceinline__ void mfma32_acc(f32x16& acc, bf16x8 a, bf16x8 b) {     // acc stays where it is from one product to the next
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
// behind copies of the accumulator
__device__ __forceinline__ void mfma32_acc_wait(f32x16& acc, bf16x8 a, bf16x8 b) {
    asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
struct DkdvWideShape {
    static constexpr int D = 128;
    static constexpr int kWaves = 4, kThreads = 256;
    static constexpr int kTileKV = 256;                 // keys per workgroup (64 per wave)
    static constexpr int kTileQ = 32;
    static constexpr int kStages = 5;
    static constexpr int kRowBytes = D * 2, kChunksPerRow = D / 8;
    static constexpr int kQTileBytes = kTileQ * kRowBytes;
    static constexpr int kStageBytes = 2 * kQTileBytes;
    static constexpr int kQLoads = kTileQ * kChunksPerRow / kThreads;
    static constexpr int kBlockLoads = 2 * kQLoads + 1;
    static constexpr int kWaveBytes = 64 * kRowBytes;   // a wave's V tile
    static constexpr int kEpiPitch = 128;               // the epilogue turns 32 rows x 64 columns around at a time,
    static_assert(kWaves * 32 * kEpiPitch <= kStageBytes, "in the ring stage that is free at the end of a pass");
    // Behind the ring: rows of zeros, the rows 0, 8, 16 and 24 of a Q and of a dO block that are nothing but zeros (the reads of
    // columns use the rows between them only through a lane's offset), and between them the statistics of the stages, 256 bytes a wave.
    static constexpr int kZeros = kStages * kStageBytes, kZeroPitch = 8 * kRowBytes;
    static constexpr int kRingBytes = kZeros + 7 * kZeroPitch + kRowBytes;
    static_assert(kStages <= 7 && kRowBytes + kWaves * 256 <= kZeroPitch && kStageBytes == 8 * kZeroPitch, "the statistics of stage s lie behind the zeros of row 8 s");
};

template <bool CAUSAL, bool TAIL, bool SPILL>
__global__ __launch_bounds__(256, 1)
void attn_bwd_dkdv_wide_kernel(const bf16* __restrict__ Q, const bf16* __restrict__ K, const bf16* __restrict__ V,
                               const bf16* __restrict__ dO, const float* __restrict__ LSE, const float* __restrict__ Delta,
                               bf16* __restrict__ dK, bf16* __restrict__ dV,
                               int Nq, int Nk, int num_kv_tiles, int total_units, float scale, int hq, int hkv, int stride,
                               char* __restrict__ DS, int n_qb, int units)
{
    using S = DkdvWideShape;
    constexpr int D = S::D, kSteps = D / 16;
    __shared__ __attribute__((aligned(1024))) char ring[S::kRingBytes];
    __shared__ __attribute__((aligned(1024))) char own[S::kWaves * S::kWaveBytes];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int l32 = lane & 31;
    const int h = lane >> 5;
    const int j16 = lane & 15;
    const int ghalf = (lane >> 4) & 1;
    const float score_scale = scale < kLeastScale ? scale * 0x1p64f : scale;     // (see shrink_k)
    const float c = score_scale * kLog2e;
    const int heads_per_kv = hq / hkv;
    const int off = TAIL ? Nk - Nq : 0;
    char* const mine = own + wave * S::kWaveBytes;

    auto q_head_row = [&](int bh) { return (size_t)((bh / hkv) * hq + (bh % hkv) * heads_per_kv) * Nq; };
    auto pass_ibegin = [&](int kt) {
        if (!CAUSAL) return 0;
        const int first = kt * S::kTileKV - off;
        return first > 0 ? first & ~(S::kTileQ - 1) : 0;
    };
    auto pass_nblocks = [&](int ibegin) { return 2 * ((Nq - ibegin + 2 * S::kTileQ - 1) / (2 * S::kTileQ)); };
    auto pass_tile = [&](int vu, int half, int& bh, int& kt) {
        const int logical = xcd_remap(vu, total_units);
        bh = logical / units;
        const int unit = logical % units;
        kt = half == 0 ? unit : num_kv_tiles - 1 - unit;
    };
    auto next_pass = [&](int& vu, int& half) {
        if (CAUSAL && half == 0) {
            const int unit = xcd_remap(vu, total_units) % units;
            if (num_kv_tiles - 1 - unit >= units) { half = 1; return; }
        }
        vu += stride;
        half = 0;
    };

    // ---- query-block prefetch (the cursor of the kernel above)
    int q_src[S::kQLoads];
#pragma unroll
    for (int it = 0; it < S::kQLoads; it++) {
        int s = it * S::kThreads + tid;
        int row = s / S::kChunksPerRow, pc = s % S::kChunksPerRow;
        q_src[it] = row * D + ((pc ^ swz<D>(row)) * 8);
    }
    const float* const stat_src = (lane < 32 ? LSE : Delta) + l32;
    int p_vu = blockIdx.x, p_half = 0, p_nblocks = 0, p_g = 0, p_ibegin = 0;
    size_t p_head_row = 0, p_row = 0;
    int p_i0 = 0, p_left = 0, p_advance = S::kTileQ, p_stage = 0;
    auto next_stage = [&](int at) { return at + S::kStageBytes == S::kStages * S::kStageBytes ? 0 : at + S::kStageBytes; };
    auto producer_head = [&]() __attribute__((always_inline)) {
        p_row = p_head_row + (size_t)p_g * Nq + p_ibegin;
        p_i0 = p_ibegin;
        p_left = p_nblocks;
    };
    auto producer_open = [&]() __attribute__((always_inline)) {
        int bh, kt;
        pass_tile(p_vu, p_half, bh, kt);
        p_ibegin = pass_ibegin(kt);
        p_head_row = q_head_row(bh);
        p_nblocks = pass_nblocks(p_ibegin);
        p_g = 0;
        producer_head();
    };
    auto producer_turn = [&]() __attribute__((always_inline)) {
        if (++p_g < heads_per_kv) { producer_head(); return; }
        next_pass(p_vu, p_half);
        if (p_vu < total_units) { producer_open(); return; }
        p_row -= p_advance;                 // exhausted: stay on the last block
        p_i0 -= p_advance;
        p_advance = 0;
        p_left = 0x7fffffff;
    };
    size_t e_head_row = 0, e_row = 0;       // of the block being fetched
    int e_i0 = 0, e_stage = 0;
    auto prepare = [&]() __attribute__((always_inline)) {
        e_row = p_row;
        e_i0 = p_i0;
        e_head_row = p_row - p_i0;
        e_stage = p_stage;
        p_stage = next_stage(p_stage);
        p_row += p_advance;
        p_i0 += p_advance;
        --p_left;
    };
    auto prepare_turn = [&]() __attribute__((always_inline)) {
        if (__builtin_expect(p_left == 0, 0)) producer_turn();
    };
    auto wave_stat = [&](int stage) { return (float*)(ring + S::kZeros + S::kRowBytes + (stage >> 3) + wave * 256); };
    auto emit = [&](int which) __attribute__((always_inline)) {
        char* base = ring + e_stage;
        if (which < 2 * S::kQLoads) {       // Q rows, then dO rows
            const int it = which % S::kQLoads;
            const bf16* block = (which < S::kQLoads ? Q : dO) + e_row * D;
            char* dst = base + (which < S::kQLoads ? 0 : S::kQTileBytes) + it * (S::kThreads * 16) + wave * 1024;
            if (TAIL) {
                const int r = e_i0 + (it * S::kThreads + tid) / S::kChunksPerRow;
                load_global_to_lds16_untracked(block + q_src[it] - (r < Nq ? 0 : r - (Nq - 1)) * D, dst);
            } else {
                load_global_to_lds16_sbase_untracked(block, (uint32_t)q_src[it] * 2, dst);
            }
        } else {
            const float* src = stat_src + e_row;
            if (TAIL && e_i0 + l32 >= Nq) src = lane < 32 ? g_lse_pad : Delta + e_head_row + (Nq - 1);
            load_global_to_lds4_untracked(src, (const char*)wave_stat(e_stage));
        }
    };
    const float stat_mul = lane < 32 ? -1.0f / score_scale : -1.0f;
    auto scale_stat = [&](int stage) __attribute__((always_inline)) { float* st = wave_stat(stage) + lane; *st = *st * stat_mul; };

    // ---- per-lane LDS offsets
    const int row_lane = l32 * S::kRowBytes + ((h ^ swz<D>(l32)) << 4);
    const int trq_row = 4 * h + (j16 >> 2);
    const int trq_lane = trq_row * S::kRowBytes + (((2 * ghalf + ((j16 & 3) >> 1)) ^ swz<D>(trq_row)) << 4) + ((j16 & 1) << 3);

    // Offsets that depend on the lane alone are formed from a copy that the compiler does not see through, where they are used: it would
    // keep them for the whole kernel otherwise, which has no registers to spare (up to 24 went to scratch memory).
    auto opaque = [](int x) __attribute__((always_inline)) { asm volatile("" : "+v"(x)); return x; };
    bf16x8 kf[2][kSteps];                   // K fragments of the wave's two halves of 32 keys
    f32x16 dk_acc[2][D / 32], dv_acc[2][D / 32], sc[2], dc[2], st_l, st_d;
    struct Products { bf16x8 p[2][2], d[2][2]; };       // bf16 P, dS of a block: [half][16 queries]
    Products even, odd;

    auto load_kv = [&](int bh, int kt) __attribute__((always_inline)) {
        const int ln = opaque(lane);
        const int key0 = kt * S::kTileKV + wave * 64;
        const size_t head_row = (size_t)bh * Nk;
        const int key_first = !TAIL || key0 < Nk ? key0 : Nk - 1, last = TAIL ? Nk - 1 - key_first : 63;
#pragma unroll
        for (int it = 0; it < S::kWaveBytes / 1024; it++) {
            const int r = it * 4 + (ln >> 4);
            load_global_to_lds16_sbase_untracked(V + (head_row + key_first) * D, (uint32_t)((TAIL && r > last ? last : r) * D + (((ln & 15) ^ swz<D>(r)) * 8)) * 2, mine + it * 1024);
        }
#pragma unroll
        for (int b = 0; b < 2; b++) {
            const int key = key0 + 32 * b + (ln & 31);
            const bf16* row = K + (head_row + ((!TAIL || key < Nk) ? key : Nk - 1)) * D;
#pragma unroll
            for (int kb = 0; kb < kSteps; kb++) kf[b][kb] = *(const bf16x8*)(row + kb * 16 + (ln >> 5) * 8);
        }
    };
    auto keep_k = [&]() __attribute__((always_inline)) {        // (the wait for K belongs here and not at its first use)
        if (__builtin_expect(scale < kLeastScale, 0)) {
#pragma unroll
            for (int b = 0; b < 2; b++)
#pragma unroll
                for (int kb = 0; kb < kSteps; kb++) shrink_k(kf[b][kb]);
        }
#pragma unroll
        for (int b = 0; b < 2; b++)
#pragma unroll
            for (int kb = 0; kb < kSteps; kb++) asm volatile("" : "+v"(kf[b][kb]));
    };
    auto step_end = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" : : : "memory");
    };
    auto read_stats = [&](int stage, int b, int g) __attribute__((always_inline)) {
        const f32x4 x = ((const f32x4*)wave_stat(stage))[8 * b + 2 * g + h];
#pragma unroll
        for (int t = 0; t < 4; t++) (b == 0 ? st_l : st_d)[4 * g + t] = x[t];
    };
    struct Rows { bf16x8 q[kSteps], d[kSteps], v[2][kSteps]; };
    struct Columns { bf16x8 q[kSteps], d[kSteps]; };
    auto read_row = [&](Rows& f, int rl, int stage, int kb, int part) __attribute__((always_inline)) {
        const int at = rl ^ ((2 * kb) << 4);
        if (part == 0) { f.q[kb] = lds_read_b128(ring + stage, at); f.d[kb] = lds_read_b128(ring + stage + S::kQTileBytes, at); }
        else { f.v[0][kb] = lds_read_b128(mine, at); f.v[1][kb] = lds_read_b128(mine + 32 * S::kRowBytes, at); }
    };
    bf16x8 row_q[2], row_d[2], row_v[2][2], col_q[2], col_d[2];         // the first fragments, read half a step ahead
    auto read_row_ahead = [&](int rl, int stage, int n) __attribute__((always_inline)) {
        const int kb = n >> 2, at = rl ^ ((2 * kb) << 4);
        if ((n & 3) == 0) row_q[kb] = lds_read_b128(ring + stage, at);
        if ((n & 3) == 1) row_d[kb] = lds_read_b128(ring + stage + S::kQTileBytes, at);
        if ((n & 3) == 2) row_v[0][kb] = lds_read_b128(mine, at);
        if ((n & 3) == 3) row_v[1][kb] = lds_read_b128(mine + 32 * S::kRowBytes, at);
    };
    auto read_tr = [&](bf16x8& f, int tl, const char* rows, int idx) __attribute__((always_inline)) {
        const int row_off = 16 * (idx / (D / 32)) * S::kRowBytes, db = idx % (D / 32);
        f = concat(lds_read_tr16(rows, (tl ^ ((4 * db) << 4)) + row_off), lds_read_tr16(rows, (tl ^ (((4 * db) ^ 2) << 4)) + row_off + 8 * S::kRowBytes));
    };

    int c_vu = blockIdx.x, c_half = 0, c_stage = 0;
    {
        int bh, kt;
        pass_tile(c_vu, c_half, bh, kt);
        producer_open();
#pragma unroll
        for (int b = 0; b < 3; b++) {
            prepare();
#pragma unroll
            for (int which = 0; which < S::kBlockLoads; which++) emit(which);
            prepare_turn();
        }
        load_kv(bh, kt);
    }
    *(uint64_t*)(ring + S::kZeros + (tid >> 5) * S::kZeroPitch + (tid & 31) * 8) = 0;
    keep_k();
    wait_vmcnt_lds_done<0>();
    scale_stat(0);
    step_end();

#pragma unroll 1
    while (c_vu < total_units) {
        int bh, kt;
        pass_tile(c_vu, c_half, bh, kt);
        const int jw0 = kt * S::kTileKV + wave * 64, my_j = jw0 + l32;
        const int i_begin = pass_ibegin(kt), n_blocks = pass_nblocks(i_begin);
        const int kv_tiles128 = (Nk + 127) / 128;
        const bool stores = SPILL && (!TAIL || (jw0 >> 7) < kv_tiles128);
        const size_t ds_head_bytes = (size_t)kv_tiles128 * n_qb * 8192;
        int i0 = i_begin, left = n_blocks;
        char* ds = nullptr;
        if (SPILL) ds = DS + ((((size_t)(bh / hkv) * hq + (size_t)(bh % hkv) * heads_per_kv) * kv_tiles128 + (jw0 >> 7)) * n_qb * 4 + ((jw0 >> 5) & 3)) * 2048
                        + lane * 16 + (size_t)(i_begin / S::kTileQ) * 8192;
        auto advance = [&]() __attribute__((always_inline)) {
            i0 += S::kTileQ;
            if (SPILL) ds += 8192;
            if (__builtin_expect(--left == 0, 0)) {     // on to the next query head
                i0 = i_begin;
                left = n_blocks;
                if (SPILL) ds += ds_head_bytes - (size_t)n_blocks * 8192;
            }
        };
#pragma unroll
        for (int b = 0; b < 2; b++)
#pragma unroll
            for (int db = 0; db < D / 32; db++)
#pragma unroll
                for (int r = 0; r < 16; r++) { dk_acc[b][db][r] = 0.f; dv_acc[b][db][r] = 0.f; }

        auto store_ds = [&](char* dst, const Products& x) __attribute__((always_inline)) {
            if (SPILL && stores) {
#pragma unroll
                for (int b = 0; b < 2; b++)
#pragma unroll
                    for (int ks = 0; ks < 2; ks++) *(bf16x8*)(dst + 2048 * b + 1024 * ks) = x.d[b][ks];
            }
        };
        // First half of a step: S, dP of its block (both halves of the keys, whose statistics are in sc, dc already).  Beside the
        // matrix instructions: the fetch of the block three ahead and the statistics of the next one.
        auto scores = [&](int stage, int stage_next, int cols, int col_lane, char* ds_last, const Products& last, bool first) __attribute__((always_inline)) {
            Rows f;
            const int rl = opaque(row_lane), tl = opaque(col_lane);
            float* const st = wave_stat(stage_next) + lane;
            float x = 0.f;
#pragma unroll
            for (int kb = 0; kb < 2; kb++) { f.q[kb] = row_q[kb]; f.d[kb] = row_d[kb]; f.v[0][kb] = row_v[0][kb]; f.v[1][kb] = row_v[1][kb]; }
#pragma unroll
            for (int kb = 0; kb < kSteps; kb++) {
                sc[0] = mfma32(f.q[kb], kf[0][kb], kb == 0 ? st_l : sc[0]);
                asm volatile("" : : "v"(sc[0][0]));
                if (kb == 0) prepare();
                if (kb >= 1 && kb <= S::kBlockLoads) emit(kb - 1);
                __builtin_amdgcn_sched_barrier(0);
                sc[1] = mfma32(f.q[kb], kf[1][kb], kb == 0 ? st_l : sc[1]);
                asm volatile("" : : "v"(sc[1][0]));
                if (kb + 2 < kSteps) read_row(f, rl, stage, kb + 2, 0);
                else read_tr(col_d[kb - 6 < 0 ? 0 : kb - 6], tl, ring + cols + S::kQTileBytes, kb - 6);
                __builtin_amdgcn_sched_barrier(0);
                dc[0] = mfma32(f.d[kb], f.v[0][kb], kb == 0 ? st_d : dc[0]);
                asm volatile("" : : "v"(dc[0][0]));
                if (kb == 2) x = *st;
                if (kb == 5) *st = x * stat_mul;
                if (SPILL && kb >= 6 && stores && !first) {
                    *(bf16x8*)(ds_last + 2048 * (kb - 6)) = last.d[kb & 1][0];
                    *(bf16x8*)(ds_last + 2048 * (kb - 6) + 1024) = last.d[kb & 1][1];
                }
                __builtin_amdgcn_sched_barrier(0);
                dc[1] = mfma32(f.d[kb], f.v[1][kb], kb == 0 ? st_d : dc[1]);
                asm volatile("" : : "v"(dc[1][0]));
                if (kb + 2 < kSteps) read_row(f, rl, stage, kb + 2, 1);
                else read_tr(col_q[kb - 6 < 0 ? 0 : kb - 6], tl, ring + cols, kb - 6);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        auto mask = [&]() __attribute__((always_inline)) {
            if (CAUSAL && __builtin_expect(i0 + off < jw0 + 63, 0)) {
                // register r <-> query i0 + 4h + (a constant): one difference per lane and half.  (Sixteen offsets that the compiler formed
                // once lay in scratch memory, and their reload waited for the fetch of block n+3 as well.)
#pragma unroll
                for (int b = 0; b < 2; b++) {
                    const int first_seen = opaque(my_j + 32 * b - off - i0 - 4 * h);
#pragma unroll
                    for (int r = 0; r < 16; r++)
                        if (8 * (r >> 2) + (r & 3) < first_seen) sc[b][r] = -INFINITY;
                }
            }
            if (TAIL && SPILL && __builtin_expect(jw0 + 63 >= Nk, 0)) {
#pragma unroll
                for (int b = 0; b < 2; b++)
#pragma unroll
                    for (int r = 0; r < 16; r++)
                        if (my_j + 32 * b >= Nk) sc[b][r] = -INFINITY;
            }
        };
        // Second half: dV^T, dK^T of the block before, and beside them P, dS of this block, one element for each matrix instruction.
        auto products = [&](int cols, int col_lane, int stage_next, const Products& last, Products& next, auto has_last, auto has_vector) __attribute__((always_inline)) {
            Columns f;
            const int tl = opaque(col_lane);
            const char* qs = ring + cols;
            const char* dos = qs + S::kQTileBytes;
            float pe[32], de[32];
            const int rl = opaque(row_lane);
            if (!decltype(has_vector)::value) {
#pragma unroll
                for (int i = 0; i < 2; i++) { read_tr(col_d[i], tl, dos, i); read_tr(col_q[i], tl, qs, i); }
            }
#pragma unroll
            for (int i = 0; i < 2; i++) { f.d[i] = col_d[i]; f.q[i] = col_q[i]; }
            auto start = [&](int e) __attribute__((always_inline)) { pe[e] = __builtin_amdgcn_exp2f(sc[e >> 4][e & 15] * c); asm volatile("" : : "v"(pe[e])); };
            auto finish = [&](int e) __attribute__((always_inline)) { de[e] = pe[e] * dc[e >> 4][e & 15]; asm volatile("" : : "v"(de[e])); };
            auto pack = [&](const float (&x)[32], int e, bf16x8& to) __attribute__((always_inline)) {
                to = cvt8(x[e], x[e + 1], x[e + 2], x[e + 3], x[e + 4], x[e + 5], x[e + 6], x[e + 7]);
                asm volatile("" : "+v"(to));
            };
#pragma unroll
            for (int i = 0; i < 32; i++) {
                const int idx = i >> 2, j = i & 3, ks = idx / (D / 32), db = idx % (D / 32);
                if (decltype(has_last)::value) {
                    f32x16& acc = j < 2 ? dv_acc[j & 1][db] : dk_acc[j & 1][db];
                    const bf16x8 a = j < 2 ? f.d[idx] : f.q[idx], b = j < 2 ? last.p[j & 1][ks] : last.d[j & 1][ks];
                    if (decltype(has_vector)::value) mfma32_acc(acc, a, b); else mfma32_acc_wait(acc, a, b);
                    if (j == 1 && idx + 2 < kSteps) read_tr(f.d[idx + 2], tl, dos, idx + 2);
                    if (j == 3 && idx + 2 < kSteps) read_tr(f.q[idx + 2], tl, qs, idx + 2);
                }
                if (decltype(has_vector)::value) {
                    start(i);
                    if (i > 0) finish(i - 1);
                    if (i % 8 == 1 && i > 8) pack(pe, i - 9, next.p[(i - 9) >> 4][((i - 9) >> 3) & 1]);
                    if (i % 8 == 2 && i > 9) pack(de, i - 10, next.d[(i - 10) >> 4][((i - 10) >> 3) & 1]);
                    if (i >= 18 && i < 26) read_row_ahead(rl, stage_next, i - 18);
                    if (i >= 24) read_stats(stage_next, (i - 24) >> 2, i & 3);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (decltype(has_vector)::value) {
                finish(31);
                pack(pe, 24, next.p[1][1]);
                pack(de, 24, next.d[1][1]);
                if (CAUSAL && __builtin_expect(i0 + S::kTileQ - 1 + off < jw0, 0)) {
#pragma unroll
                    for (int b = 0; b < 2; b++)
#pragma unroll
                        for (int ks = 0; ks < 2; ks++) next.d[b][ks] = bf16x8{};
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        auto step = [&](int stage_last, const Products& last, Products& next, bool first) __attribute__((always_inline)) {
            const int stage = c_stage, stage_next = next_stage(stage);
            c_stage = stage_next;
            char* const ds_last = ds;                   // of the block before
            // Where there is no block before, or the mask took it wholly, P = dS = 0 meet columns of zeros: its rows may hold an
            // infinity or a NaN.  (A second copy of the step without products does not fit the registers.)
            const bool none = first || (CAUSAL && i0 + S::kTileQ - 1 + off < jw0);
            const int cols = none ? S::kZeros : stage_last, col_lane = none ? 0 : trq_lane;
            if (!first) advance();
            scores(stage, stage_next, cols, col_lane, ds_last, last, first);
            mask();
            products(cols, col_lane, stage_next, last, next, std::true_type{}, std::true_type{});
            prepare_turn();
            // block n+2, fetched in the step before, has to be here; younger are that step's stores and this one's loads and stores.
            // The first step of a pass has none, and the count is the one that holds behind it too: later steps wait for
            // the stores of the step before as well.
            if (SPILL && stores && !first) wait_vmcnt<S::kBlockLoads + 4>(); else wait_vmcnt<S::kBlockLoads>();
            step_end();
        };
        // ---- the pass, an even number of blocks
#pragma unroll
        for (int b = 0; b < 2; b++)
#pragma unroll
            for (int ks = 0; ks < 2; ks++) { odd.p[b][ks] = bf16x8{}; odd.d[b][ks] = bf16x8{}; }
#pragma unroll
        for (int n = 0; n < 8; n++) { read_row_ahead(row_lane, c_stage, n); read_stats(c_stage, n >> 2, n & 3); }
        int stage_last = c_stage;
        bool first = true;
#pragma unroll 1
        for (int more = heads_per_kv * n_blocks; more > 0; more -= 2) {
            const int s0 = c_stage;
            step(stage_last, odd, even, first);
            stage_last = c_stage;
            step(s0, even, odd, false);
            first = false;
        }
        // K and V are done with: those of the next pass travel while this one's results are stored
        next_pass(c_vu, c_half);
        const bool another = c_vu < total_units;
        if (another) {
            int nbh, nkt;
            pass_tile(c_vu, c_half, nbh, nkt);
            load_kv(nbh, nkt);
        }
        store_ds(ds, odd);
        products(stage_last, trq_lane, 0, odd, even, std::true_type{}, std::false_type{});
        // the accumulators may be read from here on (the compiler does not know how long the products take)
        asm volatile("s_nop 15\n\ts_nop 15" : "+a"(dv_acc[0][0]), "+a"(dv_acc[0][1]), "+a"(dv_acc[0][2]), "+a"(dv_acc[0][3]));
        asm volatile("" : "+a"(dv_acc[1][0]), "+a"(dv_acc[1][1]), "+a"(dv_acc[1][2]), "+a"(dv_acc[1][3]));
        asm volatile("" : "+a"(dk_acc[0][0]), "+a"(dk_acc[0][1]), "+a"(dk_acc[0][2]), "+a"(dk_acc[0][3]));
        asm volatile("" : "+a"(dk_acc[1][0]), "+a"(dk_acc[1][1]), "+a"(dk_acc[1][2]), "+a"(dk_acc[1][3]));

        // ---- the pass's results
        const size_t head = (size_t)bh * Nk * D;
        char* const turn = ring + p_stage + wave * (32 * S::kEpiPitch);      // (the stage the next block will be fetched into)
        auto store_tile = [&](const f32x16 (&acc)[D / 32], float mul, bf16* dst, int key0) __attribute__((always_inline)) {
            const int ln = opaque(lane), l = ln & 31;
#pragma unroll
            for (int half = 0; half < D / 64; half++) {
#pragma unroll
                for (int db = 2 * half; db < 2 * half + 2; db++)
#pragma unroll
                    for (int q = 0; q < 4; q++) {
                        bf16x2 a = cvt2(acc[db][4 * q] * mul, acc[db][4 * q + 1] * mul);
                        bf16x2 b = cvt2(acc[db][4 * q + 2] * mul, acc[db][4 * q + 3] * mul);
                        *(bf16x4*)(turn + l * S::kEpiPitch + (((4 * (db & 1) + q) ^ (l & 7)) << 4) + 8 * (ln >> 5)) = __builtin_shufflevector(a, b, 0, 1, 2, 3);
                    }
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const int row = i * 8 + (ln >> 3);
                    const bf16x8 x = *(const bf16x8*)(turn + row * S::kEpiPitch + (((ln & 7) ^ (row & 7)) << 4));
                    if (!TAIL || key0 + row < Nk) *(bf16x8*)(dst + (size_t)(key0 + row) * D + 64 * half + (ln & 7) * 8) = x;
                }
            }
        };
#pragma unroll
        for (int b = 0; b < 2; b++) {
            store_tile(dk_acc[b], scale, dK + head, jw0 + 32 * b);
            store_tile(dv_acc[b], 1.0f, dV + head, jw0 + 32 * b);
        }
        if (another) keep_k();
        wait_vmcnt<0>();
        step_end();                         // (no wave fetches into the stage of the last block before all are done with it)
    }
}

// Whether tiles of 256 keys take less time than tiles of 128: us of the workgroup with most units, a block of 32 queries at
// 1.07 (128 keys, 0.1 more where it may be masked) and 1.85 us (256), the ends of a pass at 4 and 7.  A unit is a key tile, or
// a causal pair of them.  Fitted to 720 backward calls of 1 to 8192 queries and 128 to 16384 keys, grouped or not, with and without a mask
// and stored dS, both ways timed, and checked on 420 others: the choice takes 0.15 % more than the better way on average; of the 840 with at
// least 128 queries 363 take the 256-key tiles, their whole call 9 % faster on average; 17 of all lose more than 1 %, one of them 14 and one 10.
// (With 0.5 us for a masked block, as when those went through scratch memory, 1 % more; us, 128 keys and 256: B9 Hq24 Hkv12 Nq160 Nk794
// causal 111, 96; B12 Hq64 Hkv16 Nq143 Nk4680 1366, 1176.  With 6 us for the ends 27 of 300 calls of few queries lost up to 9 %.)
static bool dkdv_wide_pays(int B, int H, int Hkv, int Nq, int Nk, bool causal, int cus)
{
    auto us = [&](int keys, double block_us, double masked_us, double pass_us) {
        const int tiles = (Nk + keys - 1) / keys;
        const bool paired = causal && (keys == 256 || pair_tiles((long long)B * Hkv, tiles, cus));
        const int units = paired ? (tiles + 1) / 2 : tiles, passes = paired && tiles > 1 ? 2 : 1;
        const long long rounds = ((long long)B * Hkv * units + cus - 1) / cus;
        // of a causal pair both passes together; otherwise the longest pass
        double blocks = Nq / 32.0 * passes;
        const double late = ((tiles - 1) * (double)keys - (Nk - Nq)) / 32;      // blocks that the last tile does not see
        if (passes == 2 && late > 0) blocks -= late;
        const double masked = causal ? (Nk < keys ? Nk : keys) / 32.0 * passes : 0;
        return rounds * ((blocks * block_us + masked * masked_us) * (H / Hkv) + passes * pass_us);
    };
    return us(256, 1.85, 0, 7) < us(128, 1.07, 0.1, 4);
}

template <bool CAUSAL, bool TAIL, bool SPILL>
static hipError_t launch_dkdv_wide(const void* q, const void* k, const void* v, const void* d_o,
                                   const float* lse, const float* delta, void* dk, void* dv,
                                   int B, int H, int Hkv, int Nq, int Nk, float scale, hipStream_t stream, void* ds, int cus)
{
    using S = DkdvWideShape;
    const int num_kv_tiles = (Nk + S::kTileKV - 1) / S::kTileKV;
    const int units = CAUSAL ? (num_kv_tiles + 1) / 2 : num_kv_tiles;
    const int total_units = B * Hkv * units;
    const int grid = total_units < cus ? total_units : cus;
    hipLaunchKernelGGL((attn_bwd_dkdv_wide_kernel<CAUSAL, TAIL, SPILL>), dim3(grid), dim3(S::kThreads), 0, stream,
                       (const bf16*)q, (const bf16*)k, (const bf16*)v, (const bf16*)d_o, lse, delta,
                       (bf16*)dk, (bf16*)dv, Nq, Nk, num_kv_tiles, total_units, scale, H, Hkv, grid, (char*)ds, ds_query_blocks(Nq), units);
    return hipGetLastError();
}

template <int D, bool CAUSAL>
static hipError_t launch_dkdv_t(const void* q, const void* k, const void* v, const void* d_o,
                                const float* lse, const float* delta, void* dk, void* dv,
                                int B, int H, int Hkv, int Nq, int Nk, float scale, hipStream_t stream, void* ds,
                                int n_splits, int q_splits, float* part)
{
    using S = DkdvShape<D>;
    int cus = 0;
    hipError_t e = compute_unit_count(&cus);
    if (e != hipSuccess) return e;
    const int resident = cus * (D == 64 ? 2 : 1);               // as many workgroups as fit at once
    if (!part) n_splits = q_splits = 1;
    if constexpr (D == 128)
        if (!part && dkdv_wide_pays(B, H, Hkv, Nq, Nk, CAUSAL, cus)) {
            const bool tail = Nq != Nk || Nk % DkdvWideShape::kTileKV;
            auto launch = tail ? (ds ? launch_dkdv_wide<CAUSAL, true, true> : launch_dkdv_wide<CAUSAL, true, false>)
                               : (ds ? launch_dkdv_wide<CAUSAL, false, true> : launch_dkdv_wide<CAUSAL, false, false>);
            return launch(q, k, v, d_o, lse, delta, dk, dv, B, H, Hkv, Nq, Nk, scale, stream, ds, cus);
        }
    const bool paired = CAUSAL && pair_tiles((long long)B * Hkv * n_splits, (Nk + S::kTileKV - 1) / S::kTileKV, cus);
    const bool tail = Nq != Nk || Nk % S::kTileKV || paired != CAUSAL;
    auto launch = part ? (ds ? launch_dkdv_tt<D, CAUSAL, true, true, true> : launch_dkdv_tt<D, CAUSAL, true, false, true>)
                : tail ? (ds ? launch_dkdv_tt<D, CAUSAL, true, true, false> : launch_dkdv_tt<D, CAUSAL, true, false, false>)
                       : (ds ? launch_dkdv_tt<D, CAUSAL, false, true, false> : launch_dkdv_tt<D, CAUSAL, false, false, false>);
    return launch(q, k, v, d_o, lse, delta, dk, dv, B, H, Hkv, Nq, Nk, scale, stream, ds, resident, paired, n_splits, q_splits, part);
}

// ds != nullptr: the kernel also stores its dS blocks there (ds_spill_bytes(...) bytes) for launch_attn_bwd_dq_from_ds.
// part != nullptr: the queries are split n_splits ways (dkdv_splits()), partial sums in part.
hipError_t launch_attn_bwd_dkdv(const void* q, const void* k, const void* v, const void* d_o,
                                const float* lse, const float* delta, void* dk, void* dv,
                                int B, int H, int Hkv, int Nq, int Nk, int D, int causal, float scale, hipStream_t stream,
                                void* ds, int n_splits, int q_splits, float* part)
{
    auto launch = D == 128 ? (causal ? launch_dkdv_t<128, true> : launch_dkdv_t<128, false>)
                           : (causal ? launch_dkdv_t<64, true> : launch_dkdv_t<64, false>);
    return launch(q, k, v, d_o, lse, delta, dk, dv, B, H, Hkv, Nq, Nk, scale, stream, ds, n_splits, q_splits, part);
}

// ------------------------------------------------------------------------------------------
// kernel 3: dQ
// ------------------------------------------------------------------------------------------
template <int D>
struct DqShape {
    static constexpr int kWaves = 4;
    static constexpr int kThreads = 256;
    static constexpr int kTileQ = 128;                  // queries per workgroup (32 per wave)
    static constexpr int kTileKV = 64;                  // keys per LDS stage
    static constexpr int kRowBytes = D * 2;
    static constexpr int kChunksPerRow = D / 8;
    static constexpr int kTileBytes = kTileKV * kRowBytes;
    static constexpr int kStageBytes = 2 * kTileBytes;  // K tile then V tile
    static constexpr int kLoadsPerTile = kTileKV * kChunksPerRow / kThreads;   // per thread, per tensor
};

// FUSED: Delta is not an input: the kernel computes Delta_i = sum_d dO_id O_id for its own rows (a
// lane already holds its query's dO row), writes it to DeltaOut for the dK/dV kernel that follows,
// and uses it; the separate Delta pass over O and dO is then not needed.
template <int D, bool CAUSAL, bool TAIL, bool FUSED>
__global__ __launch_bounds__(256, 2)
void attn_bwd_dq_kernel(const bf16* __restrict__ Q, const bf16* __restrict__ K, const bf16* __restrict__ V,
                        const bf16* __restrict__ dO, const float* __restrict__ LSE, const float* __restrict__ Delta,
                        bf16* __restrict__ dQ, int Nq, int Nk, int num_q_tiles, int total_wg, float scale, int hq, int hkv,
                        const bf16* __restrict__ O, float* __restrict__ DeltaOut, int pair_tiles)
{
    using S = DqShape<D>;
    __shared__ __attribute__((aligned(1024))) char stage0[S::kStageBytes];
    __shared__ __attribute__((aligned(1024))) char stage1[S::kStageBytes];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int l32 = lane & 31;
    const int h = lane >> 5;

    // Work unit: one query tile, or, when causal, the pair (last - u, u): tile t streams the keys up
    // to its diagonal, so the pairs carry (nearly) the same work and the launch is balanced.
    // Nq queries, Nk keys; TAIL and the causal alignment as in the kernels above.
    const bool paired = CAUSAL && (!TAIL || pair_tiles);
    const int units = paired ? (num_q_tiles + 1) / 2 : num_q_tiles;
    const int logical = xcd_remap(blockIdx.x, total_wg);
    const int bh = logical / units;
    const int unit = logical % units;
    // grouped-query attention: query head h of a batch entry reads key/value head h / (hq / hkv)
    const size_t head = (size_t)bh * Nq * D;
    const size_t kv_head = (size_t)((bh / hq) * hkv + (bh % hq) / (hq / hkv)) * Nk * D;
    const int off = TAIL ? Nk - Nq : 0;          // causal: query i sees keys <= i + off
    const bf16* Kh = K + kv_head;
    const bf16* Vh = V + kv_head;
#pragma unroll 1
    for (int pass = 0; pass < (paired ? 2 : 1); pass++) {
    const int qt = pass == 0 ? num_q_tiles - 1 - unit : unit;
    if (pass == 1 && qt == num_q_tiles - 1 - unit) break;   // odd tile count: the middle tile has no partner
    const int q0 = qt * S::kTileQ + wave * 32;
    const int my_q = q0 + l32;
    // The lengths need not be multiples of the tile sizes: the kernel works on padded sequences,
    // reads of rows past the end are redirected to the last row, keys >= Nk are masked, query rows
    // >= Nq are not stored.
    const int my_q_ld = (!TAIL || my_q < Nq) ? my_q : Nq - 1;
    const float c = scale * kLog2e;

    // ---- Q_i, dO_i fragments (B operands of S^T = K Q^T and dP^T = V dO^T) and the row statistics
    bf16x8 qf[D / 16], dof[D / 16];
#pragma unroll
    for (int kb = 0; kb < D / 16; kb++) {
        qf[kb] = *(const bf16x8*)(Q + head + (size_t)my_q_ld * D + kb * 16 + h * 8);
        dof[kb] = *(const bf16x8*)(dO + head + (size_t)my_q_ld * D + kb * 16 + h * 8);
    }
    const float lse2 = LSE[(size_t)bh * Nq + my_q_ld] * kLog2e;
    float delta;
    if (FUSED) {
        float part = 0.f;       // this lane's half of the row (columns 16*kb + 8*h .. +7)
#pragma unroll
        for (int kb = 0; kb < D / 16; kb++) {
            const bf16x8 of = *(const bf16x8*)(O + head + (size_t)my_q_ld * D + kb * 16 + h * 8);
#pragma unroll
            for (int e = 0; e < 8; e++) part = __builtin_fmaf((float)of[e], (float)dof[kb][e], part);
        }
        delta = half_sum(part);
        if (h == 0 && (!TAIL || my_q < Nq)) DeltaOut[(size_t)bh * Nq + my_q] = delta;
    } else {
        delta = Delta[(size_t)bh * Nq + my_q_ld];
    }

    // ---- direct-to-LDS tile loads (same slot arithmetic as the forward kernel)
    int kv_src[S::kLoadsPerTile];
#pragma unroll
    for (int it = 0; it < S::kLoadsPerTile; it++) {
        int s = it * S::kThreads + tid;
        int row = s / S::kChunksPerRow, pc = s % S::kChunksPerRow;
        kv_src[it] = row * D + ((pc ^ swz<D>(row)) * 8);
    }
    auto issue_tile = [&](char* base, int tile) {
        const int j0 = tile * S::kTileKV;
        const bf16* kt = Kh + (size_t)j0 * D;
        const bf16* vt = Vh + (size_t)j0 * D;
        if (!TAIL || j0 + S::kTileKV <= Nk) {
#pragma unroll
            for (int it = 0; it < S::kLoadsPerTile; it++)
                load_global_to_lds16(kt + kv_src[it], base + wave * 1024 + it * (S::kThreads * 16));
#pragma unroll
            for (int it = 0; it < S::kLoadsPerTile; it++)
                load_global_to_lds16(vt + kv_src[it], base + S::kTileBytes + wave * 1024 + it * (S::kThreads * 16));
        } else {
            // the tile runs past the last key: rows >= Nk fetch row Nk-1 instead (they are masked later)
#pragma unroll
            for (int it = 0; it < S::kLoadsPerTile; it++) {
                const int row = j0 + (it * S::kThreads + tid) / S::kChunksPerRow;
                const int back = (row < Nk ? 0 : row - (Nk - 1)) * D;   // elements to step back
                load_global_to_lds16(kt + kv_src[it] - back, base + wave * 1024 + it * (S::kThreads * 16));
                load_global_to_lds16(vt + kv_src[it] - back, base + S::kTileBytes + wave * 1024 + it * (S::kThreads * 16));
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    // ---- per-lane LDS offsets
    // row operand (A of S^T and dP^T): row 32b + l32, logical chunk 2*kb + h
    const int row_lane = l32 * S::kRowBytes + ((h ^ swz<D>(l32)) << 4);
    // transposed operand from the K tile (A of dQ^T = K^T dS^T): rows 16*kk + 4h + j16/4 (+8)
    const int j16 = lane & 15;
    const int tr_row = 4 * h + (j16 >> 2);
    const int tr_lane = tr_row * S::kRowBytes + (((2 * ((lane >> 4) & 1) + ((j16 & 3) >> 1)) ^ swz<D>(tr_row)) << 4) + ((j16 & 1) << 3);

    f32x16 dq_acc[D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; db++)
#pragma unroll
        for (int r = 0; r < 16; r++) dq_acc[db][r] = 0.f;

    // dP - Delta: the products of dO and V start from -Delta, as in the dK/dV kernel, which takes a subtraction from each of the
    // elements that the vector ALU works on.  This kernel, us: B16 H16 N4096 causal D128 1559, 1520, D64 842, 800; B2 Hq16 Hkv4 N1001 D64
    // 20.7, 20.2.
    f32x16 minus_delta;
#pragma unroll
    for (int r = 0; r < 16; r++) minus_delta[r] = -delta;
    asm volatile("" : "+v"(minus_delta));        // (sixteen registers; the compiler would fill them again for every block)

    auto compute_tile = [&](const char* ks, int tile) {
        const int j0 = tile * S::kTileKV;
        if (CAUSAL && j0 > q0 + 31 + off) return;    // every key of the tile is masked for this wave
        const char* vs = ks + S::kTileBytes;
        // the tile crosses this wave's diagonal, or runs past the last key
        const bool diag = (CAUSAL && (j0 + S::kTileKV - 1 > q0 + off)) || (TAIL && j0 + S::kTileKV > Nk);
        // The tile is processed in two halves of 32 keys, so that only one half's S^T / dP^T
        // accumulators are live at a time.
#pragma unroll
        for (int b = 0; b < 2; b++) {
            f32x16 s, dp;
#pragma unroll
            for (int r = 0; r < 16; r++) s[r] = 0.f;
#pragma unroll
            for (int kb = 0; kb < D / 16; kb++) {
                const int off = (row_lane ^ ((2 * kb) << 4)) + b * 32 * S::kRowBytes;
                s = mfma32(lds_read_b128(ks, off), qf[kb], s);
                dp = mfma32(lds_read_b128(vs, off), dof[kb], kb == 0 ? minus_delta : dp);
            }
            // P^T and dS^T: lane <-> query my_q, register r <-> key j0 + 32b + 8*(r/4) + 4h + r%4.
            // Only a tile on the diagonal needs the mask: it pushes the masked scores to -inf in a
            // branch of its own (P = 2^-inf = 0), so the common case carries no compare / select.
            if (diag) {
#pragma unroll
                for (int r = 0; r < 16; r++) {
                    const int key = j0 + 32 * b + 8 * (r >> 2) + 4 * h + (r & 3);
                    if ((CAUSAL && key > my_q + off) || (TAIL && key >= Nk)) s[r] = -INFINITY;
                }
            }
#pragma unroll
            for (int r = 0; r < 16; r++) {
                const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], c, -lse2));
                s[r] = p * dp[r];
            }
            // dQ^T += K^T dS^T, 16 keys per MFMA
#pragma unroll
            for (int k2 = 0; k2 < 2; k2++) {
                const int kk = 2 * b + k2, r0 = 8 * k2;
                bf16x8 dsb = cvt8(s[r0 + 0], s[r0 + 1], s[r0 + 2], s[r0 + 3],
                                  s[r0 + 4], s[r0 + 5], s[r0 + 6], s[r0 + 7]);
#pragma unroll
                for (int db = 0; db < D / 32; db++) {
                    const int row_off = 16 * kk * S::kRowBytes;
                    const int x0 = (4 * db) << 4, x1 = ((4 * db) ^ 2) << 4;
                    bf16x4 a0 = lds_read_tr16(ks, (tr_lane ^ x0) + row_off);
                    bf16x4 a1 = lds_read_tr16(ks, (tr_lane ^ x1) + row_off + 8 * S::kRowBytes);
                    dq_acc[db] = mfma32(concat(a0, a1), dsb, dq_acc[db]);
                }
            }
        }
    };

    // key tiles this workgroup visits: an even count that covers every key visible to its last query
    int n_tiles;
    if (!TAIL) {
        n_tiles = (CAUSAL ? qt * S::kTileQ + S::kTileQ : num_q_tiles * S::kTileQ) / S::kTileKV;
    } else {
        int n_keys = Nk;
        if (CAUSAL && qt * S::kTileQ + S::kTileQ + off < n_keys) n_keys = qt * S::kTileQ + S::kTileQ + off;
        n_tiles = 2 * ((n_keys + 2 * S::kTileKV - 1) / (2 * S::kTileKV));
    }
    int t_begin = 0;
    // A start the compiler does not know keeps the tile's address scalar (otherwise a 64-bit vector addition per load and
    // tile).  This kernel, us: B16 H16 N4096 causal D64 848, 830, D128 1600, 1548; N2000 D64 264, 246.
    asm volatile("" : "+s"(t_begin));
    issue_tile(stage0, t_begin);
    wait_vmcnt<0>();
    __syncthreads();
    for (int t = t_begin; t < n_tiles; t += 2) {
        issue_tile(stage1, t + 1);
        compute_tile(stage0, t);
        wait_vmcnt<0>();
        __syncthreads();
        if (t + 2 < n_tiles) issue_tile(stage0, t + 2);
        compute_tile(stage1, t + 1);
        wait_vmcnt<0>();
        __syncthreads();
    }

    // ---- epilogue: dQ = scale * acc; lane <-> query, register r of block db <-> column 32db + 8*(r/4) + 4h + r%4
    if (!TAIL || my_q < Nq) {
        bf16* dQr = dQ + head + (size_t)my_q * D;
#pragma unroll
        for (int db = 0; db < D / 32; db++)
#pragma unroll
            for (int g = 0; g < 4; g++) {
                bf16x2 lo = cvt2(dq_acc[db][4 * g + 0] * scale, dq_acc[db][4 * g + 1] * scale);
                bf16x2 hi = cvt2(dq_acc[db][4 * g + 2] * scale, dq_acc[db][4 * g + 3] * scale);
                *(bf16x4*)(dQr + 32 * db + 8 * g + 4 * h) = __builtin_shufflevector(lo, hi, 0, 1, 2, 3);
            }
    }
    }   // pass (the loop above ends with a barrier, so both stages are free again)
}

template <int D, bool CAUSAL, bool TAIL, bool FUSED>
static hipError_t launch_dq_tt(const void* q, const void* k, const void* v, const void* d_o,
                               const float* lse, const float* delta, void* dq,
                               int B, int H, int Hkv, int Nq, int Nk, float scale, hipStream_t stream,
                               const void* o, float* delta_out, bool paired)
{
    using S = DqShape<D>;
    const int num_q_tiles = (Nq + S::kTileQ - 1) / S::kTileQ;
    const int total = B * H * (paired ? (num_q_tiles + 1) / 2 : num_q_tiles);
    hipLaunchKernelGGL((attn_bwd_dq_kernel<D, CAUSAL, TAIL, FUSED>), dim3(total), dim3(S::kThreads), 0, stream,
                       (const bf16*)q, (const bf16*)k, (const bf16*)v, (const bf16*)d_o, lse, delta,
                       (bf16*)dq, Nq, Nk, num_q_tiles, total, scale, H, Hkv, (const bf16*)o, delta_out, paired);
    return hipGetLastError();
}

template <int D, bool CAUSAL>
static hipError_t launch_dq_t(const void* q, const void* k, const void* v, const void* d_o,
                              const float* lse, const float* delta, void* dq,
                              int B, int H, int Hkv, int Nq, int Nk, float scale, hipStream_t stream,
                              const void* o, float* delta_out)
{
    using S = DqShape<D>;
    int cus = 0;
    hipError_t e = compute_unit_count(&cus);
    if (e != hipSuccess) return e;
    const bool paired = CAUSAL && pair_tiles((long long)B * H, (Nq + S::kTileQ - 1) / S::kTileQ, cus);
    const bool tail = Nq != Nk || Nq % S::kTileQ || paired != CAUSAL;
    auto launch = o ? (tail ? launch_dq_tt<D, CAUSAL, true, true> : launch_dq_tt<D, CAUSAL, false, true>)
                    : (tail ? launch_dq_tt<D, CAUSAL, true, false> : launch_dq_tt<D, CAUSAL, false, false>);
    return launch(q, k, v, d_o, lse, delta, dq, B, H, Hkv, Nq, Nk, scale, stream, o, delta_out, paired);
}

// o != nullptr: Delta is computed from o and d_o inside the kernel and written to delta_out (delta is not read).
hipError_t launch_attn_bwd_dq(const void* q, const void* k, const void* v, const void* d_o,
                              const float* lse, const float* delta, void* dq,
                              int B, int H, int Hkv, int Nq, int Nk, int D, int causal, float scale, hipStream_t stream,
                              const void* o, float* delta_out)
{
    if (D == 128) return causal ? launch_dq_t<128, true>(q, k, v, d_o, lse, delta, dq, B, H, Hkv, Nq, Nk, scale, stream, o, delta_out)
                                : launch_dq_t<128, false>(q, k, v, d_o, lse, delta, dq, B, H, Hkv, Nq, Nk, scale, stream, o, delta_out);
    return causal ? launch_dq_t<64, true>(q, k, v, d_o, lse, delta, dq, B, H, Hkv, Nq, Nk, scale, stream, o, delta_out)
                  : launch_dq_t<64, false>(q, k, v, d_o, lse, delta, dq, B, H, Hkv, Nq, Nk, scale, stream, o, delta_out);
}

// ------------------------------------------------------------------------------------------
// kernel 4: dQ from the dS blocks that kernel 2 stored
// ------------------------------------------------------------------------------------------
template <int D, int WAVES>
struct DqDsShape {
    static constexpr int kWaves = WAVES;
    static constexpr int kThreads = 64 * kWaves;
    static constexpr int kTileQ = 32 * kWaves;          // queries per workgroup (32 per wave)
    static constexpr int kTileKV = 64;                  // keys per step
    static constexpr int kRowBytes = D * 2;
    static constexpr int kChunksPerRow = D / 8;
    static constexpr int kKTileBytes = kTileKV * kRowBytes;
    static constexpr int kKStages = 4;                  // ring of K tiles, filled three tiles ahead
    static constexpr int kDsTileBytes = 2 * 2048;       // the two 32-key blocks of one wave and one step
    static constexpr int kDsAhead = 4;                  // dS tiles held in registers ahead of their use
    static constexpr int kKLoads = kTileKV * kChunksPerRow / kThreads;   // per thread and tile
    static constexpr int kDsLoads = kDsTileBytes / 1024;                  // per lane and tile
    static constexpr int kLdsBytes = kKStages * kKTileBytes + kWaves * 2 * kDsTileBytes;
    // vector-memory operations a wave issues per step, and how many of them are younger than the K tile
    // that must have landed at the end of a step (see the loop)
    static constexpr int kOpsPerStep = kKLoads + kDsLoads;
    static constexpr int kWaitCount = kDsLoads + 2 * kOpsPerStep;
};

// 16 bytes per lane from global memory into registers, issued through inline assembly so that the
// compiler does not place a wait of its own before the first use: the data is only touched after the
// loop's own wait (wait_vmcnt<>) and a claim_loaded() on the registers.
__device__ __forceinline__ void load16_untracked(bf16x8& dst, const void* gptr) {
    asm volatile("global_load_dwordx4 %0, %1, off" : "=v"(dst) : "v"(gptr) : "memory");
}
__device__ __forceinline__ void claim_loaded(bf16x8& r) { asm volatile("" : "+v"(r) : : "memory"); }

// dQ_i = scale * sum_j dS_ij K_j: one workgroup per 256-query tile (causal: balanced pairs of tiles), wave w
// owns queries 32w..32w+31 and keeps dQ^T in registers while the workgroup walks 64-key tiles.  The kernel is
// bound by reading dS (2 bytes per query-key pair) from HBM, so everything is arranged around keeping many
// bytes in flight: each wave loads its own dS blocks into registers four steps ahead (they are private to the
// wave: no barrier is involved), K tiles go to a four-stage LDS ring by direct loads three steps ahead, and
// the single wait per step is for a K tile that is older than three steps' worth of dS loads (the counter
// retires in issue order), so those stay in flight across the barrier.
// dQ^T += K^T dS^T needs dS^T with the QUERY on lanes, and the stored blocks have the KEY on lanes: a wave
// writes the block it is about to use into a private LDS buffer, the 16-byte piece of (key, half, h) at
// (key * 4 + half * 2 + h) * 16, and takes the operand out with transposing reads (4 keys x 4 query quads per
// 16 lanes: every bank once).  No mask code: kernel 2 stored zeros for masked pairs, padding queries and
// padding keys; a wave does not compute on tiles that lie wholly beyond its diagonal, which kernel 2 may not
// have written: its loads of such tiles are redirected to its last real tile.
//
// Four waves instead of eight (a tile of 128 queries) where the launch then still fits the compute units at once:
// the time of a step on a compute unit is that of its waves' LDS reads.  Whole backward, causal D128: B2 Hq16 Hkv4
// N1001 112 -> 100 us, B1 H16 N4096 269 -> 248, B4 H16 N1024 99 -> 91.
template <int D, bool CAUSAL, bool TAIL, int WAVES>
__global__ __launch_bounds__(64 * WAVES, 1)
void attn_bwd_dq_from_ds_kernel(const bf16* __restrict__ K, const char* __restrict__ DS, bf16* __restrict__ dQ,
                                int Nq, int Nk, int num_q_tiles, int total_wg, float scale, int hq, int hkv,
                                int num_kv_tiles, int n_qb, int pair_tiles)
{
    using S = DqDsShape<D, WAVES>;
    __shared__ __attribute__((aligned(1024))) char smem[S::kLdsBytes];
    char* const kring = smem;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int l32 = lane & 31;
    const int h = lane >> 5;
    char* const dsbuf = smem + S::kKStages * S::kKTileBytes + wave * (2 * S::kDsTileBytes);   // two buffers of this wave

    const bool paired = CAUSAL && (!TAIL || pair_tiles);
    const int units = paired ? (num_q_tiles + 1) / 2 : num_q_tiles;
    const int logical = xcd_remap(blockIdx.x, total_wg);
    const int bh = logical / units;                  // query head
    const int unit = logical % units;
    const size_t head = (size_t)bh * Nq * D;
    const size_t kv_head = (size_t)((bh / hq) * hkv + (bh % hq) / (hq / hkv)) * Nk * D;
    const int off = TAIL ? Nk - Nq : 0;              // causal: query i sees keys <= i + off
    const bf16* Kh = K + kv_head;
    const char* DSh = DS + (size_t)bh * num_kv_tiles * n_qb * 8192;

    // K tile loads: slot arithmetic of the other kernels
    int k_src[S::kKLoads];
#pragma unroll
    for (int it = 0; it < S::kKLoads; it++) {
        int s = it * S::kThreads + tid;
        int row = s / S::kChunksPerRow, pc = s % S::kChunksPerRow;
        k_src[it] = row * D + ((pc ^ swz<D>(row)) * 8);
    }
    // where this lane's 16-byte piece of a stored half-block goes in the wave's LDS buffer (half s adds 32)
    const int piece_off = (l32 * 4 + h) * 16;
    // transposed operand from the K tile (A of dQ^T = K^T dS^T): rows 16*kk + 4h + j16/4 (+8)
    const int j16 = lane & 15;
    const int tr_row = 4 * h + (j16 >> 2);
    const int tr_lane = tr_row * S::kRowBytes + (((2 * ((lane >> 4) & 1) + ((j16 & 3) >> 1)) ^ swz<D>(tr_row)) << 4) + ((j16 & 1) << 3);
    // dS^T operand (B): 16-lane group G = lane / 16 covers queries 16 * (G % 2) .. + 15 (= half G % 2 of the
    // block) and keys 4 * (G / 2) + j16 / 4 (+ 8) of a 16-key step; lane j of the group points at the query
    // quad j % 4, i.e. (h = quad % 2, g = quad / 2) of the stored layout
    const int ds_lane = (4 * h + (j16 >> 2)) * 64 + ((lane >> 4) & 1) * 32 + (j16 & 1) * 16 + ((j16 & 3) >> 1) * 8;

#pragma unroll 1
    for (int pass = 0; pass < (paired ? 2 : 1); pass++) {
    const int qt = pass == 0 ? num_q_tiles - 1 - unit : unit;
    if (pass == 1 && qt == num_q_tiles - 1 - unit) break;   // odd tile count: the middle tile has no partner
    const int q0 = qt * S::kTileQ + wave * 32;
    const int my_q = q0 + l32;
    const int qb = qt * (S::kTileQ / 32) + wave;     // this wave's query block

    // 64-key tiles the workgroup walks (every key visible to its last query), rounded up to the unroll of the loop
    int n_tiles;
    if (!TAIL) {
        n_tiles = (CAUSAL ? qt * S::kTileQ + S::kTileQ : Nk) / S::kTileKV;
    } else {
        int n_keys = Nk;
        if (CAUSAL && qt * S::kTileQ + S::kTileQ + off < n_keys) n_keys = qt * S::kTileQ + S::kTileQ + off;
        n_tiles = 2 * ((n_keys + 2 * S::kTileKV - 1) / (2 * S::kTileKV));
    }
    const int n_steps = (n_tiles + 3) & ~3;
    // the last tile this wave computes on; -1: none (a wave of padding rows)
    int last_tile = n_tiles - 1;
    if (CAUSAL) { const int d = (q0 + 31 + off) / S::kTileKV; if (d < last_tile) last_tile = d; }
    if (TAIL && q0 >= Nq) last_tile = -1;
    // block (key tile 0, query block 0) of the head is always written: the stand-in for a wave without tiles
    const char* ds_row = last_tile >= 0 ? DSh + (size_t)qb * 8192 : DSh;

    auto issue_k = [&](int tile) {                   // into ring stage tile % 4
        char* base = kring + (tile & (S::kKStages - 1)) * S::kKTileBytes + wave * 1024;
        if (tile > n_tiles - 1) tile = n_tiles - 1;  // (beyond the walk: the last tile again, into a stage nobody reads any more)
        const int j0 = tile * S::kTileKV;
        const bf16* kt = Kh + (size_t)j0 * D;
#pragma unroll
        for (int it = 0; it < S::kKLoads; it++) {
            int back = 0;
            if (TAIL) {                              // rows >= Nk fetch row Nk-1 (their dS is 0)
                const int row = j0 + (it * S::kThreads + tid) / S::kChunksPerRow;
                back = (row < Nk ? 0 : row - (Nk - 1)) * D;
            }
            load_global_to_lds16_untracked(kt + k_src[it] - back, base + it * (S::kThreads * 16));
        }
    };
    // the two 32-key blocks of step `tile` for this wave's queries: blocks 2*(tile%2), +1 of key tile tile/2
    auto issue_ds = [&](bf16x8 (&r)[4], int tile) {
        if (tile > last_tile) tile = last_tile < 0 ? 0 : last_tile;
        const char* blk = ds_row + ((size_t)(tile >> 1) * n_qb * 4 + 2 * (tile & 1)) * 2048 + lane * 16;
#pragma unroll
        for (int n = 0; n < 4; n++) load16_untracked(r[n], blk + n * 1024);
    };

    f32x16 dq_acc[D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; db++)
#pragma unroll
        for (int r = 0; r < 16; r++) dq_acc[db][r] = 0.f;

    auto compute_tile = [&](const char* ks, const char* dss) {
#pragma unroll
        for (int kk = 0; kk < 4; kk++) {             // 16 keys per step
            const int ds_off = (kk >> 1) * 2048 + (kk & 1) * 1024;
            bf16x4 b0 = lds_read_tr16(dss, ds_lane + ds_off);
            bf16x4 b1 = lds_read_tr16(dss, ds_lane + ds_off + 512);
            const bf16x8 dsb = concat(b0, b1);
#pragma unroll
            for (int db = 0; db < D / 32; db++) {
                const int row_off = 16 * kk * S::kRowBytes;
                const int x0 = (4 * db) << 4, x1 = ((4 * db) ^ 2) << 4;
                bf16x4 a0 = lds_read_tr16(ks, (tr_lane ^ x0) + row_off);
                bf16x4 a1 = lds_read_tr16(ks, (tr_lane ^ x1) + row_off + 8 * S::kRowBytes);
                dq_acc[db] = mfma32(concat(a0, a1), dsb, dq_acc[db]);
            }
        }
    };

    // One step.  Issue order inside a step: the K tile three steps ahead, then the dS tile four steps ahead.
    // At the end of step t the K tile of step t+1 must have landed; younger than it are the dS loads of its own
    // step and everything of the two steps since: kWaitCount operations, which stay in flight.
    bf16x8 set0[4], set1[4], set2[4], set3[4];
    auto step = [&](bf16x8 (&r)[4], int t) {
        char* dss = dsbuf + (t & 1) * S::kDsTileBytes;
#pragma unroll
        for (int n = 0; n < 4; n++) claim_loaded(r[n]);
        // piece (block c = n / 2, half s = n % 2) of this lane -> its transposable place
#pragma unroll
        for (int n = 0; n < 4; n++) *(bf16x8*)(dss + (n >> 1) * 2048 + (n & 1) * 32 + piece_off) = r[n];
        issue_k(t + 3);
        issue_ds(r, t + 4);
        __builtin_amdgcn_sched_barrier(0);
        if (t <= last_tile) compute_tile(kring + (t & (S::kKStages - 1)) * S::kKTileBytes, dss);
        __builtin_amdgcn_sched_barrier(0);
        wait_vmcnt_lds_done<S::kWaitCount>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };

    // prologue in the loop's own issue order (steps -4 .. -1 without their computation)
    issue_ds(set0, 0);
    issue_k(0); issue_ds(set1, 1);
    issue_k(1); issue_ds(set2, 2);
    issue_k(2); issue_ds(set3, 3);
    wait_vmcnt<S::kWaitCount>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll 1
    for (int t = 0; t < n_steps; t += 4) {
        step(set0, t);
        step(set1, t + 1);
        step(set2, t + 2);
        step(set3, t + 3);
    }
    wait_vmcnt<0>();          // the redirected loads of the last steps must not outlive this pass (LDS, registers)
    // Nobody uses what the last of them bring, but their registers have to stay taken until they are here: the compiler
    // would give them to the epilogue's row numbers and accumulators, which a late load then overwrites.
#pragma unroll
    for (int n = 0; n < 4; n++) { claim_loaded(set0[n]); claim_loaded(set1[n]); claim_loaded(set2[n]); claim_loaded(set3[n]); }
    __builtin_amdgcn_s_barrier();

    if (!TAIL || my_q < Nq) {
        bf16* dQr = dQ + head + (size_t)my_q * D;
#pragma unroll
        for (int db = 0; db < D / 32; db++)
#pragma unroll
            for (int g = 0; g < 4; g++) {
                bf16x2 lo = cvt2(dq_acc[db][4 * g + 0] * scale, dq_acc[db][4 * g + 1] * scale);
                bf16x2 hi = cvt2(dq_acc[db][4 * g + 2] * scale, dq_acc[db][4 * g + 3] * scale);
                *(bf16x4*)(dQr + 32 * db + 8 * g + 4 * h) = __builtin_shufflevector(lo, hi, 0, 1, 2, 3);
            }
    }
    }   // pass
}

template <int D, bool CAUSAL, bool TAIL, int WAVES>
static hipError_t launch_dq_from_ds_tt(const void* k, const void* ds, void* dq,
                                       int B, int H, int Hkv, int Nq, int Nk, float scale, hipStream_t stream, bool paired)
{
    using S = DqDsShape<D, WAVES>;
    auto kern = attn_bwd_dq_from_ds_kernel<D, CAUSAL, TAIL, WAVES>;
    const int num_q_tiles = (Nq + S::kTileQ - 1) / S::kTileQ;
    const int num_kv_tiles = (Nk + 127) / 128;
    const int total = B * H * (paired ? (num_q_tiles + 1) / 2 : num_q_tiles);
    hipLaunchKernelGGL(kern, dim3(total), dim3(S::kThreads), 0, stream,
                       (const bf16*)k, (const char*)ds, (bf16*)dq, Nq, Nk, num_q_tiles, total, scale, H, Hkv,
                       num_kv_tiles, ds_query_blocks(Nq), paired);
    return hipGetLastError();
}

template <int D, bool CAUSAL>
static hipError_t launch_dq_from_ds_t(const void* k, const void* ds, void* dq,
                                      int B, int H, int Hkv, int Nq, int Nk, float scale, hipStream_t stream)
{
    int cus = 0;
    hipError_t e = compute_unit_count(&cus);
    if (e != hipSuccess) return e;
    const int tiles = (Nq + 127) / 128;
    const long long small = (long long)B * H * (CAUSAL ? (tiles + 1) / 2 : tiles);      // workgroups of four waves
    auto launch = small <= cus               ? launch_dq_from_ds_tt<D, CAUSAL, true, 4>
                : (Nq != Nk || Nq % 256) ? launch_dq_from_ds_tt<D, CAUSAL, true, 8> : launch_dq_from_ds_tt<D, CAUSAL, false, 8>;
    return launch(k, ds, dq, B, H, Hkv, Nq, Nk, scale, stream, CAUSAL && (small > cus || pair_tiles((long long)B * H, tiles, cus)));
}

hipError_t launch_attn_bwd_dq_from_ds(const void* k, const void* ds, void* dq,
                                      int B, int H, int Hkv, int Nq, int Nk, int D, int causal, float scale, hipStream_t stream)
{
    auto launch = D == 128 ? (causal ? launch_dq_from_ds_t<128, true> : launch_dq_from_ds_t<128, false>)
                           : (causal ? launch_dq_from_ds_t<64, true> : launch_dq_from_ds_t<64, false>);
    return launch(k, ds, dq, B, H, Hkv, Nq, Nk, scale, stream);
}

}  // namespace tk
