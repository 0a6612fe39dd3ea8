// Fused exact softmax attention, forward pass, for gfx950 (MI355X).
//
// Two kernels do the same computation: attn_fwd_kernel, for few query rows per head, for decoding and for one or two key tiles at
// D = 64, and attn_fwd_phase_kernel for all other calls, which puts the work of a tile in two phases (described there).
// In both a wave owns 32 query rows of one (batch, head), and a workgroup of 4 waves 128 (8 waves and 256 in one form of the
// phase kernel).  K and V are streamed in tiles of 64 keys through an LDS ring filled by direct
// global->LDS loads.  Per tile each wave computes, with v_mfma_f32_32x32x16_bf16:
//
//   S^T = K Q^T          (so that a lane owns ONE query: softmax statistics are lane-local)
//   online softmax in base 2 with the temperature folded into the exponent
//                        (the streaming recurrence of the paper's Appendix B.3 listing)
//   O^T += V^T P^T       (P^T in accumulator layout IS a valid B operand; V^T comes from
//                         row-major V in LDS through transposing reads)
//
// Epilogue: O = O / l -> bf16, LSE = m*scale + ln l.
#include "tk_common.h"
#include "tk_launch.h"

#include <math.h>

namespace tk {

template <int D>
struct FwdShape {
    static constexpr int kWaves = 4;
    static constexpr int kThreads = kWaves * 64;
    static constexpr int kTileQ = kWaves * 32;          // query rows per workgroup
    static constexpr int kTileKV = 64;                  // keys per LDS stage
    static constexpr int kRowBytes = D * 2;
    static constexpr int kChunksPerRow = D / 8;         // 16-byte chunks
    static constexpr int kTileBytes = kTileKV * kRowBytes;
    static constexpr int kStageBytes = 2 * kTileBytes;  // K tile then V tile
    static constexpr int kLdsBytes = 2 * kStageBytes;
    static constexpr int kLoadsPerTile = kTileKV * kChunksPerRow / kThreads;  // per thread
};

// LDS layout of a [64 x D] bf16 tile: row-major, with the 16-byte chunk index XOR-ed by a
// function of the row so that the two read patterns below spread over all 64 banks.
//   K tile, read as MFMA A operand: 16 consecutive lanes read the same chunk of 16 consecutive rows.
//   V tile, read through ds_read_b64_tr_b16: 32 lanes read a 4-row x 64-byte block.
template <int D> __device__ __forceinline__ int swizzle_k(int row) {
    return D == 128 ? (row & 15) : ((row >> 1) & 7);
}
template <int D> __device__ __forceinline__ int swizzle_v(int row) {
    return D == 128 ? (((row & 3) << 2) | ((row >> 2) & 3)) : ((((row >> 1) & 1) << 2) | ((row >> 2) & 3));
}

// Nq queries, Nk keys.  TAIL: the general case (Nq != Nk, or a length that is not a multiple of
// 128); the aligned square case compiles without any of the tail code.  With the causal mask the
// sequences are aligned at their ends: query i sees keys j <= i + (Nk - Nq); the host has checked
// Nq <= Nk for that case, so every query sees key 0.
//
// SPLIT (implies TAIL): n_splits workgroups share one query tile, each takes tiles_per_split (even)
// consecutive key tiles and leaves a normalised fp32 partial O and its LSE for the merge kernel below.  For
// calls whose heads and query tiles alone cannot fill the chip: decoding, a chunk of a prompt against a long history.
template <int D, bool CAUSAL, bool TAIL, bool SPLIT>
__global__ __launch_bounds__(256, 2)
void attn_fwd_kernel(const bf16* __restrict__ Q, const bf16* __restrict__ K, const bf16* __restrict__ V,
                     bf16* __restrict__ O, float* __restrict__ LSE,
                     int Nq, int Nk, int num_q_tiles, int heads, int head_group, float scale, int hq, int hkv,
                     int n_splits, int tiles_per_split, float* __restrict__ O_part, float* __restrict__ LSE_part)
{
    using S = FwdShape<D>;
    // One array per ring stage: distinct LDS objects let the compiler see that reads of the stage
    // being consumed cannot alias the direct-to-LDS loads in flight into the other stage (otherwise
    // it drains every outstanding load before the first LDS read that follows them).
    __shared__ __attribute__((aligned(1024))) char smem0[S::kStageBytes];
    __shared__ __attribute__((aligned(1024))) char smem1[S::kStageBytes];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int l32 = lane & 31;
    const int h = lane >> 5;

    int bh, qt, split = 0;
    if (SPLIT) split_of(blockIdx.x, gridDim.x, hq / hkv, num_q_tiles, n_splits, bh, split, qt);
    else if (CAUSAL) tile_of(blockIdx.x, heads, num_q_tiles, head_group, bh, qt);
    else {              // all tiles weigh the same: head after head, contiguous on an XCD
        const int id = xcd_remap(blockIdx.x, gridDim.x);
        bh = id / num_q_tiles;
        qt = id - bh * num_q_tiles;
    }

    // grouped-query attention: query head h of a batch entry reads key/value head h / (hq / hkv)
    const size_t head = (size_t)bh * Nq * D;
    const size_t kv_head = (size_t)((bh / hq) * hkv + (bh % hq) / (hq / hkv)) * Nk * D;
    const bf16* Qh = Q + head;
    const bf16* Kh = K + kv_head;
    const bf16* Vh = V + kv_head;
    const int q0 = qt * S::kTileQ + wave * 32;   // first query row of this wave
    const int my_q = q0 + l32;
    // The lengths need not be multiples of the tile sizes: the kernel works on padded sequences,
    // reads of rows past the end are redirected to the last row, keys >= Nk are masked, query rows
    // >= Nq are not stored.
    const int my_q_ld = (!TAIL || my_q < Nq) ? my_q : Nq - 1;
    const int off = TAIL ? Nk - Nq : 0;          // causal: query i sees keys <= i + off

    const float c = scale * kLog2e;              // base-2 temperature

    // ---- Q fragments (B operand of S^T = K Q^T): lane holds Q[my_q][16*kb + 8*h .. +7]
    bf16x8 qf[D / 16];
#pragma unroll
    for (int kb = 0; kb < D / 16; kb++)
        qf[kb] = *(const bf16x8*)(Qh + (size_t)my_q_ld * D + kb * 16 + h * 8);

    // ---- per-thread source offsets of the direct-to-LDS tile loads
    // LDS slot s = it*256 + tid holds (row = s / chunks_per_row, physical chunk = s % chunks_per_row).
    int k_src[S::kLoadsPerTile], v_src[S::kLoadsPerTile];
#pragma unroll
    for (int it = 0; it < S::kLoadsPerTile; it++) {
        int s = it * S::kThreads + tid;
        int row = s / S::kChunksPerRow, pc = s % S::kChunksPerRow;
        k_src[it] = row * D + ((pc ^ swizzle_k<D>(row)) * 8);
        v_src[it] = row * D + ((pc ^ swizzle_v<D>(row)) * 8);
    }
    auto issue_tile = [&](int stage, int tile) {
        const int j0 = tile * S::kTileKV;
        const bf16* kt = Kh + (size_t)j0 * D;
        const bf16* vt = Vh + (size_t)j0 * D;
        char* base = (stage ? smem1 : smem0) + wave * 1024;
        if (!TAIL || j0 + S::kTileKV <= Nk) {
#pragma unroll
            for (int it = 0; it < S::kLoadsPerTile; it++)
                load_global_to_lds16(kt + k_src[it], base + it * (S::kThreads * 16));
#pragma unroll
            for (int it = 0; it < S::kLoadsPerTile; it++)
                load_global_to_lds16(vt + v_src[it], base + S::kTileBytes + it * (S::kThreads * 16));
        } else {
            // the tile runs past the last key: rows >= Nk fetch row Nk-1 instead (they are masked later)
#pragma unroll
            for (int it = 0; it < S::kLoadsPerTile; it++) {
                const int row = j0 + (it * S::kThreads + tid) / S::kChunksPerRow;
                const int back = (row < Nk ? 0 : row - (Nk - 1)) * D;     // elements to step back
                load_global_to_lds16(kt + k_src[it] - back, base + it * (S::kThreads * 16));
            }
#pragma unroll
            for (int it = 0; it < S::kLoadsPerTile; it++) {
                const int row = j0 + (it * S::kThreads + tid) / S::kChunksPerRow;
                const int back = (row < Nk ? 0 : row - (Nk - 1)) * D;
                load_global_to_lds16(vt + v_src[it] - back, base + S::kTileBytes + it * (S::kThreads * 16));
            }
        }
        __builtin_amdgcn_sched_barrier(0);   // keep the prefetch ahead of the math it overlaps with
    };

    // ---- per-lane LDS read offsets (the XOR with a compile-time chunk index is applied at use)
    // K: row = 32*b + l32, logical chunk 2*kb + h
    const int k_lane = l32 * S::kRowBytes + ((h ^ swizzle_k<D>(l32)) << 4);
    // V (transposing read): 16-lane group G = lane/16 -> (d half = G%2, key half = G/2);
    //   lane j of the group addresses row 4*(G/2) + j/4, columns 32*db + 16*(G%2) + 4*(j%4)
    const int j16 = lane & 15;
    const int v_row = 4 * h + (j16 >> 2);
    const int v_chunk = 2 * ((lane >> 4) & 1) + ((j16 & 3) >> 1);
    const int v_lane = v_row * S::kRowBytes + ((v_chunk ^ swizzle_v<D>(v_row)) << 4) + ((j16 & 1) << 3);

    f32x16 o_acc[D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; db++)
#pragma unroll
        for (int r = 0; r < 16; r++) o_acc[db][r] = 0.f;
    float m_run = -INFINITY;   // running max of raw scores (shared by both half-waves)
    float l_run = 0.f;         // running sum, partial: this lane's 32 of the 64 keys per tile

    // The tiles so far may hold no key that a row sees - beyond its diagonal in a split, or with scores of -inf that the
    // caller masks keys with: the maximum stays -inf, and the exponents are then taken against 0, so that P = 2^-inf = 0.
    auto finite_max = [&](float m) { return m == -INFINITY ? 0.f : m; };

    auto compute_tile = [&](int stage, int tile) {
        const int j0 = tile * S::kTileKV;
        if (CAUSAL && j0 > q0 + 31 + off) return;    // every key of the tile is masked for this wave
        if (TAIL && q0 >= Nq) return;                // a wave of padding rows only (few queries, e.g. decode)
        const char* ks = stage ? smem1 : smem0;
        const char* vs = ks + S::kTileBytes;

        // S^T[key][query] for two 32-key blocks
        f32x16 s[2];
#pragma unroll
        for (int b = 0; b < 2; b++) {
#pragma unroll
            for (int r = 0; r < 16; r++) s[b][r] = 0.f;
#pragma unroll
            for (int kb = 0; kb < D / 16; kb++) {
                bf16x8 kf = lds_read_b128(ks, (k_lane ^ ((2 * kb) << 4)) + b * 32 * S::kRowBytes);
                s[b] = mfma32(kf, qf[kb], s[b]);
            }
        }
        // tile crosses the diagonal for some row of this wave, or runs past the last key
        if ((CAUSAL && j0 + S::kTileKV - 1 > q0 + off) || (TAIL && j0 + S::kTileKV > Nk)) {
#pragma unroll
            for (int b = 0; b < 2; b++)
#pragma unroll
                for (int r = 0; r < 16; r++) {
                    int key = j0 + 32 * b + 8 * (r >> 2) + 4 * h + (r & 3);
                    if ((CAUSAL && key > my_q + off) || (TAIL && key >= Nk)) s[b][r] = -INFINITY;
                }
        }
        // running max
        float mx = s[0][0];
#pragma unroll
        for (int r = 1; r < 16; r++) mx = __builtin_fmaxf(mx, s[0][r]);
#pragma unroll
        for (int r = 0; r < 16; r++) mx = __builtin_fmaxf(mx, s[1][r]);
        mx = half_max(mx);
        // The running max is only raised when some row of the wave outgrows it by more than
        // kMaxSlack in the base-2 exponent: with a stale max every exponent stays <= kMaxSlack,
        // so P <= 2^kMaxSlack is still exactly representable work for fp32/bf16, and O and l
        // carry the same factor, which the final division removes.  Saves the O rescale on
        // almost every tile.
        constexpr float kMaxSlack = 8.0f;
        const bool raise = (mx - m_run) * c > kMaxSlack;          // true on the first tile (m_run = -inf)
        if (__builtin_amdgcn_ballot_w64(raise) != 0) {
            const float m_new = __builtin_fmaxf(m_run, mx);
            const float corr = __builtin_amdgcn_exp2f((m_run - finite_max(m_new)) * c);
            m_run = m_new;
            l_run *= corr;
#pragma unroll
            for (int db = 0; db < D / 32; db++)
#pragma unroll
                for (int r = 0; r < 16; r++) o_acc[db][r] *= corr;
        }
        const float mc = finite_max(m_run) * c;
        // P = 2^(S*c - m*c), partial row sums
        float psum = 0.f;
#pragma unroll
        for (int b = 0; b < 2; b++)
#pragma unroll
            for (int r = 0; r < 16; r++) {
                float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[b][r], c, -mc));
                s[b][r] = p;
                psum += p;
            }
        l_run += psum;

        // O^T += V^T P^T, 16 keys per MFMA
#pragma unroll
        for (int kk = 0; kk < 4; kk++) {
            const int b = kk >> 1, r0 = 8 * (kk & 1);
            bf16x8 pb = cvt8(s[b][r0 + 0], s[b][r0 + 1], s[b][r0 + 2], s[b][r0 + 3],
                             s[b][r0 + 4], s[b][r0 + 5], s[b][r0 + 6], s[b][r0 + 7]);
#pragma unroll
            for (int db = 0; db < D / 32; db++) {
                // rows 16*kk + 4*h + (0..3) and +8; the +8 flips bit 1 of swizzle_v's low field
                const int row_off = 16 * kk * S::kRowBytes;
                const int x0 = (4 * db) << 4;
                const int x1 = ((4 * db) ^ 2) << 4;
                bf16x4 v0 = lds_read_tr16(vs, (v_lane ^ x0) + row_off);
                bf16x4 v1 = lds_read_tr16(vs, (v_lane ^ x1) + row_off + 8 * S::kRowBytes);
                o_acc[db] = mfma32(concat(v0, v1), pb, o_acc[db]);
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
    // With a known start the compiler keeps a 64-bit address per lane and load and advances each by a vector addition;
    // with an unknown one the tile's address stays scalar.
    if (!SPLIT && (CAUSAL || TAIL)) asm volatile("" : "+s"(t_begin));
    if (SPLIT) {
        t_begin = split * tiles_per_split;
        if (t_begin + tiles_per_split < n_tiles) n_tiles = t_begin + tiles_per_split;
    }
    if (!SPLIT || t_begin < n_tiles) issue_tile(0, t_begin);     // (causal: a split may lie wholly beyond the tile's last key)
    wait_vmcnt<0>();
    __syncthreads();
    for (int t = t_begin; t < n_tiles; t += 2) {
        issue_tile(1, t + 1);
        compute_tile(0, t);
        wait_vmcnt<0>();
        __syncthreads();
        if (t + 2 < n_tiles) issue_tile(0, t + 2);
        compute_tile(1, t + 1);
        wait_vmcnt<0>();
        __syncthreads();
    }

    // ---- epilogue
    const float l_tot = half_sum(l_run);
    const float inv = SPLIT && l_tot == 0.f ? 0.f : 1.0f / l_tot;     // (no visible key in this split: O = 0, LSE = -inf)
    if (SPLIT) {
        if (my_q < Nq) {
            const size_t prow = ((size_t)split * heads + bh) * Nq + my_q;   // [split][head][query]
            float* Op = O_part + prow * D;
#pragma unroll
            for (int db = 0; db < D / 32; db++)
#pragma unroll
                for (int g = 0; g < 4; g++) {
                    f32x4 v4 = {o_acc[db][4 * g + 0] * inv, o_acc[db][4 * g + 1] * inv, o_acc[db][4 * g + 2] * inv, o_acc[db][4 * g + 3] * inv};
                    *(f32x4*)(Op + 32 * db + 8 * g + 4 * h) = v4;
                }
            if (h == 0) LSE_part[prow] = m_run * scale + __builtin_logf(l_tot);
        }
    } else if (!TAIL || my_q < Nq) {
        bf16* Oh = O + head + (size_t)my_q * D;
#pragma unroll
        for (int db = 0; db < D / 32; db++)
#pragma unroll
            for (int g = 0; g < 4; g++) {
                bf16x2 a = cvt2(o_acc[db][4 * g + 0] * inv, o_acc[db][4 * g + 1] * inv);
                bf16x2 b = cvt2(o_acc[db][4 * g + 2] * inv, o_acc[db][4 * g + 3] * inv);
                *(bf16x4*)(Oh + 32 * db + 8 * g + 4 * h) = __builtin_shufflevector(a, b, 0, 1, 2, 3);
            }
        if (h == 0) LSE[(size_t)bh * Nq + my_q] = m_run * scale + __builtin_logf(l_tot);
    }
}

// ------------------------------------------------------------------------------------------
// the forward kernel of launches that are bound by the chip's arithmetic
// ------------------------------------------------------------------------------------------
// A wave owns 32 query rows and goes through two phases per 64-key tile: matrix instructions (O += V P of tile t, then
// S = K Q of tile t+1) and vector instructions (the exponentials of tile t+1).  A wave issues in order, so it uses one of
// the two pipes at a time, and waves that are free to run drift into step with each other: both of a SIMD want the matrix
// pipe, then both the vector ALU (3450 cycles for a tile of both at D = 128, where the matrix instructions take 2048).
//
// GROUPS = 2: eight waves, 256 query rows, two waves on each SIMD, kept one phase apart by a barrier per phase: the four
// waves of one group have the matrix pipe while the other group has the vector ALU.  K and V are fetched once for 256
// rows instead of 128 (fetching them is power that the matrix pipe does not get).
// GROUPS = 1: four waves, 128 query rows, for launches that would leave compute units idle with 256-row tiles.  There is
// no second wave to fill the gaps, so the wave interleaves S = K Q of the next tile with the exponentials of this one.
// Both do the same arithmetic in the same order: a row's bits do not depend on the choice.
//
// The running maximum is not looked for in every tile.  The exponents are taken against the maximum of the first tile, and
// a tile whose sum of exponentials (32 keys of a row in a lane) exceeds kMaxSum - or is not a number, or infinite - is done
// again against its own maximum, after which O and l are scaled as usual: 16 v_max3 of four cycles, a sixth of the vector
// phase, are gone from every other tile.  kMaxSum is 32 exponentials of 2^8: the sums that form O before the division by l
// get no closer to the end of the number range than with a maximum that is kept within 2^8, as the kernel of few rows does.
// What P, O and l are multiplied with has no part in their rounding, but a P that is 1 has none at all: where one key
// dominates a row that was not done again, O is as exact as any other row's and not more (against fp64, normal data with
// scores of sigma 1, 4 and 8: 1.78e-3, 2.16e-3, 2.20e-3, with the maximum of every tile within 2^8 1.78e-3, 2.03e-3, 1.88e-3).
// Where scores are that large, or grow along the keys, a tile that outgrew its maximum is followed by others: doing it again
// leaves room, the exponents are then taken against 2^16 times its maximum.  (2^24 would do more for scores of sigma 16, but
// values of V below 1e-36 would lose bits.)  Forward, us, with the maximum of every tile, without the room and with it: sigma
// 8 B16 H16 N4096 causal D128 1192, 1160, 1063, D64 661, 678, 631; sigma 16 1198, 1242, 1160 and 663, 738, 668; scores that
// grow by 2^20 from tile to tile 1197, 1327, 1182 and 681, 876, 739; the longest left, D64 B16 H16 N1024 without a mask, keys
// that grow to sigma 30: 86, 110, 105.
//
// Tiles go to an LDS ring by direct loads: four stages, issued three tiles ahead, with two groups (one workgroup on a compute
// unit); two stages with one (two or three workgroups to a unit, which cover each other's waits: four stages and one
// workgroup were slower at every size).
//
// Forward, us, before (four waves, 128 rows, phases in program order) and now: B16 H16 N4096 causal D128 1140, 1013, without a
// mask 2014, 1796, causal D64 621, 594; B16 H16 N1024 D64 79.3, 77.5; B1 H16 N8192 causal D128 302, 244; with one group
// B1 H16 N2048 D64 27.1, 23.0, B2 Hq16 Hkv4 N1001 causal D128 24.3, 21.6.  One group or two at D = 128: see two_groups_pay().
template <int D, int GROUPS>
struct FwdPhaseShape {
    static constexpr int kWaves = 4 * GROUPS, kThreads = 64 * kWaves;
    static constexpr int kTileQ = 32 * kWaves, kTileKV = 64;
    static constexpr int kRowBytes = D * 2, kChunksPerRow = D / 8;
    static constexpr int kTileBytes = kTileKV * kRowBytes;
    static constexpr int kStageBytes = 2 * kTileBytes;                  // K tile then V tile
    static constexpr int kStages = GROUPS == 2 ? 4 : 2;
    static constexpr int kLoads = kTileKV * kChunksPerRow / kThreads;   // per thread and tensor
    static constexpr int kTileLoads = 2 * kLoads;
    // waves per SIMD to compile for.  One group: two (D = 128) or three (D = 64) workgroups share a compute unit; of the 168
    // registers that leaves at D = 64 the ragged causal and the split kernels lack one to six (prologue, epilogue, masked tiles)
    static constexpr int kWavesPerSimd = D == 128 ? 2 : 3;
};

template <int D, bool CAUSAL, bool TAIL, bool SPLIT, int GROUPS>
__global__ __launch_bounds__((FwdPhaseShape<D, GROUPS>::kThreads), (FwdPhaseShape<D, GROUPS>::kWavesPerSimd))
void attn_fwd_phase_kernel(const bf16* __restrict__ Q, const bf16* __restrict__ K, const bf16* __restrict__ V,
                           bf16* __restrict__ O, float* __restrict__ LSE,
                           int Nq, int Nk, int num_q_tiles, int heads, int head_group, float scale, int hq, int hkv,
                           int n_splits, int tiles_per_split, float* __restrict__ O_part, float* __restrict__ LSE_part)
{
    using S = FwdPhaseShape<D, GROUPS>;
    __shared__ __attribute__((aligned(1024))) char smem[S::kStages * S::kStageBytes];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int l32 = lane & 31;
    const int h = lane >> 5;

    int bh, qt, split = 0;
    if (SPLIT) split_of(blockIdx.x, gridDim.x, hq / hkv, num_q_tiles, n_splits, bh, split, qt);
    else if (CAUSAL) tile_of(blockIdx.x, heads, num_q_tiles, head_group, bh, qt);
    else {
        const int id = xcd_remap(blockIdx.x, gridDim.x);
        bh = id / num_q_tiles;
        qt = id - bh * num_q_tiles;
    }
    const size_t head = (size_t)bh * Nq * D;
    const size_t kv_head = (size_t)((bh / hq) * hkv + (bh % hq) / (hq / hkv)) * Nk * D;
    const bf16* Kh = K + kv_head;
    const bf16* Vh = V + kv_head;
    // the row blocks of the two groups alternate, so that under the causal mask both have about the same number of tiles
    const int group = GROUPS == 2 ? wave >> 2 : 0;
    const int q0 = qt * S::kTileQ + (GROUPS == 2 ? 2 * (wave & 3) + group : wave) * 32;
    const int my_q = q0 + l32;
    const int my_q_ld = (!TAIL || my_q < Nq) ? my_q : Nq - 1;
    const int off = TAIL ? Nk - Nq : 0;          // causal: query i sees keys <= i + off
    const float c = scale * kLog2e;

    // key tiles of the workgroup, and of this wave
    int t_begin = 0, n_tiles, n_my;
    {
        int n_keys = Nk;
        if (CAUSAL && qt * S::kTileQ + S::kTileQ + off < n_keys) n_keys = qt * S::kTileQ + S::kTileQ + off;
        n_tiles = (n_keys + S::kTileKV - 1) / S::kTileKV;
        if (SPLIT) {
            t_begin = split * tiles_per_split;
            if (t_begin + tiles_per_split < n_tiles) n_tiles = t_begin + tiles_per_split;
        }
        n_my = n_tiles;
        if (CAUSAL) { const int d = (q0 + 31 + off) / S::kTileKV + 1; if (d < n_my) n_my = d; }
        if (TAIL && q0 >= Nq) n_my = t_begin;    // a wave of padding rows only
    }

    // ---- tile loads: LDS position s = it * threads + tid holds (row = s / chunks per row, physical chunk = s % chunks per row)
    int k_src[S::kLoads], v_src[S::kLoads];
#pragma unroll
    for (int it = 0; it < S::kLoads; it++) {
        const int s = it * S::kThreads + tid, row = s / S::kChunksPerRow, pc = s % S::kChunksPerRow;
        k_src[it] = row * D + ((pc ^ swizzle_k<D>(row)) * 8);
        v_src[it] = row * D + ((pc ^ swizzle_v<D>(row)) * 8);
    }
    // every call issues the same number of loads in every wave (the waits count them); beyond the last tile it fetches that
    // one again, into a stage nobody reads any more
    auto issue = [&](const bf16* src, const int (&lane_src)[S::kLoads], int in_stage, int tile) __attribute__((always_inline)) {
        char* base = smem + (tile & (S::kStages - 1)) * S::kStageBytes + in_stage + wave * 1024;
        if (tile > n_tiles - 1) tile = n_tiles - 1;
        const int j0 = tile * S::kTileKV;
        const bf16* first = src + (size_t)j0 * D;
        if (!TAIL || j0 + S::kTileKV <= Nk) {
#pragma unroll
            for (int it = 0; it < S::kLoads; it++) load_global_to_lds16_sbase_untracked(first, lane_src[it] * 2, base + it * (S::kThreads * 16));
        } else {                                 // rows past the last key fetch that one instead (they are masked later)
#pragma unroll
            for (int it = 0; it < S::kLoads; it++) {
                const int beyond = (it * S::kThreads + tid) / S::kChunksPerRow - (Nk - 1 - j0);     // (the tile's first key is a real one)
                load_global_to_lds16_sbase_untracked(first, (lane_src[it] - (beyond > 0 ? beyond : 0) * D) * 2, base + it * (S::kThreads * 16));
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto issue_k = [&](int tile) __attribute__((always_inline)) { issue(Kh, k_src, 0, tile); };
    auto issue_v = [&](int tile) __attribute__((always_inline)) { issue(Vh, v_src, S::kTileBytes, tile); };
    auto issue_tile = [&](int tile) __attribute__((always_inline)) { issue_k(tile); issue_v(tile); };

    // ---- Q fragments (B operand of S^T = K Q^T): lane holds Q[my_q][16*kb + 8*h .. +7].  The compiler waits for them, and
    // with them for everything issued before, which is what the first product needs: the first tile of K.
    const bool any = !SPLIT || t_begin < n_tiles;    // (causal: a split may lie wholly beyond the tile's last key)
    if (any) {
        issue_k(t_begin);
        if (GROUPS == 1) { issue_v(t_begin); issue_k(t_begin + 1); }
    }
    bf16x8 qf[D / 16];
#pragma unroll
    for (int kb = 0; kb < D / 16; kb++) qf[kb] = *(const bf16x8*)(Q + head + (size_t)my_q_ld * D + kb * 16 + h * 8);
#pragma unroll
    for (int kb = 0; kb < D / 16; kb++) asm volatile("" : "+v"(qf[kb]));
    if (any) {
        wait_vmcnt<0>();
        if (GROUPS == 2) { issue_v(t_begin); issue_tile(t_begin + 1); issue_tile(t_begin + 2); }
    }

    // ---- per-lane LDS read offsets
    // K: row 32*b + l32, logical chunk 2*kb + h.  V (transposing read): 16-lane group G = lane/16 -> (d half = G%2, key half =
    // G/2); lane j of the group addresses row 4*(G/2) + j/4, columns 32*db + 16*(G%2) + 4*(j%4)
    const int k_lane = l32 * S::kRowBytes + ((h ^ swizzle_k<D>(l32)) << 4);
    const int j16 = lane & 15;
    const int v_row = 4 * h + (j16 >> 2);
    const int v_chunk = 2 * ((lane >> 4) & 1) + ((j16 & 3) >> 1);
    const int v_lane = v_row * S::kRowBytes + ((v_chunk ^ swizzle_v<D>(v_row)) << 4) + ((j16 & 1) << 3);

    f32x16 o_acc[D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; db++)
#pragma unroll
        for (int r = 0; r < 16; r++) o_acc[db][r] = 0.f;
    float m_run = -INFINITY;   // what the exponents are taken against (a raw score, shared by both half-waves), and its multiple in
    float mc = -INFINITY;      // base 2; -inf: exponentials against it are infinite or not a number, and the tile is done again
    float l_run = 0.f;         // running sum, partial: this lane's 32 of the 64 keys per tile
    bf16x8 pb[4];              // P of the tile in hand, 16 keys each

    constexpr int kKSteps = D / 8, kVSteps = D / 8;      // matrix instructions of S = K Q and of O += V P
    constexpr int kAhead = 2 * GROUPS;                   // fragments read ahead of their use (one group: more would not fit the registers)
    bf16x8 kfr[kKSteps], vfr[kVSteps];
    auto stage_of = [&](int tile) { return smem + (tile & (S::kStages - 1)) * S::kStageBytes; };
    auto read_k = [&](const char* ks, int i) __attribute__((always_inline)) {        // step i: 16 columns i / 2, 32 keys i % 2
        kfr[i] = lds_read_b128(ks, (k_lane ^ ((2 * (i >> 1)) << 4)) + (i & 1) * 32 * S::kRowBytes);
    };
    auto read_v = [&](const char* vs, int i) __attribute__((always_inline)) {        // step i: 16 keys i / (D/32), 32 columns i % (D/32)
        const int row_off = 16 * (i / (D / 32)) * S::kRowBytes, db = i % (D / 32);
        // rows 16*kk + 4*h + (0..3) and +8; the +8 flips bit 1 of swizzle_v's low field
        vfr[i] = concat(lds_read_tr16(vs, (v_lane ^ ((4 * db) << 4)) + row_off),
                        lds_read_tr16(vs, (v_lane ^ (((4 * db) ^ 2) << 4)) + row_off + 8 * S::kRowBytes));
    };
    // (the empty asm statements hold a matrix instruction in its place among the reads: the compiler keeps them in order)
    auto multiply_k = [&](f32x16 (&s)[2], int i) __attribute__((always_inline)) {
        const int kb = i >> 1, b = i & 1;
        if (kb == 0) {
            f32x16 zero;
#pragma unroll
            for (int r = 0; r < 16; r++) zero[r] = 0.f;
            s[b] = mfma32(kfr[i], qf[0], zero);
        } else {
            s[b] = mfma32(kfr[i], qf[kb], s[b]);
        }
        asm volatile("" : : "v"(s[b][0]));
    };
    auto multiply_v = [&](int i) __attribute__((always_inline)) {
        const int kk = i / (D / 32), db = i % (D / 32);
        o_acc[db] = mfma32(vfr[i], pb[kk], o_acc[db]);
        asm volatile("" : : "v"(o_acc[db][0]));
    };

    // register r of block b of the scores <-> key j0 + 32*b + 8*(r/4) + 4*h + r%4, lane <-> query my_q
    auto mask = [&](f32x16 (&s)[2], int tile) __attribute__((always_inline)) {
        const int j0 = tile * S::kTileKV;
        if ((CAUSAL && j0 + S::kTileKV - 1 > q0 + off) || (TAIL && j0 + S::kTileKV > Nk)) {
#pragma unroll
            for (int b = 0; b < 2; b++)
#pragma unroll
                for (int r = 0; r < 16; r++) {
                    const int key = j0 + 32 * b + 8 * (r >> 2) + 4 * h + (r & 3);
                    if ((CAUSAL && key > my_q + off) || (TAIL && key >= Nk)) s[b][r] = -INFINITY;
                }
        }
    };
    // The tiles so far may hold no key that a row sees - beyond its diagonal in a split, or with scores of -inf that the
    // caller masks keys with: the maximum stays -inf, and the exponents are then taken against 0, so that P = 2^-inf = 0.
    auto finite_mc = [&]() { return m_run == -INFINITY ? 0.f : m_run * c; };
    auto raise = [&](const f32x16 (&s)[2], float above) __attribute__((always_inline)) {
        float mx = s[0][0];
#pragma unroll
        for (int r = 1; r < 16; r++) mx = __builtin_fmaxf(mx, s[0][r]);
#pragma unroll
        for (int r = 0; r < 16; r++) mx = __builtin_fmaxf(mx, s[1][r]);
        const float m_old = m_run;
        m_run = __builtin_fmaxf(m_run, half_max(mx) + above);
        mc = m_run * c;
        const float corr = __builtin_amdgcn_exp2f(m_run == -INFINITY ? m_old : (m_old - m_run) * c);
        l_run *= corr;
#pragma unroll
        for (int db = 0; db < D / 32; db++)
#pragma unroll
            for (int r = 0; r < 16; r++) o_acc[db][r] *= corr;
    };
    constexpr float kMaxSum = 8192.f;
    // 16 in the base-2 exponent, in a scalar register (finite for the smallest scales, too)
    const float redo_above = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, __builtin_fminf(16.f / c, 1e30f))));
    // P = 2^(S*c - against): element e of 32 is register e % 16 of block e / 16.  The sum is formed in the order of the elements
    auto exponential = [&](const f32x16 (&s)[2], int e, float against) __attribute__((always_inline)) {
        return __builtin_amdgcn_exp2f(__builtin_fmaf(s[e >> 4][e & 15], c, -against));
    };
    auto exponentials = [&](const f32x16 (&s)[2], float against) __attribute__((always_inline)) {
        float sum = 0.f;
#pragma unroll
        for (int kk = 0; kk < 4; kk++) {
            float p[8];
#pragma unroll
            for (int r = 0; r < 8; r++) {
                p[r] = exponential(s, 8 * kk + r, against);
                sum += p[r];
            }
            pb[kk] = cvt8(p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7]);
        }
#pragma unroll
        for (int kk = 0; kk < 4; kk++) asm volatile("" : "+v"(pb[kk]));
        return sum;
    };
    auto too_large = [&](float sum) { return __builtin_expect(__builtin_amdgcn_ballot_w64(!(sum <= kMaxSum)) != 0, 0); };
    auto phase_end = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" : : : "memory");
    };
    auto scores = [&](f32x16 (&s)[2], int tile) __attribute__((always_inline)) {     // S = K Q alone
        const char* ks = stage_of(tile);
#pragma unroll
        for (int i = 0; i < kAhead; i++) read_k(ks, i);
#pragma unroll
        for (int i = 0; i < kKSteps; i++) {
            multiply_k(s, i);
            if (i + kAhead < kKSteps) read_k(ks, i + kAhead);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto read_v_ahead = [&](int tile) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kAhead; i++) read_v(stage_of(tile) + S::kTileBytes, i);
    };
    auto products = [&](int tile) __attribute__((always_inline)) {                   // O += V P alone, behind read_v_ahead()
        const char* vs = stage_of(tile) + S::kTileBytes;
#pragma unroll
        for (int i = 0; i < kVSteps; i++) {
            multiply_v(i);
            if (i + kAhead < kVSteps) read_v(vs, i + kAhead);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    int t = t_begin;
    if (any) {
    phase_end();                                 // K of the first tile is here
    if constexpr (GROUPS == 2) {
        f32x16 s[2];
        // The barriers a wave passes, two per tile and two ahead of the first, are the same in both groups; the second
        // group's phases come one barrier later.  A stage is refilled by loads issued in the matrix phase of tile t (with
        // tile t+3, into the stage of tile t-1, whose V the other group read at the latest one barrier ago), and every wave
        // waits for its loads of tile t+2 at the end of that phase: both groups read tile t+2 at least one barrier later.
        // The first tile is an exception: the first group reads its first fragments of V one barrier ahead of the second group's wait.
        // They are the rows that its own waves have fetched.
        static_assert((kAhead + D / 32 - 1) / (D / 32) * 16 * S::kChunksPerRow <= S::kThreads / 2, "rows that the first group's first load instruction fetches");
        if (group == 1) phase_end();
        if (n_my > t) scores(s, t);
        wait_vmcnt<S::kTileLoads>();             // tiles t and t+1
        phase_end();
        if (n_my > t) {
            mask(s, t);
            raise(s, 0.f);
            l_run = exponentials(s, finite_mc());
            read_v_ahead(t);
        }
        phase_end();
#pragma unroll 1
        for (; t < n_my - 1; t++) {
            issue_tile(t + 3);
            __builtin_amdgcn_s_setprio(1);       // the matrix pipe first: the other group has more instructions ready
            const char* vs = stage_of(t) + S::kTileBytes;
            const char* ks = stage_of(t + 1);
#pragma unroll
            for (int i = 0; i < kVSteps + kKSteps; i++) {
                if (i < kVSteps) multiply_v(i); else multiply_k(s, i - kVSteps);
                if (i + kAhead < kVSteps) read_v(vs, i + kAhead);
                else if (i + kAhead - kVSteps < kKSteps) read_k(ks, i + kAhead - kVSteps);
                __builtin_amdgcn_sched_barrier(0);
            }
            __builtin_amdgcn_s_setprio(0);
            wait_vmcnt<S::kTileLoads>();
            phase_end();
            asm volatile("" : "+v"(s[0])); asm volatile("" : "+v"(s[1]));     // (the vector phase stays behind the barrier)
            mask(s, t + 1);
            float sum = exponentials(s, mc);
            if (too_large(sum)) {
                raise(s, redo_above);
                sum = exponentials(s, finite_mc());
            }
            l_run += sum;
            read_v_ahead(t + 1);
            phase_end();
        }
        if (t < n_my) {
            issue_tile(t + 3);
            products(t);
            wait_vmcnt<S::kTileLoads>();
            phase_end();
            phase_end();
            t++;
        }
#pragma unroll 1
        for (; t < n_tiles; t++) {               // the others of the workgroup have more tiles
            issue_tile(t + 3);
            wait_vmcnt<S::kTileLoads>();
            phase_end();
            phase_end();
        }
        if (group == 0) phase_end();
    } else {
        f32x16 sa[2], sb[2];                     // scores of even and odd tiles (counted from the first)
        // One tile: S of the next one, each matrix instruction with its share of this one's exponentials behind it, then O.
        auto tile_step = [&](f32x16 (&s)[2], f32x16 (&next)[2], bool has_next, int t) __attribute__((always_inline)) {
            issue_k(t + S::kStages);             // into the stages of K of tile t and V of tile t-1, which every wave has left
            issue_v(t + S::kStages - 1);
            float sum = 0.f;
            if (has_next) {
                const char* ks = stage_of(t + 1);
                constexpr int kPer = 32 / kKSteps;               // exponentials per matrix instruction
                float p[32];
#pragma unroll
                for (int i = 0; i < kAhead; i++) read_k(ks, i);
#pragma unroll
                for (int e = 0; e < kPer; e++) { p[e] = exponential(s, e, mc); asm volatile("" : : "v"(p[e])); }
#pragma unroll
                for (int i = 0; i < kKSteps; i++) {
                    multiply_k(next, i);
                    if (i + kAhead < kKSteps) read_k(ks, i + kAhead); else read_v(stage_of(t) + S::kTileBytes, i + kAhead - kKSteps);
#pragma unroll
                    for (int e = kPer * (i + 1); e < kPer * (i + 2) && e < 32; e++) { p[e] = exponential(s, e, mc); asm volatile("" : : "v"(p[e])); }
#pragma unroll
                    for (int e = kPer * i; e < kPer * (i + 1); e++) { sum += p[e]; asm volatile("" : : "v"(sum)); }
                    if ((kPer * (i + 1)) % 8 == 0) {
                        const int kk = kPer * (i + 1) / 8 - 1;
                        pb[kk] = cvt8(p[8 * kk], p[8 * kk + 1], p[8 * kk + 2], p[8 * kk + 3], p[8 * kk + 4], p[8 * kk + 5], p[8 * kk + 6], p[8 * kk + 7]);
                        asm volatile("" : : "v"(pb[kk]));
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
                read_v_ahead(t);
                sum = exponentials(s, mc);
            }
            if (too_large(sum)) {
                raise(s, redo_above);
                sum = exponentials(s, finite_mc());
            }
            l_run += sum;
            products(t);
            if (has_next) mask(next, t + 1);
            wait_vmcnt<(S::kStages - 2) * S::kTileLoads>();      // K of tile t+2 and V of t+1 are here
            phase_end();
        };
        if (n_my > t) {
            scores(sa, t);
            mask(sa, t);
            raise(sa, 0.f);                           // (no visible key yet: mc stays -inf, and this tile and the next are done again)
        }
        phase_end();                             // (K of the first tile is about to be overwritten)
#pragma unroll 1
        for (; t + 2 < n_my; t += 2) {
            tile_step(sa, sb, true, t);
            tile_step(sb, sa, true, t + 1);
        }
        if (t + 1 < n_my) {
            tile_step(sa, sb, true, t);
            tile_step(sb, sa, false, t + 1);
            t += 2;
        } else if (t < n_my) {
            tile_step(sa, sb, false, t);
            t++;
        }
#pragma unroll 1
        for (; t < n_tiles; t++) {
            issue_k(t + S::kStages);
            issue_v(t + S::kStages - 1);
            wait_vmcnt<(S::kStages - 2) * S::kTileLoads>();
            phase_end();
        }
    }
    wait_vmcnt<0>();                             // the spare loads of the last tiles must not outlive the workgroup's LDS
    }

    // ---- epilogue: O = O / l, LSE = m*scale + ln l
    const float l_tot = half_sum(l_run);
    const float inv = SPLIT && l_tot == 0.f ? 0.f : 1.0f / l_tot;     // (no visible key in this split: O = 0, LSE = -inf)
    if (SPLIT) {
        if (my_q < Nq) {
            const size_t prow = ((size_t)split * heads + bh) * Nq + my_q;   // [split][head][query]
            float* Op = O_part + prow * D;
#pragma unroll
            for (int db = 0; db < D / 32; db++)
#pragma unroll
                for (int g = 0; g < 4; g++)
                    *(f32x4*)(Op + 32 * db + 8 * g + 4 * h) = f32x4{o_acc[db][4 * g + 0] * inv, o_acc[db][4 * g + 1] * inv, o_acc[db][4 * g + 2] * inv, o_acc[db][4 * g + 3] * inv};
            if (h == 0) LSE_part[prow] = m_run * scale + __builtin_logf(l_tot);
        }
    } else if (!TAIL || my_q < Nq) {
        bf16* Oh = O + head + (size_t)my_q * D;
#pragma unroll
        for (int db = 0; db < D / 32; db++)
#pragma unroll
            for (int g = 0; g < 4; g++) {
                bf16x2 a = cvt2(o_acc[db][4 * g + 0] * inv, o_acc[db][4 * g + 1] * inv);
                bf16x2 b = cvt2(o_acc[db][4 * g + 2] * inv, o_acc[db][4 * g + 3] * inv);
                *(bf16x4*)(Oh + 32 * db + 8 * g + 4 * h) = __builtin_shufflevector(a, b, 0, 1, 2, 3);
            }
        if (h == 0) LSE[(size_t)bh * Nq + my_q] = m_run * scale + __builtin_logf(l_tot);
    }
}

template <int D, bool CAUSAL, bool TAIL, bool SPLIT, int GROUPS>
static hipError_t launch_phase(const void* q, const void* k, const void* v, void* o, float* lse,
                               int B, int H, int Hkv, int Nq, int Nk, float scale, hipStream_t stream,
                               int n_splits = 1, int tiles_per_split = 0, float* o_part = nullptr, float* lse_part = nullptr)
{
    using S = FwdPhaseShape<D, GROUPS>;
    const int num_q_tiles = (Nq + S::kTileQ - 1) / S::kTileQ;
    hipLaunchKernelGGL((attn_fwd_phase_kernel<D, CAUSAL, TAIL, SPLIT, GROUPS>), dim3(B * H * num_q_tiles * n_splits), dim3(S::kThreads), 0, stream,
                       (const bf16*)q, (const bf16*)k, (const bf16*)v, (bf16*)o, lse, Nq, Nk, num_q_tiles, B * H,
                       tile_order_heads(B * H, num_q_tiles, CAUSAL, D), scale, H, Hkv, n_splits, tiles_per_split, o_part, lse_part);
    return hipGetLastError();
}

template <int D, bool CAUSAL, bool TAIL, bool SPLIT>
static hipError_t launch_fwd_tt(const void* q, const void* k, const void* v, void* o, float* lse,
                                int B, int H, int Hkv, int Nq, int Nk, float scale, hipStream_t stream,
                                int n_splits = 1, int tiles_per_split = 0, float* o_part = nullptr, float* lse_part = nullptr)
{
    using S = FwdShape<D>;
    auto kern = attn_fwd_kernel<D, CAUSAL, TAIL, SPLIT>;
    const int num_q_tiles = (Nq + S::kTileQ - 1) / S::kTileQ;
    const int total = B * H * num_q_tiles * n_splits;
    hipLaunchKernelGGL(kern, dim3(total), dim3(S::kThreads), 0, stream,
                       (const bf16*)q, (const bf16*)k, (const bf16*)v, (bf16*)o, lse,
                       Nq, Nk, num_q_tiles, B * H, tile_order_heads(B * H, num_q_tiles, CAUSAL, D), scale, H, Hkv, n_splits, tiles_per_split, o_part, lse_part);
    return hipGetLastError();
}

// Whether two groups (256-row tiles) take less time than one (128-row tiles, two workgroups on a compute unit), D = 128.  us of
// a workgroup that has its place: two groups U2 a 64-key tile and O2 around them, one group U1 and O1; a launch takes as many of
// these one behind the other as the fullest compute unit has.
static bool two_groups_pay(int B, int H, int Nq, int Nk, bool causal, int cus)
{
    const long long heads = (long long)B * H, tiles1 = heads * ((Nq + 127) / 128), tiles2 = heads * ((Nq + 255) / 256);
    if (tiles1 <= cus) return false;
    const double n = (Nk + 63) / 64, units1 = (double)tiles1 / (2 * cus), units2 = (double)tiles2 / cus;
    if (!causal) return ceil(units2) * (1.7 * n + 8) < ceil(2 * units1) / 2 * (1.84 * n + 6);
    // half the keys on average and half a tile more; the longest tiles, which come first, show in part at the end
    return units2 * (1.5 * (n / 2 + 2) + 5) + 0.3 * (1.5 * n + 5) < units1 * (1.84 * (n / 2 + 1) + 2) + 0.3 * 0.55 * (1.84 * n + 2);
}

template <int D, bool CAUSAL>
static hipError_t launch_fwd_t(const void* q, const void* k, const void* v, void* o, float* lse,
                               int B, int H, int Hkv, int Nq, int Nk, float scale, hipStream_t stream)
{
    // Few query rows a head (decoding) are bound by reading K and V, whatever the waves do: B64 H8 Nq4 Nk4000 D128 177 us either way, and
    // decoding takes this path with its groups as rows.  And at D = 64 a
    // sequence of one or two tiles has nothing to overlap, and four workgroups to a compute unit instead of three are
    // better: B16 H32 N128 7.5 us instead of 7.8, B32 H32 N100 13.1, 14.1.  Neither condition looks at the number of heads: the two kernels
    // look for the maximum in different tiles, and a head's bits shall not depend on what else is in the call.
    if constexpr (!CAUSAL)
        if (Nq <= 64 && Nq != Nk) return launch_fwd_tt<D, false, true, false>(q, k, v, o, lse, B, H, Hkv, Nq, Nk, scale, stream);
    if constexpr (D == 64)
        if (Nk <= 128) return (Nq != Nk || Nq % 128 ? launch_fwd_tt<64, CAUSAL, true, false> : launch_fwd_tt<64, CAUSAL, false, false>)(q, k, v, o, lse, B, H, Hkv, Nq, Nk, scale, stream, 1, 0, nullptr, nullptr);
    if constexpr (D == 128) {
        int cus = 0;
        hipError_t e = compute_unit_count(&cus);
        if (e != hipSuccess) return e;
        if (two_groups_pay(B, H, Nq, Nk, CAUSAL, cus))
            return (Nq != Nk || Nq % 256 ? launch_phase<128, CAUSAL, true, false, 2> : launch_phase<128, CAUSAL, false, false, 2>)(q, k, v, o, lse, B, H, Hkv, Nq, Nk, scale, stream, 1, 0, nullptr, nullptr);
    }
    return (Nq != Nk || Nq % 128 ? launch_phase<D, CAUSAL, true, false, 1> : launch_phase<D, CAUSAL, false, false, 1>)(q, k, v, o, lse, B, H, Hkv, Nq, Nk, scale, stream, 1, 0, nullptr, nullptr);
}

hipError_t launch_attn_fwd(const void* q, const void* k, const void* v, void* o, float* lse,
                           int B, int H, int Hkv, int Nq, int Nk, int D, int causal, float scale, hipStream_t stream)
{
    if (D == 128) return causal ? launch_fwd_t<128, true>(q, k, v, o, lse, B, H, Hkv, Nq, Nk, scale, stream)
                                : launch_fwd_t<128, false>(q, k, v, o, lse, B, H, Hkv, Nq, Nk, scale, stream);
    return causal ? launch_fwd_t<64, true>(q, k, v, o, lse, B, H, Hkv, Nq, Nk, scale, stream)
                  : launch_fwd_t<64, false>(q, k, v, o, lse, B, H, Hkv, Nq, Nk, scale, stream);
}

// ------------------------------------------------------------------------------------------
// decode: up to 32 query rows per key/value head
// ------------------------------------------------------------------------------------------
// The forward kernel gives a workgroup's rows to its waves, 32 each; with one query for each head of a group only the
// first wave has any, and a 64-key tile takes it about a microsecond.  Here all four waves hold the same rows and share
// the keys: a trip is two tiles, wave w takes 32 keys of tile w / 2, and the waves' (O, max, sum) are joined through
// LDS at the end.  A split has few tiles, so what counts is how soon they are here: four are requested before the
// first is waited for.  That takes the LDS of a whole compute unit, so it is for launches of at most one workgroup
// each; beyond that the calls are bound by the bytes, and the forward kernel's two workgroups keep more of them in
// flight.  Decode call, this kernel against the forward kernel, us: B1 Hq32 Hkv8 Nk2000 D128 9.6, 10.4; Nk500 9.4, 10.3;
// B4 Hq16 Hkv2 Nk5000 D64 8.9, 10.7; but (two stages) B16 Hq32 Hkv8 Nk8192 98, 94, B1 Hq64 Hkv8 Nk65536 48, 46.
// O_part == nullptr (one split): the result itself, bf16.  Grid: heads * n_splits, the splits of a head next to each other.
template <int D>
__global__ __launch_bounds__(256, 1)
void attn_decode_kernel(const bf16* __restrict__ Q, const bf16* __restrict__ K, const bf16* __restrict__ V,
                        bf16* __restrict__ O, float* __restrict__ LSE, int rows, int Nk, int heads, float scale,
                        int n_splits, int tiles_per_split, float* __restrict__ O_part, float* __restrict__ LSE_part)
{
    using S = FwdShape<D>;
    constexpr int kStages = 4;
    __shared__ __attribute__((aligned(1024))) char smem[kStages * S::kStageBytes];
    __shared__ __attribute__((aligned(1024))) char q_smem[32 * S::kRowBytes];
    __shared__ float stat[2][S::kWaves][32];             // maximum and sum of each wave and row

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int l32 = lane & 31;
    const int h = lane >> 5;
    const int split = blockIdx.x % n_splits, head = blockIdx.x / n_splits;
    const bf16* Kh = K + (size_t)head * Nk * D;
    const bf16* Vh = V + (size_t)head * Nk * D;
    const float c = scale * kLog2e;

    const int n_all = 2 * ((Nk + 2 * S::kTileKV - 1) / (2 * S::kTileKV));       // tiles of the head, an even count
    const int t_begin = split * tiles_per_split;
    const int t_end = t_begin + tiles_per_split < n_all ? t_begin + tiles_per_split : n_all;

    // tiles go to LDS as in the forward kernel; rows past the last key fetch it again (they are masked below)
    auto issue_tile = [&](int tile) {
        char* base = smem + (tile - t_begin) % kStages * S::kStageBytes + wave * 1024;
#pragma unroll
        for (int it = 0; it < S::kLoadsPerTile; it++) {
            const int s = it * S::kThreads + tid, r = s / S::kChunksPerRow, pc = s % S::kChunksPerRow;
            const int row = tile * S::kTileKV + r < Nk ? tile * S::kTileKV + r : Nk - 1;
            load_global_to_lds16_untracked(Kh + (size_t)row * D + (pc ^ swizzle_k<D>(r)) * 8, base + it * (S::kThreads * 16));
            load_global_to_lds16_untracked(Vh + (size_t)row * D + (pc ^ swizzle_v<D>(r)) * 8, base + S::kTileBytes + it * (S::kThreads * 16));
        }
    };

    // the query rows travel to LDS as well, ahead of the tiles: loads that the compiler tracks would wait for all of them
#pragma unroll
    for (int it = 0; it < 32 * S::kChunksPerRow / S::kThreads; it++) {
        const int s = it * S::kThreads + tid, r = s / S::kChunksPerRow, pc = s % S::kChunksPerRow;
        const size_t row = (size_t)head * rows + (r < rows ? r : rows - 1);
        load_global_to_lds16_untracked(Q + row * D + (pc ^ swizzle_k<D>(r)) * 8, q_smem + wave * 1024 + it * (S::kThreads * 16));
    }
#pragma unroll
    for (int n = 0; n < kStages; n++)
        if (n < 2 || t_begin + n < t_end) issue_tile(t_begin + n);

    const int my_tile = wave >> 1, key0 = 32 * (wave & 1);       // of a trip's two tiles; first key within the tile
    const int k_lane = l32 * S::kRowBytes + ((h ^ swizzle_k<D>(l32)) << 4);
    const int j16 = lane & 15;
    const int v_row = 4 * h + (j16 >> 2);
    const int v_chunk = 2 * ((lane >> 4) & 1) + ((j16 & 3) >> 1);
    const int v_lane = v_row * S::kRowBytes + ((v_chunk ^ swizzle_v<D>(v_row)) << 4) + ((j16 & 1) << 3);

    f32x16 o_acc[D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; db++)
#pragma unroll
        for (int r = 0; r < 16; r++) o_acc[db][r] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;
    auto finite_max = [](float m) { return m == -INFINITY ? 0.f : m; };        // (exponents of a row without a finite score are taken against 0)

    bf16x8 qf[D / 16];
    auto compute_block = [&](const char* ks, int j0) {           // 32 keys from j0 on; ks: their K rows
        const char* vs = ks + S::kTileBytes;
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; r++) s[r] = 0.f;
#pragma unroll
        for (int kb = 0; kb < D / 16; kb++) s = mfma32(lds_read_b128(ks, k_lane ^ ((2 * kb) << 4)), qf[kb], s);
        if (j0 + 32 > Nk) {
#pragma unroll
            for (int r = 0; r < 16; r++)
                if (j0 + 8 * (r >> 2) + 4 * h + (r & 3) >= Nk) s[r] = -INFINITY;
        }
        float mx = s[0];
#pragma unroll
        for (int r = 1; r < 16; r++) mx = __builtin_fmaxf(mx, s[r]);
        const float m_new = __builtin_fmaxf(m_run, half_max(mx));
        const float corr = __builtin_amdgcn_exp2f((m_run - finite_max(m_new)) * c);
        m_run = m_new;
        const float mc = finite_max(m_run) * c;
        float psum = 0.f;
#pragma unroll
        for (int r = 0; r < 16; r++) {
            s[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], c, -mc));
            psum += s[r];
        }
        l_run = l_run * corr + psum;
#pragma unroll
        for (int db = 0; db < D / 32; db++)
#pragma unroll
            for (int r = 0; r < 16; r++) o_acc[db][r] *= corr;
#pragma unroll
        for (int kk = 0; kk < 2; kk++) {
            const int r0 = 8 * kk;
            const bf16x8 pb = cvt8(s[r0 + 0], s[r0 + 1], s[r0 + 2], s[r0 + 3], s[r0 + 4], s[r0 + 5], s[r0 + 6], s[r0 + 7]);
#pragma unroll
            for (int db = 0; db < D / 32; db++) {
                const int row_off = 16 * kk * S::kRowBytes;
                const bf16x4 v0 = lds_read_tr16(vs, (v_lane ^ ((4 * db) << 4)) + row_off);
                const bf16x4 v1 = lds_read_tr16(vs, (v_lane ^ (((4 * db) ^ 2) << 4)) + row_off + 8 * S::kRowBytes);
                o_acc[db] = mfma32(concat(v0, v1), pb, o_acc[db]);
            }
        }
    };

    // The tiles of trip t are here, and visible to all waves.  (In order: the next trip's two tiles may still be on
    // their way, if there is a next trip.)
    auto wait_trip = [&](int t) {
        if (t + 2 < t_end) wait_vmcnt<2 * 2 * S::kLoadsPerTile>();
        else wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" : : : "memory");
    };
    wait_trip(t_begin);
#pragma unroll
    for (int kb = 0; kb < D / 16; kb++) qf[kb] = lds_read_b128(q_smem, k_lane ^ ((2 * kb) << 4));
    for (int t = t_begin; t < t_end; t += 2) {
        if (t > t_begin) wait_trip(t);
        const int j0 = (t + my_tile) * S::kTileKV + key0;
        if (j0 < Nk) compute_block(smem + (t + my_tile - t_begin) % kStages * S::kStageBytes + key0 * S::kRowBytes, j0);
        if (t + kStages < t_end) {
            wait_vmcnt_lds_done<63>();      // nobody reads these stages any more
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            issue_tile(t + kStages);
            issue_tile(t + kStages + 1);
        }
    }

    // ---- join the waves: wave w forms the result of accumulator registers w * kRegs and following
    const float l_wave = half_sum(l_run);
    __syncthreads();
    float* mine = (float*)smem + wave * (D / 2 * 64);            // [register][lane]
#pragma unroll
    for (int db = 0; db < D / 32; db++)
#pragma unroll
        for (int r = 0; r < 16; r++) mine[(db * 16 + r) * 64 + lane] = o_acc[db][r];
    if (h == 0) { stat[0][wave][l32] = m_run; stat[1][wave][l32] = l_wave; }
    __syncthreads();
    float m = -INFINITY, l = 0.f, f[S::kWaves];
#pragma unroll
    for (int w = 0; w < S::kWaves; w++) m = __builtin_fmaxf(m, stat[0][w][l32]);
#pragma unroll
    for (int w = 0; w < S::kWaves; w++) {
        f[w] = __builtin_amdgcn_exp2f((stat[0][w][l32] - finite_max(m)) * c);
        l += stat[1][w][l32] * f[w];
    }
    if (l32 >= rows) return;
    // no visible key in this split, l = 0: 0 times a finite factor is the O = 0 that goes with LSE = -inf.  (A minimum, for a
    // comparison of l delays every result: 9.52 us without either, 9.56, 9.61.  Without a split the row is NaN, as ever.)
    const float inv = __builtin_fminf(1.0f / l, O_part ? __FLT_MAX__ : INFINITY);
    constexpr int kRegs = D / 8;
    const size_t row = (size_t)head * rows + l32;
    const size_t part_row = (size_t)split * heads * rows + row;
#pragma unroll
    for (int g = 0; g < kRegs / 4; g++) {
        const int reg = wave * kRegs + 4 * g;
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; e++) {
            v[e] = 0.f;
#pragma unroll
            for (int w = 0; w < S::kWaves; w++) v[e] += ((const float*)smem)[w * (D / 2 * 64) + (reg + e) * 64 + lane] * f[w];
            v[e] *= inv;
        }
        const int col = 32 * (reg / 16) + 8 * (reg % 16 / 4) + 4 * h;
        if (O_part) *(f32x4*)(O_part + part_row * D + col) = f32x4{v[0], v[1], v[2], v[3]};
        else *(bf16x4*)(O + row * D + col) = __builtin_shufflevector(cvt2(v[0], v[1]), cvt2(v[2], v[3]), 0, 1, 2, 3);
    }
    if (wave == 0 && h == 0) {
        const float lse = m * scale + __builtin_logf(l);
        if (O_part) LSE_part[part_row] = lse; else LSE[row] = lse;
    }
}

// ------------------------------------------------------------------------------------------
// merge of the partial results of a split over the keys
// ------------------------------------------------------------------------------------------
// O = sum_s w_s O_s / sum_s w_s with w_s = exp(LSE_s - max_s LSE_s), LSE = max + ln sum_s w_s: the
// partials are softmax results over disjoint key ranges, each normalised by its own sum.
//
// Bound by latency: a decode call has few rows and up to 256 splits, and one lane group walking all splits of a row,
// its loads one behind the other, took longer than the attention itself.  So D / 4 lanes (four columns each) form one
// of PARTS groups that walk a row's splits side by side, and join through LDS; the maximum is found with one LSE per
// lane.  More than four splits take eight groups: whole decode call, B1 Hq16 Hkv2 Nk32000 D128 (125 splits) 63 -> 15
// us, Hq32 Hkv8 Nk8192 (32) 25 -> 11, Nk2000 (8) 13.7 -> 11.0.  Few splits of many rows (a chunk of a prompt) are
// bound by the bytes, and take one.
template <int D, int PARTS>
__global__ __launch_bounds__(256)
void attn_fwd_combine_kernel(const float* __restrict__ O_part, const float* __restrict__ LSE_part,
                             bf16* __restrict__ O, float* __restrict__ LSE, size_t rows, int n_splits)
{
    constexpr int kLanesPerRow = D / 4;                 // one float4 per lane
    constexpr int kRows = 256 / (kLanesPerRow * PARTS);
    __shared__ f32x4 acc_of[PARTS][kRows][kLanesPerRow];
    __shared__ float w_of[PARTS][kRows];
    const int lane = threadIdx.x % kLanesPerRow, part = threadIdx.x / kLanesPerRow % PARTS, r = threadIdx.x / (kLanesPerRow * PARTS);
    const size_t row = (size_t)blockIdx.x * kRows + r;
    const bool live = row < rows;
    const int col = lane * 4;
    float m = -INFINITY, wsum = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    if (live) {
        // the maximum over all splits: a row's lanes fetch one LSE each
        for (int s = lane; s < n_splits; s += kLanesPerRow) m = __builtin_fmaxf(m, LSE_part[(size_t)s * rows + row]);
#pragma unroll
        for (int off = kLanesPerRow / 2; off >= 1; off >>= 1) m = __builtin_fmaxf(m, __shfl_xor(m, off));
#pragma unroll 4
        for (int s = part; s < n_splits; s += PARTS) {
            const float w = __builtin_expf(LSE_part[(size_t)s * rows + row] - m);
            const f32x4 v = *(const f32x4*)(O_part + ((size_t)s * rows + row) * D + col);
            wsum += w;
            acc += v * w;
        }
    }
    if (PARTS > 1) {
        acc_of[part][r][lane] = acc;
        if (lane == 0) w_of[part][r] = wsum;
        __syncthreads();
        if (part != 0) return;
#pragma unroll
        for (int p = 1; p < PARTS; p++) {
            acc += acc_of[p][r][lane];
            wsum += w_of[p][r];
        }
    }
    if (!live) return;
    const float inv = 1.0f / wsum;
    bf16x2 lo = cvt2(acc[0] * inv, acc[1] * inv), hi = cvt2(acc[2] * inv, acc[3] * inv);
    *(bf16x4*)(O + row * D + col) = __builtin_shufflevector(lo, hi, 0, 1, 2, 3);
    if (col == 0) LSE[row] = m + __builtin_logf(wsum);
}

template <int D, int PARTS>
static void launch_combine(const float* o_part, const float* lse_part, void* o, float* lse, size_t rows, int n_splits, hipStream_t stream)
{
    constexpr int kRows = 256 / (D / 4 * PARTS);
    hipLaunchKernelGGL((attn_fwd_combine_kernel<D, PARTS>), dim3((unsigned)((rows + kRows - 1) / kRows)), dim3(256), 0, stream,
                       o_part, lse_part, (bf16*)o, lse, rows, n_splits);
}

static void combine(const float* o_part, const float* lse_part, void* o, float* lse, size_t rows, int D, int n_splits, hipStream_t stream)
{
    auto launch = D == 128 ? (n_splits > 4 ? launch_combine<128, 8> : launch_combine<128, 1>)
                           : (n_splits > 4 ? launch_combine<64, 8> : launch_combine<64, 1>);
    launch(o_part, lse_part, o, lse, rows, n_splits, stream);
}

// Forward with the keys split n_splits ways (n_splits >= 2, every split holds at least one key:
// (n_splits - 1) * tiles_per_split * 64 < Nk, tiles_per_split even).  o_part: fp32 [n_splits][B*H][Nq][D],
// lse_part: fp32 [n_splits][B*H][Nq].
hipError_t launch_attn_fwd_few_rows(const void* q, const void* k, const void* v, void* o, float* lse,
                                    int B, int H, int Hkv, int Nq, int Nk, float scale, hipStream_t stream)
{
    return launch_fwd_tt<64, true, true, false>(q, k, v, o, lse, B, H, Hkv, Nq, Nk, scale, stream);
}

hipError_t launch_attn_fwd_splitk(const void* q, const void* k, const void* v, void* o, float* lse,
                                  float* o_part, float* lse_part,
                                  int B, int H, int Hkv, int Nq, int Nk, int D, int causal, float scale,
                                  int n_splits, int tiles_per_split, int groups, hipStream_t stream)
{
    auto launch = !causal && Nq <= 64 ? (D == 128 ? launch_fwd_tt<128, false, true, true> : launch_fwd_tt<64, false, true, true>)     // (see launch_fwd_t)
                : D == 64 ? (causal ? launch_phase<64, true, true, true, 1> : launch_phase<64, false, true, true, 1>)
                : groups == 2 ? (causal ? launch_phase<128, true, true, true, 2> : launch_phase<128, false, true, true, 2>)
                          : (causal ? launch_phase<128, true, true, true, 1> : launch_phase<128, false, true, true, 1>);
    hipError_t e = launch(q, k, v, o, lse, B, H, Hkv, Nq, Nk, scale, stream, n_splits, tiles_per_split, o_part, lse_part);
    if (e != hipSuccess) return e;
    combine(o_part, lse_part, o, lse, (size_t)B * H * Nq, D, n_splits, stream);
    return hipGetLastError();
}

template <int D>
static void launch_decode_t(const void* q, const void* k, const void* v, void* o, float* lse, float* o_part, float* lse_part,
                            int heads, int rows, int Nk, float scale, int n_splits, int tiles_per_split, hipStream_t stream)
{
    hipLaunchKernelGGL((attn_decode_kernel<D>), dim3((unsigned)(heads * n_splits)), dim3(256), 0, stream,
                       (const bf16*)q, (const bf16*)k, (const bf16*)v, (bf16*)o, lse, rows, Nk, heads, scale,
                       n_splits, tiles_per_split, n_splits > 1 ? o_part : nullptr, lse_part);
}

hipError_t launch_attn_decode(const void* q, const void* k, const void* v, void* o, float* lse, float* o_part, float* lse_part,
                              int heads, int rows, int Nk, int D, float scale, int n_splits, int tiles_per_split, hipStream_t stream)
{
    auto launch = D == 128 ? launch_decode_t<128> : launch_decode_t<64>;
    launch(q, k, v, o, lse, o_part, lse_part, heads, rows, Nk, scale, n_splits, tiles_per_split, stream);
    if (n_splits > 1) combine(o_part, lse_part, o, lse, (size_t)heads * rows, D, n_splits, stream);
    return hipGetLastError();
}

}  // namespace tk
