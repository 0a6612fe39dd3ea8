// Host-side launchers implemented by the kernel translation units.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

#include <atomic>

namespace tk {

// Compute units of the current device (persistent kernels size their grid by it).  The attribute is
// queried once per device and cached; a launch then costs one hipGetDevice (a thread-local read).
inline hipError_t compute_unit_count(int* cus) {
    constexpr int kMaxDevices = 64;
    static std::atomic<int> cache[kMaxDevices];      // 0 = not queried yet
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < kMaxDevices) {
        const int hit = cache[dev].load(std::memory_order_relaxed);
        if (hit > 0) { *cus = hit; return hipSuccess; }
    }
    e = hipDeviceGetAttribute(cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess && dev >= 0 && dev < kMaxDevices) cache[dev].store(*cus, std::memory_order_relaxed);
    return e;
}

// Heads that tile_of() walks together.  Without a mask all tiles weigh the same: one head per XCD, the best
// reuse of its L2.  With the causal mask a tile's work grows with its index, and the workgroups of an XCD (32 compute
// units) are best given out longest first: d heads per XCD, as many as keep d * tiles within 96 at D = 128 and 256 at D = 64,
// preferably a divisor of an XCD's share.  (One head after the other gives a compute unit the same tile index of two heads, two long
// ones or two short ones: with the forward's kernel before the present one B2 H16 N2048 D128 62 -> 50 us, B1 Hq32 Hkv8 N3001 111 -> 89 us;
// more heads than this and the L2 and the balance at the end both get worse: the first of these 54 us with 6 heads, 56 us with 8.)
// The limits, timed with the present kernels: at D = 128, of 227 sizes with 128-row tiles, two workgroups to a compute unit, and 112
// with 256-row tiles, one to a unit, 96 takes 1.6 and 1.4 % more than the best of 48 to 384, and the best single one, 160 to 192, 1.1 and
// 1.0 %, with a twelfth of the sizes slower by 2 % and more.  At D = 64, three workgroups to a unit, of 800 sizes with 130 to 8192
// queries 256 takes 0.5 % more than the best of 1 to 384, 96 3.7 %: of the two 256 is faster by 2 % and more in 276, slower in 9;
// us (96, 256): B2 H13 N7808 271, 213; B7 Hq4 Hkv2 N6074 177, 144; B9 Hq26 Hkv13 N995 50, 56; 54 sizes of 8192 to 40000 gain 2.5 % on average.
// Where there is none and the last group would be no more than half as large, its few heads leave the units of an XCD to
// their short end: of six tiles and more the next divisor up to 4 * d is taken, of three or five groups of equal size.  us
// (one head per XCD, a group that leaves a rest, this; before the present kernels): B14 H4 N3584 D128 214, 224, 183; B4 H14 N1832 D128 78, 81, 64; B1
// Hq104 Hkv13 N1179 D64 34, 38, 32; B10 Hq52 Hkv13 N373 D128 48, 54, 47; of 244 such sizes 16 had become slower than with one
// head.  (Of two or four tiles, where long and short ones alternate on a unit either way, the rest does no harm: B5 Hq104
// Hkv13 N256 D128 33, 29.5, in equal groups 32.)
inline int tile_order_heads(int heads, int tiles, bool causal, int D) {
    const int per_xcd = (heads + 7) / 8, limit = D == 64 ? 256 : 96;
    int d = 1;
    if (causal) {
        d = limit / tiles < per_xcd ? limit / tiles : per_xcd;
        if (d < 1) d = 1;
        const int most = d;
        bool found = false;
        for (int e = most; 2 * e > most && !found; e--)
            if (per_xcd % e == 0) { d = e; found = true; }
        if (!found && heads % 8 == 0 && 2 * (per_xcd % most) <= most) {
            if (tiles < 6 && tiles % 2) {
                const int groups = (per_xcd + most - 1) / most;
                d = (per_xcd + groups - 1) / groups;
            }
            for (int e = most + 1; tiles >= 6 && e <= 4 * most && !found; e++)
                if (per_xcd % e == 0) { d = e; found = true; }
        }
    }
    return 8 * d < heads ? 8 * d : heads;
}

// H query heads share Hkv key/value heads in groups of H / Hkv consecutive heads (Hkv == H: plain
// multi-head attention); Nq queries, Nk keys per head (causal: aligned at their ends, Nq <= Nk).
// q, o, d_o, dq: [B,H,Nq,D]; k, v, dk, dv: [B,Hkv,Nk,D]; lse, delta: [B,H,Nq].
hipError_t launch_attn_fwd(const void* q, const void* k, const void* v, void* o, float* lse,
                           int B, int H, int Hkv, int Nq, int Nk, int D, int causal, float scale, hipStream_t stream);

// The same with the kernel of few query rows: D = 64, the causal mask, Nq < Nk.
hipError_t launch_attn_fwd_few_rows(const void* q, const void* k, const void* v, void* o, float* lse,
                                    int B, int H, int Hkv, int Nq, int Nk, float scale, hipStream_t stream);

// The same forward with the keys split n_splits (>= 2) ways and a merge kernel behind it.  o_part: fp32 [n_splits][B*H][Nq][D]; lse_part: fp32 [n_splits][B*H][Nq];
// tiles_per_split: even number of 64-key tiles per split, (n_splits - 1) * tiles_per_split * 64 < Nk.  groups: 2 for workgroups of
// 256 query rows (D = 128, and more than 64 rows or the causal mask), otherwise 1.
hipError_t launch_attn_fwd_splitk(const void* q, const void* k, const void* v, void* o, float* lse,
                                  float* o_part, float* lse_part,
                                  int B, int H, int Hkv, int Nq, int Nk, int D, int causal, float scale,
                                  int n_splits, int tiles_per_split, int groups, hipStream_t stream);

// Decoding on a launch of at most one workgroup a compute unit: `rows` (<= kDecodeRows) query rows for each of `heads` key/value heads, the keys split n_splits (>= 1) ways as
// above.  q, o: [heads, rows, D]; k, v: [heads, Nk, D]; lse: [heads, rows].
constexpr int kDecodeRows = 32;
hipError_t launch_attn_decode(const void* q, const void* k, const void* v, void* o, float* lse, float* o_part, float* lse_part,
                              int heads, int rows, int Nk, int D, float scale, int n_splits, int tiles_per_split, hipStream_t stream);

// Delta_i = sum_d dO_id O_id
hipError_t launch_attn_bwd_delta(const void* o, const void* d_o, float* delta,
                                 int B, int H, int N, int D, hipStream_t stream);

// The dS blocks that the dK/dV kernel can leave behind for launch_attn_bwd_dq_from_ds: one 2 KB block per
// (query head, 128-key tile, 32-query block, wave of 32 keys).  Query blocks per head: the dK/dV kernel walks
// them in pairs from a multiple of 32, so up to two past the last real one.
inline int ds_query_blocks(int Nq) { return Nq / 32 + 2; }
inline size_t ds_spill_bytes(int B, int H, int Nq, int Nk) {
    return (size_t)B * H * (size_t)((Nk + 127) / 128) * (size_t)ds_query_blocks(Nq) * 8192;
}

// Whether the tiles of a causal backward launch are paired, long with short, for equal work per workgroup: not where
// each has a compute unit of its own without: the longest tile alone is then the shorter way, by one tile in `tiles`
// and a start-up.  Whole backward, us, paired and not: B2 Hq16 Hkv4 N1001 D128 98, 80; B2 H12 N700 D64 45, 36; but with
// 32 tiles B1 H8 N4096 D128 215, 223, storing dS 171, 190 (half the compute units hold a higher clock), between 17 and 26 tiles a tenth
// either way, and with two workgroups to a compute unit, two long ones or two short ones, B1 H16 N4096 D64 148, 217.  (A single
// tile has no partner either way, and counts as paired: without a pair the kernels for ragged lengths are taken, B2 Hq128 Hkv16
// N128 D128 44, 51.)
inline bool pair_tiles(long long heads, int tiles, int compute_units) { return heads * tiles > compute_units || tiles > 16 || tiles == 1; }

// Ways to split the queries of a key tile over workgroups of the dK/dV kernel, as far as the units still fit the compute
// units at once (with more units the split only adds the traffic of the partial sums): n_splits in all, of which
// q_splits share the query blocks of a head and n_splits / q_splits the query heads of a group.
//   Heads: the largest divisor of the group that fits.  Fewer than 256 queries are not split: the stream of a unit is
// then short next to the launch of the kernel that adds up.  Whole causal backward, us, unsplit and split: B2 Hq16 Hkv4 N1001
// D128 147, 80; B1 Hq32 Hkv8 N4096 573, 481 (two ways); B1 Hq64 Hkv1 N3000 5380, 640; B1 Hq8 Hkv1 N300 94, 38;
// at D = 64 B1 Hq32 Hkv8 N2048 198, 101.
//   Blocks: with other numbers of queries than keys and no mask (with equal lengths and no groups a head's bits do not
// depend on the number of heads; with a mask the late key tiles have few blocks), down to 512 queries, and only to one
// workgroup a compute unit.  Backward, us: B1 H4 Nq4096 Nk64 D64 87, 24; B1 H8 Nq3000 Nk200 D128 98, 46; but with two
// workgroups to some compute units B4 H16 Nq1000 Nk300 D64 47, 53, and with 150 queries each B2 H16 Nq300 Nk128 20, 25 (the
// last two with an earlier form of the kernel, as such splits are not made).
//   Whether it pays: the partial sums and their launch have to cost less than the shorter streams save (dkdv_us()).
struct DkdvSplits {
    int n_splits, q_splits;
};
// blocks of a head in one of q_splits parts, an even number; the last part may be shorter
__host__ __device__ inline int dkdv_q_chunk(int Nq, int q_splits) { return 2 * (((Nq + 63) / 64 + q_splits - 1) / q_splits); }

// Microseconds of the dK/dV kernel split that way: the longest stream of blocks of a workgroup at 0.7 us a block (D = 64) or
// 1.07 (D = 128), 1.4 times that where two workgroups share a compute unit; a split adds 2 us and its partial sums, written
// and read, at 4 TB/s.  Fitted to 437 backward calls with 256 to 4000 queries for which a split fits, each timed with and without: the choice
// takes 0.08 % more than the better one on average, 9 lose more than 1 %, at most 8.  Splitting wherever the units fit loses up to a
// fifth, us (unsplit, split): B5 Hq32 Hkv16 N268 D64 33, 41 (two workgroups to a compute unit); B3 Hq32 Hkv8 Nq309 Nk1060 D128 causal
// 107, 127 (split tiles are too many to go unpaired, and the pairs are as long as the single tiles were).  The times of the kernel with
// 128-key tiles: none of these calls would take 256-key tiles unsplit, which want more tiles than compute units.
inline double dkdv_us(int B, int H, int Hkv, int Nq, int Nk, int D, bool causal, int compute_units, DkdvSplits p) {
    const int tiles = (Nk + 127) / 128, heads = p.n_splits / p.q_splits;
    const bool paired = causal && pair_tiles((long long)B * Hkv * p.n_splits, tiles, compute_units);
    const int units = paired ? (tiles + 1) / 2 : tiles;
    auto blocks_of = [&](int tile) {            // blocks of a head that a tile's pass streams
        int first = causal ? tile * 128 - (Nk - Nq) : 0;
        first = first > 0 ? first & ~31 : 0;
        const int n = 2 * ((Nq - first + 63) / 64);
        return !causal && n > dkdv_q_chunk(Nq, p.q_splits) ? dkdv_q_chunk(Nq, p.q_splits) : n;
    };
    int longest = blocks_of(0);
    for (int u = 0; paired && u < units; u++) {
        const int n = blocks_of(u) + (tiles - 1 - u >= units ? blocks_of(tiles - 1 - u) : 0);
        if (n > longest) longest = n;
    }
    const double shared = D == 64 && (long long)B * Hkv * units * p.n_splits > compute_units ? 1.4 : 1.0;
    const double sum_us = p.n_splits == 1 ? 0.0 : 2.0 + 16.0 * p.n_splits * B * Hkv * Nk * D / 4.0e6;
    return longest * (double)(H / Hkv / heads) * (D == 64 ? 0.7 : 1.07) * shared + sum_us;
}

// heads_only: a call without memory for the partial sums of split blocks
inline DkdvSplits dkdv_splits(int B, int H, int Hkv, int Nq, int Nk, int D, bool causal, int compute_units, bool heads_only) {
    const int tiles = (Nk + 127) / 128, group = H / Hkv;
    const long long units = (long long)B * Hkv * (causal ? (tiles + 1) / 2 : tiles);
    const long long resident = (long long)compute_units * (D == 64 ? 2 : 1);
    if (Nq < 256) return {1, 1};
    int heads = group;
    while (heads > 1 && (group % heads || units * heads > resident)) heads--;
    int blocks = 1;
    if (!causal && Nq != Nk && !heads_only) {
        const long long fit = compute_units / (units * heads), most = Nq / 512, ways = fit < most ? fit : most;
        blocks = ways < 1 ? 1 : (int)ways;
        const int pairs = (Nq + 63) / 64, chunk = dkdv_q_chunk(Nq, blocks) / 2;
        blocks = (pairs + chunk - 1) / chunk;           // no part is empty
    }
    const DkdvSplits p = {heads * blocks, blocks}, unsplit = {1, 1};
    if (p.n_splits > 1 && dkdv_us(B, H, Hkv, Nq, Nk, D, causal, compute_units, p) >= dkdv_us(B, H, Hkv, Nq, Nk, D, causal, compute_units, unsplit))
        return unsplit;
    return p;
}
// fp32 partial sums of dK and dV
inline size_t dkdv_part_bytes(int B, int Hkv, int Nk, int D, int n_splits) {
    return (size_t)n_splits * 2 * B * Hkv * Nk * D * sizeof(float);
}

// dK, dV (key-tile parallel).  ds != nullptr: also store the dS blocks there (ds_spill_bytes(B, H, Nq, Nk) bytes).
// part != nullptr: n_splits > 1 ways (dkdv_splits(...)), partial sums in part (dkdv_part_bytes(...) bytes).
hipError_t launch_attn_bwd_dkdv(const void* q, const void* k, const void* v, const void* d_o,
                                const float* lse, const float* delta, void* dk, void* dv,
                                int B, int H, int Hkv, int Nq, int Nk, int D, int causal, float scale, hipStream_t stream,
                                void* ds = nullptr, int n_splits = 1, int q_splits = 1, float* part = nullptr);

// dQ = scale * dS K from the blocks a launch_attn_bwd_dkdv call with the same shape arguments stored
hipError_t launch_attn_bwd_dq_from_ds(const void* k, const void* ds, void* dq,
                                      int B, int H, int Hkv, int Nq, int Nk, int D, int causal, float scale, hipStream_t stream);

// dQ (query-tile parallel).  With o != nullptr the kernel computes Delta itself from o and d_o, writes it to
// delta_out (for the dK/dV kernel launched after it) and does not read delta.
hipError_t launch_attn_bwd_dq(const void* q, const void* k, const void* v, const void* d_o,
                              const float* lse, const float* delta, void* dq,
                              int B, int H, int Hkv, int Nq, int Nk, int D, int causal, float scale, hipStream_t stream,
                              const void* o = nullptr, float* delta_out = nullptr);

// bf16 matrix multiply C = A B: A [M,K], B [K,N], C [M,N] row-major; M >= 1, N and K multiples of 8
hipError_t launch_gemm(const void* a, const void* b, void* c, int M, int N, int K, hipStream_t stream);

// rotary positional encoding: x, o [B,H,N,D]; sin, cos [N, D/2]
hipError_t launch_rotary(const void* x, const void* sn, const void* cs, void* o,
                         int B, int H, int N, int D, hipStream_t stream);

// bare MFMA stream (measurement aid): 32 MFMAs per wave per iteration
hipError_t launch_mfma_probe(const void* operands, float* sink, int workgroups, int iters, hipStream_t stream);

}  // namespace tk
