// Filtered attention backward on the matrix cores (Sec. 3.1, Eq. 3-4), bf16 in,
// fp32 softmax statistics and accumulators.  Two deterministic kernels, no atomics:
//
//   dQ kernel   (Eq. 3 dS*K-hat + Eq. 4 dS*K-check in one pass): a block owns 128
//               kept queries of one (sequence, query head) and walks over ALL key
//               tiles up to the last query's original position; P is rebuilt
//               from the saved LSE, so filtered keys contribute exactly as in
//               the forward pass.
//   dK/dV kernel (Eq. 3): a block owns 128 KEPT keys of one (sequence, QUERY head) and
//               walks over the kept queries at or after them; rows of filtered
//               tokens are never formed.  Kept rows are in position order, so
//               causality is "compact query index >= compact key index".  With
//               grouped heads each query head writes an fp32 partial and a small
//               kernel sums the G partials of a KV head in a fixed order.
//
// Block order: the (head, sequence) index varies fastest and the tile index
// slowest with the heaviest tiles first, so that the 8 XCDs (block id mod 8)
// receive equal shares of every tile weight and the tail of the launch is made
// of light blocks.  K/V (dQ kernel) and Q/dO (dK/dV kernel) tiles go from global
// memory straight into LDS (16 bytes per lane), one tile ahead of the MFMAs.
//
// Operand orientation is chosen so that no score tile ever goes through LDS:
// the dQ kernel forms S^T = K*Q^T (accumulator lane = query, registers = keys),
// which is already the B-operand layout of dQ^T += K^T*dS^T; the dK/dV kernel forms
// S = Q*K^T (lane = key, registers = queries), the B-operand layout of
// dV^T += dO^T*P and dK^T += Q^T*dS.  The first operand of those products has the
// token dimension as K; it is fetched from the same [token][d] LDS tile with
// the LDS transpose read (ds_read_b64_tr_b16).  A lane ends up with four
// neighbouring columns of one row of dQ, dK or dV.
//
// 16x16x32 bf16 MFMA operand layout (lane l, slot = l%16, qd = l/16):
//   A: row = slot,  k = 8*qd + e (e = 0..7)      B: col = slot, k = 8*qd + e
//   D: col = slot,  row = 4*qd + v   (v = 0..3)
// so two accumulators of 16 rows each, packed into one operand, carry rows
// {4qd + e, 16 + 4qd + e}; the transpose reads fetch exactly those rows for the other operand.
// Large attention calls run at the chip's power limit (on all-zero inputs the same instructions take 0.76 to 0.83 of the time), and
// this MFMA moves half the accumulator bytes per flop that the 32x32x16 one does.  It also leaves four registers with the same row
// terms instead of sixteen, so that dP can accumulate from -D on instead of a subtraction per score (with 32x32x16 the sixteen
// registers of -D spilled).  Whole attention call with the larger MFMA and with this one, the other work spread between the MFMAs and their
// order back and forth (what each of these gives stands where it is done), [2 x 2048 of 4096 rows, 32/8 heads, d = 128] 388 and 349 us, [8192 of
// 16384, 24/8] 1879 and 1671, [2 x 4096, 24/8] 732 and 677; d = 64 [4 x 2048, 32/4] 297 and 271, [4915 of 8192, 8/8] 163 and 147,
// [3 x 459 of 1531, 32/4] 55.0 and 51.8.
#include <algorithm>

#include "common.h"
#include "mfma_util.h"

namespace cf {

typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_t;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4_t;
typedef __attribute__((address_space(3))) s16x4_t* lds_s16x4_ptr;

static constexpr float LOG2E = 1.4426950408889634f;

struct AttnParams {
    const bf16_t *q_kept, *k_full, *v_full, *do_kept;
    float* stat;                   // [2][Hq][n_kept]: log2(e)*LSE and -D = -rowsum(dO*O) of every kept row and head
    // The attention output's kept rows; when set, the dQ kernel forms the row terms from them and writes stat (the dK/dV
    // kernel behind it loads 64 rows of a head at a time).  Null: attn_stats_kernel has written stat already.
    const bf16_t* o_kept;
    const float* lse_full;
    const int32_t *idx, *cu_kept;
    bf16_t *dq_kept, *dk_kept, *dv_kept;
    float *dk_part, *dv_part;      // [G/hp][n_kept][Hkv*d] fp32 partials, one per block of hp query heads (G > hp only)
    float* dq_part;                // [ranges][n_kept][Hq*d] fp32 partials (more than one range only)
    // Key ranges that the dQ blocks of a query tile share out (see attn_dq_plan): seven limits of 9 bits, the k-th one the most
    // 128-row tiles with which k + 2 ranges or more are taken.  One word next to the sizes: with the rule itself
    // evaluated here instead a call took 1.1 us more (of 16 at S = 384).  One word for each of the dQ kernel's tiles: a chain on coarse
    // tiles takes longer.
    uint64_t dq_limits_fine, dq_limits_coarse;
    // Up to the first many live rows the dQ blocks take tiles of 64 queries (see attn_dq_kernel), but for those of more than the second
    // and at most the third.
    int dq_fine_rows, dq_coarse_above, dq_coarse_rows;
    // Up to the first many live rows the dK/dV blocks at d = 64 take tiles of 64 keys (attn_dkv64_kernel), but for those of more than the
    // second and at most the third.
    int dkv_fine_rows, dkv_coarse_above, dkv_coarse_rows;
    int dkv_both;                  // both dK/dV kernels of d = 64 are launched: fine tiles are attn_dkv64_kernel's, others attn_dkv_kernel's
    int n_slots;                   // dK/dV blocks that the device holds at a time (the kernel sizes its blocks' work by it)
    int B, S, Hq, Hkv;
    // Nullable, both or none: rotary tables [S][d/2].  dQ and dK leave rotated back to before the rotary embedding, at the original
    // positions of their rows: the pair (c, c + d/2) of a row lies in two registers of one lane where the results are written, and in
    // a thread of the reduction where partials are (a pass of its own over dQ and dK, which also rounds them once
    // more: 16 us at [8192 rows, 32/4 heads of 64] and [4096, 24/8 of 128]).
    const float *rope_cos, *rope_sin;
    int n_kept;                    // rows that the compact buffers are laid out for (the stride of stat and of the partials)
    const int32_t* n_dev;          // nullable: the live row count on the device, at most n_kept
    float scale;
};

static constexpr int DQ_MAX_RANGES = 8, DQ_LIMIT_BITS = 9;
__host__ __device__ inline int dq_ranges(uint64_t limits, int n_rows) {
    const int tiles = (n_rows + 127) / 128;
    int r = 1;
#pragma unroll
    for (int k = 0; k < DQ_MAX_RANGES - 1; ++k) r += tiles <= (int)((limits >> (DQ_LIMIT_BITS * k)) & ((1 << DQ_LIMIT_BITS) - 1)) ? 1 : 0;
    return r;
}

// Query heads of one KV group that a dK/dV block walks through: the largest divisor of the group size G
// that still leaves about two blocks for every one that the device holds at a time (a block costs between one and `tiles` steps
// and blocks are handed out heaviest first, so two per slot already balance); every head more in a block saves that
// block's fixed cost once and one fp32 partial.  A function of the LIVE row count, which only the
// device may know: the dK/dV blocks and the reduction evaluate it themselves and agree.
__host__ __device__ inline int attn_heads_per_block(int n_rows, int Hq, int G, int n_slots) {
    const int64_t tile_rows = (n_rows + 127) / 128;             // key tiles over all sequences, roughly
    for (int c = G; c > 1; --c)
        if (G % c == 0 && tile_rows * (Hq / c) >= 2 * (int64_t)n_slots) return c;
    return 1;
}

// Live rows up to which the dQ blocks take tiles of 64 queries, with the keys of a tile shared out inside the block: up to one
// 128-query tile per CU (d = 128) or one and a half (d = 64).  A lone block's step is a chain of LDS reads, MFMAs, exponentials and
// a barrier: half the step and twice the blocks, which fill the CUs more evenly, for twice the K/V loads.  Whole attention call, over 1500 calls
// of 4 to 64 heads at either d: with 128-255 tiles fine ones are 1.14 times as fast as coarse ones (d = 64) and 1.08 (d = 128), 256-383 tiles 1.12
// and 1.05 (0.75 to 1.36), 384-511 tiles 1.08 and 1.02 (0.83 to 1.27), 512-767 tiles 1.02 and 0.97, more 0.97 and 0.92.  [1377 rows, 32/4 heads,
// d = 64, S = 1531]: 68.3 us coarse, 60.6 fine.  All these calls by these lines: 1.076 (d = 64) and 1.044 times as fast as on coarse tiles alone; the
// better tile in every call would be 1.009 and 1.013 times as fast again, most where one long sequence makes 260 to 500 tiles ([1545 of
// 8085, 32/8 of 128] 273 coarse, as taken, and 214 fine).
// Several sequences need more room (where the rows alone say so, fine tiles are 0.75 to 1.39 times as fast as coarse ones at d = 128, 1.058 in
// the mean, and 0.84 to 1.45 at d = 64, 1.086; where these lines do, 0.957 at worst and 1.089 in the mean, 0.952 and 1.094 at d = 64):
//   * up to twelve key tiles every sequence but the first counts as 48 rows more: it ends in a part of a tile, and blocks that do not
//     fit beside the others do not pay (fine and coarse: [1200 rows in eight sequences, S = 300, 24/8 heads of 128] 56.4 and 52.6 us, [450 in three,
//     S = 300, 64/8] 57.3 and 53.9, d = 64 [768 in eight, S = 320, 64/8] 47.8 and 41.5; [1200 in four, S = 600, 24/8 of 128] 49.1 and 52.5; longer
//     chains even out: [4095 in three, S = 5460, 8/8] 137 and 175);
//   * up to four key tiles further blocks on a CU gain nothing: half the rows, a further sequence as 32 ([768 in four, S = 192,
//     32/32 of 128] 29.7 and 27.2; [400 in four, S = 200, 32/32] 22.1 and 24.7), and all of up to 128 rows a sequence where their blocks
//     take a quarter of the slots at most ([512 in four, S = 256, 32/32] 24.6 and 27.3; eight, 32/8: 32.9 and 32.4);
//   * up to two key tiles (one at d = 64) with no second tile of queries per sequence are a single short step each ([64 rows, S = 64,
//     24/8 of 128] 20.6 and 19.5, S = 128 21.5 and 20.9, d = 64 [64 rows, S = 64, 8/8] 11.9 and 11.6; [90 rows, S = 90, 24/8 of 128] 23.7 and 24.7).
// Where no sequence has a second 128-query tile, in the mean, the coarse blocks of B * Hq tiles all run from the start on two or
// three slots per CU, and fine ones pay while they leave some free (1340 calls of up to 40 such sequences, S from 300 to 2000; fine time
// over coarse, the better one in every call would be 1.007 times as fast as these lines):
//   * 65 to 128 rows each make two blocks of every one: up to 7/8 of the slots at d = 128 (up to 447 blocks 0.76 to 1.12, 0.93 in the mean, 448-479
//     1.01, 512-767 1.11, more 1.21), all at d = 64 (641-767 blocks 0.91, 768-799 0.96, 800-1023 1.11, more 1.15);
//   * 33 to 64 rows each as many blocks of half the work: up to 13/16 of them (d = 128: up to 415 blocks 0.79 to 1.02, 416-447 0.99, 448-511 1.01,
//     more 1.01; d = 64: up to 511 0.70 to 0.95, 512-624 0.99, 640-767 1.02) and again where coarse ones need a second
//     round (d = 64: 0.98; 0.91 to 1.05); up to 32 rows half of a block's waves have nothing to do (0.97 with 416 to 511 blocks at d = 128, 0.96 to 0.99
//     with 512 to 767 at d = 64).
static void attn_dq_fine_rows(const cf_layer_desc& L, AttnParams& p) {
    const int n_cu = compute_units(), tiles = L.d == 64 ? n_cu * 3 / 2 : n_cu;
    const int64_t more = L.B - 1, blocks = (int64_t)L.B * L.Hq, slots = n_cu * (L.d == 64 ? 3 : 2);
    int rows = tiles / L.Hq * 128;
    if (L.S <= 256) rows = (int)std::max<int64_t>(rows / 2 - 32 * more, 4 * blocks <= slots ? std::min<int64_t>(rows, (int64_t)128 * L.B) : 0);
    else if (L.S <= 768) rows = (int)std::max<int64_t>(std::min<int64_t>(rows, tiles * 128 / L.Hq - 48 * more), 0);
    const bool two = 2 * blocks > (L.d == 64 ? slots : slots * 7 / 8);
    int each = blocks > slots * 13 / 16 && blocks <= slots ? 32 : 64;
    if (L.S <= (L.d == 64 ? 64 : 128)) each = 0;
    p.dq_fine_rows = rows;
    p.dq_coarse_above = (int)std::min<int64_t>((int64_t)each * L.B, INT32_MAX);
    p.dq_coarse_rows = (int)std::min<int64_t>((int64_t)(two ? 128 : 64) * L.B, INT32_MAX);
}
__host__ __device__ inline bool attn_dq_fine(const AttnParams& p, int n_live) {
    return n_live <= p.dq_fine_rows && (n_live <= p.dq_coarse_above || n_live > p.dq_coarse_rows);
}

// Live rows up to which the dK/dV blocks at d = 64 take tiles of 64 keys: up to one and a quarter 128-key tiles per
// CU.  Whole attention call on coarse tiles (the better of the two kernels) over fine ones, 1500 calls of 4 to 64 heads: one sequence up to 320 tiles
// 1.08 in the mean (0.97 to 1.21), 320-511 tiles 1.02, more 0.96.  Up to 512 kept rows in a sequence, in the
// mean, each counts as 128 more: it ends in a part of a tile, of which there are twice as many, and short chains make short blocks, whose fixed
// cost counts (fine and coarse: [447 rows in three sequences, S = 298, 64/8 heads] 32.6 and 31.6 us, [1120 in sixteen, S = 1500, 32/4] 90.6 and
// 74.3; [5120 in two, S = 5120, 8/8] 91.9 and 99.8, [1216 of 1280, 32/4] 49.3 and 53.3).  Where the rows alone say so fine tiles are 1.055 times as fast,
// 0.85 at worst; with this 1.064, 0.96; what it leaves out is slower by 4 % in the mean.  (Each as 112, or up to 320 or 704 rows, changes nothing in the
// mean.  Of the rows of a single tile up to 32 gain 1 % by fine ones, 33 to 64 lose 1 and 65 to 128 gain 5.)
static void attn_dkv_fine_rows(const cf_layer_desc& L, AttnParams& p) {
    const int64_t rows = L.d == 64 ? compute_units() * 5 / 4 / L.Hq * 128 : 0;
    const int64_t less = std::max<int64_t>(rows - (int64_t)128 * L.B, 0), few = std::min<int64_t>((int64_t)512 * L.B, rows);
    p.dkv_fine_rows = (int)(few < rows ? rows : less);
    p.dkv_coarse_above = (int)(less < few ? less : rows);
    p.dkv_coarse_rows = (int)few;
}
__host__ __device__ inline bool attn_dkv_fine(const AttnParams& p, int n_live) {
    return n_live <= p.dkv_fine_rows && (n_live <= p.dkv_coarse_above || n_live > p.dkv_coarse_rows);
}

// Key ranges per query tile of the dQ kernel.  Where a batch of few heads (a tensor-parallel share) has few query tiles, each
// of them is a serial chain on a CU of its own: several blocks per tile, one per range of keys, shorten it, at the price of
// fp32 partials and their sum: [2662 of 7479 rows, 4/1 heads, d = 128], 84 tiles, 184 -> 128 us for the whole attention call (coarse ones
// 247 -> 143).
// The most ranges that a batch shape may take, which grid and workspace are sized for: at least 128 keys in a range (192 on
// coarse tiles), about four blocks per CU; with more than one tile per CU at least 1536 keys; none above two.
static int attn_dq_split(const cf_layer_desc& L, bool fine = true) {
    const int64_t tiles = (int64_t)L.Hq * L.B * ceil_div(L.S, 128), n_cu = compute_units();
    if (tiles > 2 * n_cu) return 1;
    int64_t n = 4 * n_cu / tiles;
    const int64_t longest = L.S / (tiles <= n_cu ? (fine ? 128 : 192) : 1536);
    if (n > longest) n = longest;
    return n < 1 ? 1 : (n > DQ_MAX_RANGES ? DQ_MAX_RANGES : (int)n);
}

// The ranges that a call takes of them.  What the partials cost goes with the live rows: 8 bytes per element and range,
// written and read at about 3.5 TB/s, against the chain of S keys, 6.6 ns * d per 64 of them on fine tiles, 9.4 on coarse ones (fitted to chains of
// 32x32x16 MFMAs; with these, over 1155 calls of up to 512 tiles, the best ranges in every call would be 1.011 (d = 128) and 1.005 times as
// fast as those taken; whole tiles take 1.04 times as long).  (With the fine tiles' 6.6 for both, coarse calls would be split too little: [4200 rows, 12/4 heads, d = 64] 157 us
// whole and 142 in two ranges, [3481 of 4096, 16/16] 132 and 124.)  Without KV groups the split
// also costs a launch that would not be there otherwise, about 1 us; with them that launch is there and gains 1 us by a dQ kernel
// that ends sooner.  A gain below 1/64 of the chain is none.  (Decided from the batch shape alone, calls that keep
// most of their tokens would be split as far as sparse ones: 32/32 heads, d = 128, S = 1024, all kept, four ranges 102 us, none 61.)
// In units of 1/16 ns per column: k > 1 ranges gain A(k) - k * part, A(k) = chain - chain/k - launch, part = what
// one range's partials cost; k = 1 counts as a gain of chain / 64.  The k of the largest gain, the smaller one of
// equals, is k or more exactly if some j >= k gains more than every i < k, which is a limit on part and so on the rows.  These
// limits, in tiles of 128 rows (of which a batch that may be split has 512 at most), go to the kernels.
// Returns the ranges that the grid needs: those taken where the host knows the rows, the most there may be where it does not.
static int attn_dq_plan(const cf_layer_desc& L, const RowCount& rows, bool fine, uint64_t& limits) {
    limits = 0;
    const int cap = attn_dq_split(L, fine);
    if (cap == 1) return 1;                         // from here on S <= 64 K
    const int chain = fine ? L.S * 105 / 64 : L.S * 75 / 32, launch = (L.Hq == L.Hkv ? 16000 : -16000) / L.d;
    int A[DQ_MAX_RANGES + 1] = {0, chain / 64};
    for (int k = 2; k <= cap; ++k) A[k] = chain - chain / k - launch;
    auto put = [&](int k, uint64_t v) { limits |= std::min<uint64_t>(v, (1 << DQ_LIMIT_BITS) - 1) << (DQ_LIMIT_BITS * (k - 2)); };
    for (int k = 2; k <= cap; ++k) {
        int most = -1;                              // largest part that takes k or more
        for (int j = k; j <= cap; ++j) {
            int beats = INT32_MAX;
            for (int i = 1; i < k; ++i) {
                const int lead = A[j] - A[i] - 1;
                beats = std::min(beats, lead < 0 ? -1 : lead / (i == 1 ? j : j - i));
            }
            most = std::max(most, beats);
        }
        // part = tiles * 128 rows * Hq * 32 / 875, rounded down
        put(k, most < 0 ? 0 : ((uint64_t)(most + 1) * 875 - 1) / ((uint64_t)L.Hq * 4096));
    }
    if (rows.dev != nullptr) return cap;
    const int taken = dq_ranges(limits, rows.n);
    limits = 0;
    for (int k = 2; k <= taken; ++k) put(k, ~0ull);
    return taken;
}

// Compact rows [begin, end) of sequence b.  The prefix counts are clamped to the live row count, so a
// mask that keeps more tokens than the buffers were sized for cannot send a block past their end.
__device__ __forceinline__ void seq_range(const AttnParams& p, int b, int& begin, int& end) {
    if (p.cu_kept == nullptr) {
        begin = b * p.S;
        end = (b + 1) * p.S;
        return;
    }
    const int n = live_rows(p.n_kept, p.n_dev);
    begin = min(p.cu_kept[b], n);
    end = min(p.cu_kept[b + 1], n);
}

// 16-byte chunk swizzle of a [rows][D] bf16 tile: chunk c of a row lies at c XOR this.  A pass of a ds_read_b128 mixes a chunk of
// rows 0-3 and 12-15 with its neighbour of rows 4-11 (or the other way round, see gemm.hip), and the transpose read of a half
// wave takes two neighbouring chunks of eight rows: with the four blocks of four rows numbered 0, 2, 3, 1 in the chunk's low
// bits both hit every bank once.
template <int D>
__device__ __forceinline__ int tile_swz(int row) {
    const int q = (row >> 2) & 3, low = (((q ^ (q >> 1)) & 1) << 1) | (q >> 1);
    return (D == 128 ? (row & 3) << 2 : ((row >> 1) & 1) << 2) | low;
}

// Per-lane byte offsets of the fragment reads inside a tile.  Row fragments (row lane % 16 as the MFMA's row or column, columns
// ks*32 + 8*(lane/16) on as K) ...
template <int D>
__device__ __forceinline__ unsigned frag_rows_at(int lane, int ks) {
    const int slot = lane & 15;
    return (unsigned)(slot * (D * 2) + (((ks * 4 + (lane >> 4)) ^ tile_swz<D>(slot)) << 4));
}
// ... and token fragments (column nt*16 + lane % 16 as the MFMA's row, rows 4*(lane/16) + {0..3} as half of K: the
// transpose read's address for this lane).
template <int D>
__device__ __forceinline__ unsigned frag_tokens_at(int lane, int nt) {
    const int r = 4 * (lane >> 4) + ((lane & 15) >> 2);
    return (unsigned)(r * (D * 2) + (((nt * 2 + ((lane & 3) >> 1)) ^ tile_swz<D>(r)) << 4) + (lane & 1) * 8);
}

typedef __attribute__((address_space(3))) unsigned char* lds_u8_ptr;
typedef const __attribute__((address_space(3))) u32x4_t* lds_u4_cptr;
typedef const __attribute__((address_space(3))) f32x4_t* lds_f4_cptr;

__device__ __forceinline__ bf16x8_t read_rows(lds_u8_ptr q) { return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<lds_u4_cptr>(q)); }
// rows 4*(lane/16) + {0..3} and those 16 further on
template <int D>
__device__ __forceinline__ bf16x8_t read_tokens(lds_u8_ptr q) {
    typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8_t;
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)q);
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(q + 16 * (D * 2)));
    return __builtin_bit_cast(bf16x8_t, (s16x8_t)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

__device__ __forceinline__ f32x4_t mfma16(bf16x8_t a, bf16x8_t b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ unsigned pack2(float lo, float hi) {
    bf16x2_t v;
    v[0] = (__bf16)lo;
    v[1] = (__bf16)hi;
    return __builtin_bit_cast(unsigned, v);
}

// two accumulators of 16 rows as one operand
__device__ __forceinline__ bf16x8_t pack8(const f32x4_t& a, const f32x4_t& b) {
    return __builtin_bit_cast(bf16x8_t, make_uint4(pack2(a[0], a[1]), pack2(a[2], a[3]), pack2(b[0], b[1]), pack2(b[2], b[3])));
}

// One row of a head, times scale, as bf16: acc[nt] holds columns nt*16 + {0..3} from the lane's first one on, and put(nt, ..) takes
// them.  ROPE: rotated back to before the rotary embedding; rope_cos and rope_sin point to the lane's first column of the row's position.
template <int D, bool ROPE, typename Put>
__device__ __forceinline__ void round_row(const f32x4_t (&acc)[D / 16], float scale, const float* __restrict__ rope_cos,
                                          const float* __restrict__ rope_sin, Put put) {
    constexpr int NT = D / 16;
    auto round = [&](int nt, const f32x4_t& y) __attribute__((always_inline)) { put(nt, make_uint2(pack2(y[0], y[1]), pack2(y[2], y[3]))); };
    if constexpr (ROPE) {
#pragma unroll
        for (int nt = 0; nt < NT / 2; ++nt) {
            const f32x4_t c = *reinterpret_cast<const f32x4_t*>(rope_cos + nt * 16);
            const f32x4_t s = *reinterpret_cast<const f32x4_t*>(rope_sin + nt * 16);
            const f32x4_t a = acc[nt] * scale, b = acc[nt + NT / 2] * scale;
            round(nt, a * c + b * s);
            round(nt + NT / 2, b * c - a * s);
        }
    } else {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) round(nt, acc[nt] * scale);
    }
}
// ... to memory; out: the row's first column of the lane
template <int D, bool ROPE>
__device__ __forceinline__ void store_row(bf16_t* out, const f32x4_t (&acc)[D / 16], float scale, const float* __restrict__ rope_cos,
                                          const float* __restrict__ rope_sin) {
    round_row<D, ROPE>(acc, scale, rope_cos, rope_sin,
                       [&](int nt, uint2 y) __attribute__((always_inline)) { *reinterpret_cast<uint2*>(out + nt * 16) = y; });
}

// global -> LDS: a [64][D] tile goes in as 1 KB wave-loads (16 bytes per lane): wave w, load i fills
// LDS bytes [(4*i + w) KB, +1 KB) of the tile, i.e. 1024/(2D) rows, and a lane fetches the global chunk
// that belongs in its (swizzled) LDS slot.  Rows outside the source's descriptor range arrive as zeros.

// ---------------------------------------------------------------------------
// dQ kernel
// ---------------------------------------------------------------------------
// ROPE here and below: rope_cos and rope_sin are set.  (A template: as a branch behind the loop it cost calls without tables 6 % of
// the dQ kernel's time, through the registers it takes.)
// FINE: tiles of 64 queries; the two waves of a group of 32 take the first and the second 32 keys of every key tile, and their sums
// meet in LDS at the end (see attn_dq_fine_rows).
template <int D, bool ROPE, bool FINE>
__device__ __forceinline__ void attn_dq_block(const AttnParams& p, const uint64_t dq_limits, const int n_live, unsigned char* smem) {
    constexpr int KS = D / 32, NT = D / 16, QT = FINE ? 64 : 128;
    constexpr int TILE = 64 * D * 2;            // one 64-token tile in bytes
    constexpr int NLD = D / 32;                 // wave-loads per wave per tile
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int wave = FINE ? wv & 1 : wv, kw = FINE ? __builtin_amdgcn_readfirstlane(wv >> 1) : 0;   // group of 32 queries; half of the key tiles
    const int slot = lane & 15, qd = lane >> 4;
    const int h = blockIdx.x % p.Hq, b = blockIdx.x / p.Hq, g = h / (p.Hq / p.Hkv);
    const int Nq = p.Hq * D, Nkv = p.Hkv * D;
    int seq_begin, seq_end;
    seq_range(p, b, seq_begin, seq_end);
    const int cnt = seq_end - seq_begin;
    // heaviest (latest) query tiles of the sequence first; the grid is sized for an upper bound of the
    // row count, and the blocks past this sequence's tiles come last in the launch order
    const int seq_tiles = (cnt + QT - 1) / QT;
    const int ranges = dq_ranges(dq_limits, n_live);
    if ((int)blockIdx.y >= seq_tiles || (int)blockIdx.z >= ranges) return;
    const int qt = seq_tiles - 1 - blockIdx.y;
    const int j0 = seq_begin + qt * QT;
    const int rows_in_tile = min(QT, cnt - qt * QT);

    // This lane's two queries, 16 rows apart: their fragments and row terms.  D = rowsum(dO*O) is formed here, from the dO fragments that
    // the kernel holds anyway, unless a pass before had to read O for its compact copy (a pass of its own over dO and O
    // costs 16 us where the dQ kernel gets 6 us slower: [4096 rows, 32 heads, d = 128], 206 us).
    // The loads of both go out before anything waits for one; a query that does not exist takes the rows of the tile's last one (masked below,
    // never stored), unless none of its 16 does.  One after the other, the blocks of tiles with at most 16 rows, which had nothing to load for the
    // second, started earlier than those of the sequence's other tiles and took K and V through the XCD's L2 ahead of them: [7 x 129 of
    // 1085 rows, 32/4 heads, d = 128] call 94.3 us, so 86.2.  2100 calls: 1.006 (d = 128) and 1.010
    // times as fast, 0.98 at worst.
    int jq[2], pos[2];
    bool qvalid[2], some[2];
    float lse2[2], Dq[2];
    bf16x8_t qf[2][KS], dof[2][KS];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int r = wave * 32 + t * 16 + slot;
        qvalid[t] = r < rows_in_tile;
        jq[t] = j0 + min(r, rows_in_tile - 1);
        pos[t] = (p.idx ? p.idx[jq[t]] : jq[t]) - b * p.S;
        const int64_t off_q = (int64_t)jq[t] * Nq + h * D + qd * 8;
        some[t] = wave * 32 + t * 16 < rows_in_tile;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[t][ks] = dof[t][ks] = __builtin_bit_cast(bf16x8_t, make_uint4(0, 0, 0, 0));
        if (some[t]) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                qf[t][ks] = *reinterpret_cast<const bf16x8_t*>(p.q_kept + off_q + ks * 32);
                dof[t][ks] = *reinterpret_cast<const bf16x8_t*>(p.do_kept + off_q + ks * 32);
            }
        }
    }
    if (p.o_kept != nullptr) {
        // summed in the order of attn_stats_kernel, so that both give the same bits: 8 columns in sequence, then a tree
        uint4 of[2][KS];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) of[t][ks] = make_uint4(0, 0, 0, 0);
            if (some[t])
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    of[t][ks] = *reinterpret_cast<const uint4*>(p.o_kept + (int64_t)jq[t] * Nq + h * D + qd * 8 + ks * 32);
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) lse2[t] = p.lse_full[((int64_t)b * p.Hq + h) * p.S + pos[t]] * LOG2E;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            float part[KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                part[ks] = 0.f;
                const uint4 o = of[t][ks], c = __builtin_bit_cast(uint4, dof[t][ks]);
                const unsigned ow[4] = {o.x, o.y, o.z, o.w}, cw[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    part[ks] += __uint_as_float(cw[e] << 16) * __uint_as_float(ow[e] << 16);
                    part[ks] += __uint_as_float(cw[e] & 0xFFFF0000u) * __uint_as_float(ow[e] & 0xFFFF0000u);
                }
            }
#pragma unroll
            for (int o = KS / 2; o > 0; o >>= 1)
#pragma unroll
                for (int ks = 0; ks < o; ++ks) part[ks] += part[ks + o];
            Dq[t] = part[0];
            Dq[t] += __shfl_xor(Dq[t], 32, 64);     // the other quarters of the row's columns
            Dq[t] += __shfl_xor(Dq[t], 16, 64);
            if (qvalid[t] && qd == 0 && blockIdx.z == 0 && kw == 0) {
                p.stat[(int64_t)h * p.n_kept + jq[t]] = lse2[t];
                p.stat[(int64_t)(p.Hq + h) * p.n_kept + jq[t]] = -Dq[t];
            }
        }
    } else {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            lse2[t] = p.stat[(int64_t)h * p.n_kept + jq[t]];
            Dq[t] = -p.stat[(int64_t)(p.Hq + h) * p.n_kept + jq[t]];
        }
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) pos[t] = qvalid[t] ? pos[t] : -1;
    const int jlast = j0 + rows_in_tile - 1;
    const int maxpos = (p.idx ? p.idx[jlast] : jlast) - b * p.S;
    // the block's range of key tiles: all of them, or its share (possibly empty) of a split tile
    const int nkt_all = maxpos / 64 + 1, per = (nkt_all + ranges - 1) / ranges;
    const int kt0 = min((int)blockIdx.z * per, nkt_all), nkt = min(kt0 + per, nkt_all);
    // positions of the wave's last and first query: key tiles past the former are skipped, key tiles
    // that end at or before the latter are visible to every query of the wave and need no mask
    int wave_maxpos = -1, wave_minpos = -1;
    {
        const int wrows = min(32, rows_in_tile - wave * 32);
        if (wrows > 0) {
            const int jw = j0 + wave * 32 + wrows - 1;
            wave_maxpos = (p.idx ? p.idx[jw] : jw) - b * p.S;
            wave_minpos = (p.idx ? p.idx[j0 + wave * 32] : j0 + wave * 32) - b * p.S;
        }
    }
    const float scale2 = p.scale * LOG2E;
    // dP accumulates from -D on, which takes a subtraction per score out of the loop
    f32x4_t negD[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) negD[t] = f32x4_t{-Dq[t], -Dq[t], -Dq[t], -Dq[t]};

    f32x4_t acc[2][NT];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[t][nt][v] = 0.f;

    // K and V of this sequence and KV head: rows are Nkv*2 bytes apart.  A tile is loaded whole: rows past
    // the last query's position are later keys of the same sequence (masked out below) or lie outside
    // the descriptor's range (zeros).
    const i32x4_t rsK = make_rsrc(p.k_full + ((int64_t)b * p.S) * Nkv + g * D, ((int64_t)p.S * Nkv - g * D) * 2);
    const i32x4_t rsV = make_rsrc(p.v_full + ((int64_t)b * p.S) * Nkv + g * D, ((int64_t)p.S * Nkv - g * D) * 2);
    const unsigned lds0 = __builtin_amdgcn_readfirstlane(lds_addr_of(smem));
    // per-lane offset of a tile's first load inside a 64-row tile (row * stride + swizzled chunk): it never
    // changes, and load i lies 4*i*RPL rows further on with the same swizzle term
    constexpr int NCH = D / 8, RPL = 64 / NCH;
    unsigned voff0;
    {
        const int row = wv * RPL + lane / NCH;
        voff0 = (unsigned)row * (unsigned)(Nkv * 2) + (unsigned)(((lane % NCH) ^ tile_swz<D>(row)) << 4);
    }
    const unsigned wave_lds = __builtin_amdgcn_readfirstlane(lds0 + (unsigned)wv * 1024u);   // scalar: the wave's 1 KB slot
    auto issue_kv = [&](int kt, int stage) __attribute__((always_inline)) {
        const unsigned sk = wave_lds + stage * 2 * TILE;
        const unsigned step = (unsigned)(4 * RPL) * (unsigned)(Nkv * 2);
        const unsigned base = (unsigned)(kt * 64) * (unsigned)(Nkv * 2);
#pragma unroll
        for (int i = 0; i < NLD; ++i) dma16(sk + 4 * i * 1024, rsK, voff0 + (base + i * step));
#pragma unroll
        for (int i = 0; i < NLD; ++i) dma16(sk + TILE + 4 * i * 1024, rsV, voff0 + (base + i * step));
    };
    // The other columns' fragments lie at these offsets with two (rows) or three (tokens) bits of the chunk changed.
    const unsigned ra0 = frag_rows_at<D>(lane, 0), ta0 = frag_tokens_at<D>(lane, 0);
    // One 64-key tile in the LDS stage at sk.  MASKED: some key of the tile lies after some query of the
    // wave; the other tiles (most of them) spend no instruction on the mask.
    // One 32-key half of the tile at a time keeps the score registers at 2 x 16.  The LDS fragments of a group of
    // MFMAs are read between the previous ones (one group ahead).
    // key0: the first of the wave's keys in the tile, whose K rows begin at sk.
    auto tile = [&](auto MASKED_, const int key0, const unsigned sk) __attribute__((always_inline)) {
        constexpr bool masked = decltype(MASKED_)::value != 0;
        bf16x8_t fa[2][2], fc[2];
        // slot s: of V (even) or K (odd), 32 columns s / 2; part: group of 16 keys
        auto load_a = [&](int mt, int s, int part) __attribute__((always_inline)) {
            const lds_u8_ptr q = reinterpret_cast<lds_u8_ptr>(sk + (ra0 ^ (unsigned)((s / 2) << 6)));
            fa[s & 1][part] = read_rows(q + ((s & 1 ? 0 : TILE) + (mt * 32 + 16 * part) * (D * 2)));
        };
        auto load_c = [&](int mt, int nt, int buf) __attribute__((always_inline)) {
            fc[buf] = read_tokens<D>(reinterpret_cast<lds_u8_ptr>(sk + (ta0 ^ (unsigned)(nt << 5))) + mt * 32 * (D * 2));
        };
        load_a(0, 0, 0);
        load_a(0, 0, 1);
#pragma unroll
        for (int mt = 0; mt < (FINE ? 1 : 2); ++mt) {
            f32x4_t st[2][2], dpt[2][2];            // [16 keys][16 queries]
#pragma unroll
            for (int s = 0; s < 2 * KS; ++s) {
                const int ks = s / 2;
                const f32x4_t z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const int k16 = m >> 1, t = (m & 1) ^ k16;
                    if (m < 2) {
                        if (s + 1 < 2 * KS) load_a(mt, s + 1, m);
                        else if (m == 0) load_c(mt, 0, 0);
                    }
                    CF_SCHED_FENCE();
                    if (s % 2 == 0) dpt[k16][t] = mfma16(fa[0][k16], dof[t][ks], ks == 0 ? negD[t] : dpt[k16][t]);
                    else st[k16][t] = mfma16(fa[1][k16], qf[t][ks], ks == 0 ? z : st[k16][t]);
                    CF_SCHED_FENCE();
                }
            }
            // dS^T = P^T o (dP^T - D): lane = query, register = key
            bf16x8_t a[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
#pragma unroll
                for (int k16 = 0; k16 < 2; ++k16)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        float pr = __builtin_amdgcn_exp2f(st[k16][t][v] * scale2 - lse2[t]);
                        if (masked) {
                            const int key = key0 + mt * 32 + k16 * 16 + 4 * qd + v;
                            pr = key <= pos[t] ? pr : 0.f;
                        }
                        st[k16][t][v] = pr * dpt[k16][t][v];
                    }
                a[t] = pack8(st[0][t], st[1][t]);
            }
            // dQ^T += K^T * dS^T: lane = query, register = column
#pragma unroll
            for (int c = 0; c < NT; ++c) {
                if (c + 1 < NT) load_c(mt, c + 1, (c + 1) & 1);
                else if (!FINE && mt == 0) { load_a(mt + 1, 0, 0); load_a(mt + 1, 0, 1); }
                CF_SCHED_FENCE();
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const int t = (m ^ c) & 1;
                    acc[t][c] = mfma16(fc[c & 1], a[t], acc[t][c]);
                }
                CF_SCHED_FENCE();
            }
        }
    };

    auto step = [&](const int kt, const int stage) __attribute__((always_inline)) {
        const int key0 = kt * 64 + kw * 32;
        if (key0 <= wave_maxpos) {
            const unsigned sk = lds0 + stage * 2 * TILE + kw * (32 * D * 2);
            // a query that does not exist (a ragged last wave) has position -1 and is masked in every tile
            if (key0 + (FINE ? 31 : 63) <= wave_minpos && wave * 32 + 32 <= rows_in_tile) tile(ic<0>{}, key0, sk);
            else tile(ic<1>{}, key0, sk);
        }
    };
    if (kt0 < nkt) issue_kv(kt0, kt0 & 1);
    wait_vmcnt<0>();
    lds_barrier();
    for (int kt = kt0; kt < nkt; ++kt) {
        if (kt + 1 < nkt) issue_kv(kt + 1, (kt + 1) & 1);
        step(kt, kt & 1);
        wait_vmcnt<0>();
        lds_barrier();
    }

    if constexpr (FINE) {       // the second half of the keys joins the first one's wave; the last barrier has freed the tiles' LDS
        f32x4_t* buf = reinterpret_cast<f32x4_t*>(smem) + wave * (2 * NT * 64) + lane;
        if (kw == 1) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) buf[(t * NT + nt) * 64] = acc[t][nt];
        }
        lds_barrier();
        if (kw == 1) return;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[t][nt] += buf[(t * NT + nt) * 64];
    }
    // dq[query][d]: lane = query, a block's four registers = columns nt*16 + 4*qd on
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int r = wave * 32 + t * 16 + slot;
        if (r >= rows_in_tile) continue;
        const int64_t at = (int64_t)(j0 + r) * Nq + h * D + 4 * qd;
        if (ranges > 1) {       // fp32, unscaled, to the range's own partial (zeros when the range is empty)
            float* part = p.dq_part + (int64_t)blockIdx.z * p.n_kept * Nq + at;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) *reinterpret_cast<f32x4_t*>(part + nt * 16) = acc[t][nt];
            continue;
        }
        const int64_t tab = ROPE ? (int64_t)pos[t] * (D / 2) + 4 * qd : 0;
        store_row<D, ROPE>(p.dq_kept + at, acc[t], p.scale, p.rope_cos + tab, p.rope_sin + tab);
    }
}

template <int D, bool ROPE>
__global__ __launch_bounds__(256, 2) void attn_dq_kernel(AttnParams p) {
    extern __shared__ __align__(16) unsigned char smem[];   // [2 stages][K tile, V tile]
    uint64_t fine = p.dq_limits_fine, coarse = p.dq_limits_coarse;
    asm("" : "+s"(fine), "+s"(coarse));         // fetched with the first arguments, not in a round trip of its own further down
    const int n_live = live_rows(p.n_kept, p.n_dev);
    if (attn_dq_fine(p, n_live)) attn_dq_block<D, ROPE, true>(p, fine, n_live, smem);
    else attn_dq_block<D, ROPE, false>(p, coarse, n_live, smem);
}

// ---------------------------------------------------------------------------
// dK/dV kernel, one block per CU: one key tile and HP query heads per block (d = 64 has a second kernel below)
// ---------------------------------------------------------------------------
// Slot order of an iteration of the kernel's pipeline (2*N positions, N "A" slots and N "C" slots;
// see the kernel): odd iterations alternate A, C; even iterations put all C slots into the first
// 3*N/2 positions, every third of which is an A slot, and the remaining A slots behind them.
__host__ __device__ constexpr bool dkv_is_a(int N, bool even, int p) {
    return even ? (p < 3 * N / 2 ? (p % 3 == 1) : true) : (p % 2 == 0);
}
__host__ __device__ constexpr int dkv_slot_index(int N, bool even, int p) {
    int n = 0;
    for (int q = 0; q < p; ++q) n += (dkv_is_a(N, even, q) == dkv_is_a(N, even, p)) ? 1 : 0;
    return n;
}

// Rows jk of dK and dV: the results, or fp32, unscaled, to the block's own partials; `at`: offset of this lane's first column.
template <int D, bool ROPE>
__device__ __forceinline__ void store_dkv(const AttnParams& p, bool whole, int64_t at, int b, int jk, int qd, const f32x4_t (&dk)[D / 16],
                                          const f32x4_t (&dv)[D / 16]) {
    if (whole) {
        const int64_t tab = ROPE ? (int64_t)((p.idx ? p.idx[jk] : jk) - b * p.S) * (D / 2) + 4 * qd : 0;
        store_row<D, ROPE>(p.dk_kept + at, dk, p.scale, p.rope_cos + tab, p.rope_sin + tab);
        store_row<D, false>(p.dv_kept + at, dv, 1.f, nullptr, nullptr);
    } else {
#pragma unroll
        for (int nt = 0; nt < D / 16; ++nt) {
            *reinterpret_cast<f32x4_t*>(p.dk_part + at + nt * 16) = dk[nt];
            *reinterpret_cast<f32x4_t*>(p.dv_part + at + nt * 16) = dv[nt];
        }
    }
}

// A wave's 32 rows of one head, fp32 or bf16, to `out` (the first row and the head's first column; `stride` elements apart) by way of
// its own 32 * D elements of LDS, into which write(at) puts them, at(row, c) being the c-th 16 bytes of a row.
// Straight from the accumulators neighbouring lanes store to different rows, and such a store takes a cycle a lane, of 16 bytes (fp32) as
// of 8 (bf16): the write-out of a block's fp32 at d = 128 8100 to 9800 cycles (lanes traded so that eight of them write a whole
// 128-byte line: 8500), this way, with neighbouring lanes on neighbouring 16 bytes, 5950.  Where sequences are short that decides.  Whole
// attention call at d = 128, fp32 [3 x 394 of 878 rows, 32/8 heads] 75.5 and 72.7 us, [153 of 307, 32/8] 32.6 and 31.0; bf16 [2 x 137 of
// 144, 32/32] 26.3 and 23.3, [8 x 207 of 350, 16/16] 37.7 and 35.4, [1024 of 4096, 32/32] 106.6 and 104.4.
// A wave with fewer than 32 rows stores them straight, a cycle for every lane that has one: by way of LDS too [5 x 129 of 151, 32/8]
// takes 41.1 us, so 39.7, and [3 x 13 of 48, 16/16] 14.1 and 13.5.
template <int D, typename T, typename Write>
__device__ __forceinline__ void store_rows_by_lds(T* out, int64_t stride, unsigned char* buf, int lane, Write write) {
    constexpr int ROW = D * (int)sizeof(T), LPR = ROW / 16, RPS = 64 / LPR, N = 32 / RPS;   // bytes of and lanes to a row, rows to a store
    auto at = [&](int row, int chunk) __attribute__((always_inline)) {      // eight neighbouring lanes share no bank, either way
        return buf + row * ROW + ((chunk ^ (row & 7)) << 4);
    };
    write(at);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    const int r0 = lane / LPR, c = lane % LPR;
    out += r0 * stride + c * (16 / (int)sizeof(T));
#pragma unroll
    for (int i = 0; i < N; ++i) *reinterpret_cast<u32x4_t*>(out + i * RPS * stride) = *reinterpret_cast<u32x4_t*>(at(r0 + i * RPS, c));
}

template <int D, bool ROPE>
__global__ __launch_bounds__(256, 1) void attn_dkv_kernel(AttnParams p) {
    constexpr int KS = D / 32, NT = D / 16;
    constexpr int TILE = 64 * D * 2;
    constexpr int STAGE = 2 * TILE + 512;       // Q tile, dO tile, lse2[64], -D[64]
    extern __shared__ __align__(16) unsigned char smem[];

    // the wave number is the same in all lanes: saying so keeps everything derived from it in scalar registers
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int slot = lane & 15, qd = lane >> 4;
    const int G = p.Hq / p.Hkv;
    const int n_live = live_rows(p.n_kept, p.n_dev);
    if (D == 64 && p.dkv_both && attn_dkv_fine(p, n_live)) return;      // attn_dkv64_kernel takes these rows
    const int HP = attn_heads_per_block(n_live, p.Hq, G, p.n_slots);
    // The grid is one-dimensional and has a block per (key tile, sequence, query head).  Only nhb * B blocks
    // per key tile are needed; they are numbered first, key tile by key tile (heaviest first), so the blocks
    // without work all come at the end of the launch order instead of between the working ones (a block
    // needs a whole CU's LDS even to find out that it has nothing to do).
    const int nhb = p.Hq / HP;                      // head blocks per sequence
    const int per_tile = nhb * p.B;
    const int kt = blockIdx.x / per_tile, bx = blockIdx.x % per_tile;
    if (kt >= (int)gridDim.x / (p.Hq * p.B)) return;
    const int h0 = (bx % nhb) * HP, b = bx / nhb, g = h0 / G;
    const int Nq = p.Hq * D, Nkv = p.Hkv * D;
    int seq_begin, seq_end;
    seq_range(p, b, seq_begin, seq_end);
    const int cnt = seq_end - seq_begin;
    if (kt * 128 >= cnt) return;                    // early key tiles see the most queries: heaviest first
    const int c0 = seq_begin + kt * 128;            // compact row of the tile's first key
    const int keys_in_tile = min(128, cnt - kt * 128);

    const float scale2 = p.scale * LOG2E;
    const int steps = (seq_end - c0 + 63) / 64;     // query tiles from the first key to the sequence end

    f32x4_t dk[2][NT], dv[2][NT];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) dk[u][nt] = dv[u][nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // Q and dO rows of this sequence from its first key on, the current head's columns (set per head below)
    i32x4_t rsQ, rsO, rsL, rsD;
    auto open_head = [&](int h) __attribute__((always_inline)) {
        rsQ = make_rsrc(p.q_kept + (int64_t)c0 * Nq + h * D, ((int64_t)(seq_end - c0) * Nq - h * D) * 2);
        rsO = make_rsrc(p.do_kept + (int64_t)c0 * Nq + h * D, ((int64_t)(seq_end - c0) * Nq - h * D) * 2);
        rsL = make_rsrc(p.stat + (int64_t)h * p.n_kept + c0, (int64_t)(seq_end - c0) * 4);
        rsD = make_rsrc(p.stat + (int64_t)(p.Hq + h) * p.n_kept + c0, (int64_t)(seq_end - c0) * 4);
    };
    const unsigned lds0 = __builtin_amdgcn_readfirstlane(lds_addr_of(smem));
    // Per-lane byte offsets of the fragment reads inside a 64-row tile, fixed for the whole kernel: a read in the
    // loop is "stage base + this + compile-time offset".
    unsigned ra[KS], ta[NT];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) ra[ks] = frag_rows_at<D>(lane, ks);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) ta[nt] = frag_tokens_at<D>(lane, nt);
    // ---- global -> LDS.  Per-lane offsets of a tile's loads inside a 64-row step (row * stride +
    // swizzled chunk) never change; the step's row offset is added per step.  Rows past the sequence
    // end lie outside the descriptors' ranges and arrive as zeros (their statistics too), which is
    // harmless: P = exp2(0 - 0) = 1 meets dO = 0, and dS = 1 * (0 - 0) = 0.
    constexpr int NCH = D / 8, RPL = 64 / NCH, NLD = 64 / RPL / 4;
    unsigned voff[NLD];
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
        const int row = (4 * i + wave) * RPL + lane / NCH;
        voff[i] = (unsigned)row * (unsigned)(Nq * 2) + (unsigned)(((lane % NCH) ^ tile_swz<D>(row)) << 4);
    }
    auto issue_q = [&](int step, int stage) __attribute__((always_inline)) {
        const unsigned sq = lds0 + stage * STAGE;
        const unsigned base = (unsigned)(step * 64) * (unsigned)(Nq * 2);
#pragma unroll
        for (int i = 0; i < NLD; ++i) dma16(__builtin_amdgcn_readfirstlane(sq + (4 * i + wave) * 1024), rsQ, base + voff[i]);
#pragma unroll
        for (int i = 0; i < NLD; ++i) dma16(__builtin_amdgcn_readfirstlane(sq + TILE + (4 * i + wave) * 1024), rsO, base + voff[i]);
        // row statistics of the 64 queries (every wave issues the same two loads, which keeps the
        // number of loads per wave and step equal)
        const unsigned off = (unsigned)(step * 64 + lane) * 4u;
        dma4(sq + 2 * TILE, rsL, off);
        dma4(sq + 2 * TILE + 256, rsD, off);
    };
    constexpr int LPS = 2 * NLD + 2;                // loads per wave and step
    // this lane's two keys, 16 apart
    int jk[2];
    int tok[2];
    bool kvalid[2];
    bf16x8_t kf[2][KS], vf[2][KS];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        jk[u] = c0 + wave * 32 + u * 16 + slot;
        kvalid[u] = wave * 32 + u * 16 + slot < keys_in_tile;
        tok[u] = kvalid[u] ? (p.idx ? p.idx[jk[u]] : jk[u]) : 0;
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            uint4 a = make_uint4(0, 0, 0, 0), c = make_uint4(0, 0, 0, 0);
            if (kvalid[u]) {
                a = *reinterpret_cast<const uint4*>(p.k_full + (int64_t)tok[u] * Nkv + g * D + ks * 32 + qd * 8);
                c = *reinterpret_cast<const uint4*>(p.v_full + (int64_t)tok[u] * Nkv + g * D + ks * 32 + qd * 8);
            }
            kf[u][ks] = __builtin_bit_cast(bf16x8_t, a);
            vf[u][ks] = __builtin_bit_cast(bf16x8_t, c);
        }
    }
    // The keys' loads lead, their addresses take two more; behind the first rows' loads they come no earlier (2100 calls 0.998 times as fast, [3 x
    // 394 of 878 rows, 32/8 heads] 72.7 us, so 71.7).
    open_head(h0);
    issue_q(0, 0);
    issue_q(1, 1);
    issue_q(2, 2);

    // compact row less 4 * qd from which on a query sees the key; none sees one that does not exist.  The mask is one compare with a constant per
    // value ([950 of 1900 rows, 32/8 heads] 82.0 us with the row formed for each, so 81.6; 900 calls of up to 700 positions 1.004 times as fast)
    const int first_row[2] = {(kvalid[0] ? jk[0] : INT32_MAX) - 4 * qd, (kvalid[1] ? jk[1] : INT32_MAX) - 4 * qd};

    // ---- the pipeline.  The query rows go by in HALVES of 32 (two per 64-row step / LDS stage).  A
    // half n needs three kinds of work: A(n) = S and dP (8*KS MFMAs against the wave's K and V
    // fragments), B(n) = P and dS from them (vector ALU: exp2, mask, products, packing), C(n) = dV and
    // dK (4*NT MFMAs).  A wave runs alone on its SIMD, so nothing overlaps unless the instruction
    // stream interleaves it: ITERATION t issues A(t+1), B(t) and C(t-1) together, one softmax value
    // (two at d = 64) and the LDS reads of a later slot spread over the four MFMAs of a slot, a quarter ahead of each, so that in the steady
    // state the matrix core runs back to back while the exponentials of the half before and the
    // fragment reads of the slots ahead proceed under it.  Fragment reads go through a ring of four
    // register pairs and are issued three slots ahead of their MFMAs, across iteration boundaries
    // too (the LDS answers a read in a few hundred cycles when four waves keep it busy; a single slot
    // of lookahead left every group waiting for it).
    // A slot = four MFMAs, two fragments by both groups u of 16 keys: A slot s = {S[q][u] += Qfrag[q] * K[u][ks]} (s even) or
    // {dP[q][u] += dOfrag[q] * V[u][ks]} (odd) for both groups q of 16 queries, ks = s / 2 the 32 columns; C slot c = {dV[u][nt] +=
    // dOtokens[nt] * P[u]} (even) or {dK[u][nt] += Qtokens[nt] * dS[u]} (odd) for two blocks nt of 16 columns.  Back and forth: an MFMA
    // shares an operand with the one before it and the other with the one after (see gemm.hip; here and in the dQ kernel: [2 x 2048 of 4096
    // rows, 32/8 heads] call 349 and 345 us, [8192 of 16384, 24/8] 1663 and 1640).  dP accumulates from -D on.
    // Iterations come in pairs (even t = 2s, odd t = 2s+1) so that stage halves are compile-time.  In
    // the even iteration all C slots come first (with a third of the A slots between them): after
    // them no wave reads stage s-1 any more, so ONE barrier there both frees that stage for the loads
    // of step s+3 and publishes step s+1 (awaited just before it), whose rows the odd iteration's A
    // slots read.  Accumulation order of every output element is that of a plain loop over the rows.
    constexpr int NP = 2 * NT;                      // slots per iteration (NT A slots, NT C slots)
    constexpr int VPS = 16 / NP;                    // softmax values per slot
    constexpr int LOOK = NT >= 8 ? 3 : 2, RING = 4;     // the reads issued for the next iteration must follow the barrier
    static_assert(2 * KS == NT && NP % RING == 0 && (16 % NP) == 0 && NP - LOOK >= 3 * NT / 2, "slot layout");

    f32x4_t st[2][2][2], dpt[2][2][2];              // S / dP of the half being accumulated and of the one in B, by parity: [q][u]
    unsigned ap[2][2][4], ads[2][2][4];             // packed P and dS, [half parity][u]
    bf16x8_t op[RING][2];                           // fragment pairs on their way to the MFMAs
    f32x4_t lq[2], nd[2];                           // log2(e)*LSE of the queries of group q of the half in B, -D of the half in A
    const f32x4_t z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 8; ++i) st[i >> 2][(i >> 1) & 1][i & 1] = dpt[i >> 2][(i >> 1) & 1][i & 1] = z;

    // is position p of an (even / odd) iteration an A slot, and which A or C slot is it
    constexpr auto is_a = [](bool even, int p) constexpr { return dkv_is_a(NT, even, p); };
    constexpr auto slot_index = [](bool even, int p) constexpr { return dkv_slot_index(NT, even, p); };
    // reads of an A slot (row fragments of Q and dO, half hf of the stage at sb) or of a C slot (token
    // fragments) into ring entry r
    // (part: group q of queries or block of columns; -D goes with the first fragments of dO)
    auto read_a = [&](unsigned sb, int hf, int s, int r, int part) __attribute__((always_inline)) {
        const int row = hf * 32 + part * 16;
        op[r][part] = read_rows(reinterpret_cast<lds_u8_ptr>(sb + ra[s / 2]) + ((s & 1 ? TILE : 0) + row * (D * 2)));
        if (s == 1)
            nd[part] = *reinterpret_cast<lds_f4_cptr>(reinterpret_cast<lds_u8_ptr>(sb + 2 * TILE + 16 * qd) + (64 + row) * 4);
    };
    auto read_c = [&](unsigned sb, int hf, int c, int r, int part) __attribute__((always_inline)) {
        op[r][part] = read_tokens<D>(reinterpret_cast<lds_u8_ptr>(sb + ta[(c & ~1) + part]) + ((c & 1 ? 0 : TILE) + hf * 32 * (D * 2)));
    };
    // log2(e)*LSE of this lane's queries (4*qd on) of group q of half hf of the stage at sb
    auto read_lse = [&](unsigned sb, int hf, int q) __attribute__((always_inline)) {
        lq[q] = *reinterpret_cast<lds_f4_cptr>(reinterpret_cast<lds_u8_ptr>(sb + 2 * TILE + 16 * qd) + (hf * 32 + q * 16) * 4);
    };
    // P and dS of value v (key group v / 8, query 16*(v/4 % 2) + 4*qd + v%4 of half t): lane = key, register = query
    auto soft_p = [&](int par, int v, const int (&lim)[2], auto MASKED) __attribute__((always_inline)) {
        constexpr bool masked = decltype(MASKED)::value != 0;
        const int u = v >> 3, q = (v >> 2) & 1, e = v & 3;
        float pr = __builtin_amdgcn_exp2f(st[par][q][u][e] * scale2 - lq[q][e]);
        if (masked) pr = 16 * q + e >= lim[u] ? pr : 0.f;
        st[par][q][u][e] = pr;
    };
    auto soft_ds = [&](int par, int v) __attribute__((always_inline)) {
        const int u = v >> 3, q = (v >> 2) & 1, e = v & 3;
        dpt[par][q][u][e] *= st[par][q][u][e];
        if (e & 1) {
            ap[par][u][2 * q + (e >> 1)] = pack2(st[par][q][u][e - 1], st[par][q][u][e]);
            ads[par][u][2 * q + (e >> 1)] = pack2(dpt[par][q][u][e - 1], dpt[par][q][u][e]);
        }
    };
    auto operand = [](const unsigned (&w)[4]) __attribute__((always_inline)) {
        return __builtin_bit_cast(bf16x8_t, make_uint4(w[0], w[1], w[2], w[3]));
    };
    // One iteration (see above).  KIND 0: steady state; 1: the very first iteration (no half before it:
    // the C slots' MFMAs are left out, their reads are harmless); 2: the drain after the last half
    // (only the C slots' MFMAs).
    auto iteration = [&](auto EVEN_, auto MASKED, auto KIND_, const int s) __attribute__((always_inline)) {
        constexpr bool EVEN = decltype(EVEN_)::value != 0;
        constexpr int KIND = decltype(KIND_)::value;
        constexpr int hfA = EVEN ? 1 : 0, hfB = EVEN ? 0 : 1, hfC = EVEN ? 1 : 0;
        constexpr int parA = EVEN ? 1 : 0, parB = EVEN ? 0 : 1, parC = EVEN ? 1 : 0;    // parity of halves t+1, t, t-1
        const unsigned sbA = lds0 + (unsigned)((EVEN ? s : s + 1) & 3) * STAGE;
        const unsigned sbB = lds0 + (unsigned)(s & 3) * STAGE;
        const unsigned sbC = lds0 + (unsigned)((EVEN ? s + 3 : s) & 3) * STAGE;
        // the iteration after this one (the fragment reads of its first slots are issued here)
        constexpr int hfA_n = EVEN ? 0 : 1, hfB_n = EVEN ? 1 : 0, hfC_n = EVEN ? 0 : 1;
        const unsigned sbA_n = lds0 + (unsigned)((s + 1) & 3) * STAGE;
        const unsigned sbB_n = lds0 + (unsigned)((EVEN ? s : s + 1) & 3) * STAGE;
        const unsigned sbC_n = lds0 + (unsigned)(s & 3) * STAGE;
        // the mask as a compare with a constant per value: first row of half t that sees this lane's keys, less the lane's 4 * qd
        const int qrow0 = c0 + (2 * s + (EVEN ? 0 : 1)) * 32;       // compact row of the first query of half t
        const int lim[2] = {first_row[0] - qrow0, first_row[1] - qrow0};
        static_for<NP>([&](auto P) __attribute__((always_inline)) {
            constexpr int pp = decltype(P)::value;
            if constexpr (EVEN && pp == 3 * NT / 2 && KIND != 2) {
                // every C slot of this iteration has its fragments: nobody reads stage s-1 any more
                wait_vmcnt<LPS>();          // step s+1 has landed; step s+2 may be in flight
                lds_barrier();
                issue_q(s + 3, (s + 3) & 3);
            }
            // Ahead of each of the slot's four MFMAs go a quarter of what else there is to do: the fragment reads of the slot LOOK
            // positions ahead (0, 1) and softmax values of half t, with the next group's row terms fetched ahead (2, 3).  An MFMA
            // takes 16 cycles, four issue slots: in front of the four together, the matrix core waited for all of it ([2 x 2048 of 4096 rows, 32/8 heads, d =
            // 128] call 356 us, so 342; [4800 of 8000, 4/1] 228 and 209; [8192 of 16384, 24/8] 1716 and 1637).
            static_for<4>([&](auto M_) __attribute__((always_inline)) {
                constexpr int m = decltype(M_)::value;
                if constexpr (m < 2) {
                    constexpr int q = pp + LOOK;
                    if constexpr (q < NP) {
                        if constexpr (is_a(EVEN, q)) read_a(sbA, hfA, slot_index(EVEN, q), q % RING, m);
                        else read_c(sbC, hfC, slot_index(EVEN, q), q % RING, m);
                    } else if constexpr (KIND != 2) {
                        constexpr int qn = q - NP;
                        if constexpr (is_a(!EVEN, qn)) read_a(sbA_n, hfA_n, slot_index(!EVEN, qn), q % RING, m);
                        else read_c(sbC_n, hfC_n, slot_index(!EVEN, qn), q % RING, m);
                    }
                } else if constexpr (KIND != 2) {
                    constexpr int v = pp * VPS + (VPS == 2 ? m - 2 : 0);
                    if constexpr (VPS == 2 || m == 2) {
                        if constexpr (v == 0) read_lse(sbB, hfB, 1);
                        if constexpr (v == 12) read_lse(sbB_n, hfB_n, 0);
                        soft_p(parB, v, lim, MASKED);
                    }
                    if constexpr (VPS == 2 || m == 3) soft_ds(parB, v);
                }
                CF_SCHED_FENCE();
                constexpr int f = m >> 1, u = (m & 1) ^ f;      // fragment of the slot, group of keys
                if constexpr (is_a(EVEN, pp)) {
                    if constexpr (KIND != 2) {
                        constexpr int s = slot_index(EVEN, pp), ks = s / 2;
                        // Inline assembly keeps S and dP in the VGPR file, where the softmax arithmetic reads them:
                        // with the builtin the register allocator accumulates them in AGPRs and copies all 32
                        // registers of a half out again, one v_accvgpr_read each.  The price is that the compiler
                        // no longer sees these MFMAs' latency.  A softmax step reads a value five MFMAs or more after the last one that
                        // writes it (S is complete a slot before dP).  The allocator must not copy unfinished results either, which gave
                        // wrong values in a variant of this loop: test_kernel_code.py reads the built code for both.
                        if constexpr (s % 2 == 0) {
                            if constexpr (ks == 0)
                                asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(st[parA][f][u]) : "v"(op[pp % RING][f]), "v"(kf[u][ks]));
                            else
                                asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(st[parA][f][u]) : "v"(op[pp % RING][f]), "v"(kf[u][ks]));
                        } else {
                            if constexpr (ks == 0)
                                asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %3" : "=&v"(dpt[parA][f][u]) : "v"(op[pp % RING][f]), "v"(vf[u][ks]), "v"(nd[f]));
                            else
                                asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(dpt[parA][f][u]) : "v"(op[pp % RING][f]), "v"(vf[u][ks]));
                        }
                    }
                } else if constexpr (KIND != 1) {
                    constexpr int c = slot_index(EVEN, pp), nt = (c & ~1) + f;
                    if constexpr (c % 2 == 0) dv[u][nt] = mfma16(op[pp % RING][f], operand(ap[parC][u]), dv[u][nt]);
                    else dk[u][nt] = mfma16(op[pp % RING][f], operand(ads[parC][u]), dk[u][nt]);
                }
                // -D keeps its registers into the next slot with MFMAs after the one that reads it (the very first iteration has none in
                // C slots): the vector ALU must not write to them while an MFMA reads them, and three more have started by then
                if constexpr (m == 2 && KIND == 1) {
                    if constexpr (is_a(EVEN, pp) && slot_index(EVEN, pp) == 2) asm volatile("" : : "v"(nd[0]), "v"(nd[1]));
                } else if constexpr (m == 2 && pp > 0 && KIND == 0) {
                    if constexpr (is_a(EVEN, pp - 1) && slot_index(EVEN, pp - 1) == 1) asm volatile("" : : "v"(nd[0]), "v"(nd[1]));
                }
                CF_SCHED_FENCE();
            });
        });
    };

    // The block walks through HP query heads of its KV group one after the other: the K and V fragments
    // and the dK / dV accumulators stay in registers, only the Q / dO / statistics stream changes, so
    // the group's sum over these heads costs no partial buffer and a tile's fixed costs (fragment fetch,
    // write-out) are paid once per HP heads.
    for (int hi = 0; hi < HP; ++hi) {
    // Ring of four stages: the loads of step s+3 are issued in pair s, into the stage that step s-1
    // used.  Steps past the end are issued as well (every row out of range: zero fill), so the number
    // of loads in flight is the same in every pair.
    if (hi > 0) {
        lds_barrier();                              // every wave is done with the previous head's stages
        open_head(h0 + hi);
        issue_q(0, 0);
        issue_q(1, 1);
        issue_q(2, 2);
    }
    // Everything is waited for here, not only stage 0: the K and V fragments above come from ordinary
    // loads, and as long as the compiler cannot see them completed ahead of the loop it guards their
    // first use inside the loop with a wait of its own, which the hardware applies to the loads just
    // issued as well: every pair would then wait out a whole global-memory latency.
    wait_vmcnt<0>();
    lds_barrier();
    // head: A(0), then the row terms and the fragment reads that the first iteration starts with
    {
        static_for<NT>([&](auto S_) __attribute__((always_inline)) {
            constexpr int s = decltype(S_)::value, ks = s / 2;
            read_a(lds0, 0, s, s % RING, 0);
            read_a(lds0, 0, s, s % RING, 1);
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int q = m >> 1, u = (m & 1) ^ q;
                if (s % 2 == 0) st[0][q][u] = mfma16(op[s % RING][q], kf[u][ks], ks == 0 ? z : st[0][q][u]);
                else dpt[0][q][u] = mfma16(op[s % RING][q], vf[u][ks], ks == 0 ? nd[q] : dpt[0][q][u]);
            }
        });
        read_lse(lds0, 0, 0);
        static_for<LOOK>([&](auto Q_) __attribute__((always_inline)) {
            constexpr int q = decltype(Q_)::value;
            static_for<2>([&](auto M_) __attribute__((always_inline)) {
                constexpr int m = decltype(M_)::value;
                if constexpr (is_a(true, q)) read_a(lds0, 1, slot_index(true, q), q % RING, m);
                else read_c(lds0 + 3 * STAGE, 1, slot_index(true, q), q % RING, m);     // a half that does not exist: never used
            });
        });
        CF_SCHED_FENCE();
    }
    // MASKED: the pair may hold queries that lie before some of the tile's keys (the first two steps
    // of a tile) or the tile has fewer than 128 keys; every later pair of a full tile sees all of its
    // keys and spends no instruction on the mask.
    const int masked_steps = keys_in_tile < 128 ? steps : min(steps, 2);
    iteration(ic<1>{}, ic<1>{}, ic<1>{}, 0);
    iteration(ic<0>{}, ic<1>{}, ic<0>{}, 0);
    int s = 1;
    for (; s < masked_steps; ++s) {
        iteration(ic<1>{}, ic<1>{}, ic<0>{}, s);
        iteration(ic<0>{}, ic<1>{}, ic<0>{}, s);
    }
    for (; s < steps; ++s) {
        iteration(ic<1>{}, ic<0>{}, ic<0>{}, s);
        iteration(ic<0>{}, ic<0>{}, ic<0>{}, s);
    }
    iteration(ic<1>{}, ic<0>{}, ic<2>{}, steps);     // drain: C of the last half
    wait_vmcnt<0>();                                // the zero-fill loads of the steps past the end
    }

    constexpr int HALF = 32 * D * 4;
    static_assert(4 * 2 * HALF <= 4 * STAGE, "the four waves' rows lie over the stages");
    const bool whole = G == HP;
    const int64_t part = whole ? 0 : (int64_t)((h0 - g * G) / HP) * p.n_kept * Nkv;
    lds_barrier();                                  // every wave is done with the stages, and so are its loads
    if (keys_in_tile < wave * 32 + 32) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
            if (kvalid[u]) store_dkv<D, ROPE>(p, whole, part + (int64_t)jk[u] * Nkv + g * D + 4 * qd, b, jk[u], qd, dk[u], dv[u]);
        return;
    }
    unsigned char* const buf = smem + wave * (2 * HALF);
    const int64_t at0 = part + (int64_t)(c0 + wave * 32) * Nkv + g * D;
    if (whole) {
        auto rounded = [&](const f32x4_t (&acc)[2][NT], float scale, auto ROPE_) __attribute__((always_inline)) {
            return [&, scale](auto at) __attribute__((always_inline)) {
                constexpr bool rope = decltype(ROPE_)::value != 0;
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    // (tok, not loaded again: without the condition of the first load the compiler made one of both and the loops divergent, 148 us
                    // where the 3B adapter layer's kernel takes 127.5)
                    const int64_t tab = rope ? (int64_t)(tok[u] - b * p.S) * (D / 2) + 4 * qd : 0;
                    round_row<D, rope>(acc[u], scale, p.rope_cos + tab, p.rope_sin + tab, [&](int nt, uint2 y) __attribute__((always_inline)) {
                        *reinterpret_cast<uint2*>(at(u * 16 + slot, nt * 2 + (qd >> 1)) + (qd & 1) * 8) = y;
                    });
                }
            };
        };
        store_rows_by_lds<D>(p.dk_kept + at0, Nkv, buf, lane, rounded(dk, p.scale, ic<ROPE>{}));
        store_rows_by_lds<D>(p.dv_kept + at0, Nkv, buf + HALF, lane, rounded(dv, 1.f, ic<0>{}));
    } else {
        auto plain = [&](const f32x4_t (&acc)[2][NT]) __attribute__((always_inline)) {
            return [&](auto at) __attribute__((always_inline)) {
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) *reinterpret_cast<f32x4_t*>(at(u * 16 + slot, nt * 4 + qd)) = acc[u][nt];
            };
        };
        store_rows_by_lds<D>(p.dk_part + at0, Nkv, buf, lane, plain(dk));
        store_rows_by_lds<D>(p.dv_part + at0, Nkv, buf + HALF, lane, plain(dv));
    }
}

// ---------------------------------------------------------------------------
// dK/dV kernel at d = 64: two blocks per CU
// ---------------------------------------------------------------------------
// The same work split as attn_dkv_kernel (128 kept keys and HP query heads per block, halves of 32 queries), but at
// d = 64 accumulators, K/V fragments and scores of a wave take half the registers, so two waves fit a SIMD and
// overlap each other's matrix, vector and LDS phases; a plain order of the phases is then better than the software pipeline
// that a lone wave needs, as long as there are two blocks for every CU and more to follow: whole attention call at d = 64, this
// kernel and the pipelined one, [8192 rows, 32/32 heads, S = 2048] 243 and 281 us, [4096, 64/64, S = 1024] 161 and 193.  Fragment reads
// run one group of four MFMAs ahead.  The accumulation order of every element is that of the pipelined kernel.
// FINE: 64 keys per block; the two waves of a group of 32 keys take the first and the second 32 queries of every step, and their sums
// meet in LDS at the end: half the step and twice the blocks, as in the dQ kernel (attn_dkv_fine_rows says where).
template <bool ROPE, bool FINE>
__device__ __forceinline__ void attn_dkv64_block(const AttnParams& p, const int n_live, unsigned char* smem) {
    constexpr int D = 64, KS = D / 32, NT = D / 16, KT = FINE ? 64 : 128;
    constexpr int TILE = 64 * D * 2;
    constexpr int STAGE = 2 * TILE + 512;       // Q tile, dO tile, lse2[64], -D[64]
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave = FINE ? wv & 1 : wv, qh = FINE ? wv >> 1 : 0;       // group of 32 keys; half of the steps
    const int slot = lane & 15, qd = lane >> 4;
    const int G = p.Hq / p.Hkv;
    const int HP = attn_heads_per_block(n_live, p.Hq, G, p.n_slots);
    // block numbering as in attn_dkv_kernel: key tile by key tile, blocks without work last
    const int nhb = p.Hq / HP, per_tile = nhb * p.B;
    const int kt = blockIdx.x / per_tile, bx = blockIdx.x % per_tile;
    if (kt >= (int)gridDim.x / (p.Hq * p.B)) return;
    const int h0 = (bx % nhb) * HP, b = bx / nhb, g = h0 / G;
    const int Nq = p.Hq * D, Nkv = p.Hkv * D;
    int seq_begin, seq_end;
    seq_range(p, b, seq_begin, seq_end);
    const int cnt = seq_end - seq_begin;
    if (kt * KT >= cnt) return;
    const int c0 = seq_begin + kt * KT;            // compact row of the tile's first key
    const int keys_in_tile = min(KT, cnt - kt * KT);

    int jk[2];                                      // this lane's two keys, 16 apart
    bool kvalid[2];
    bf16x8_t kf[2][KS], vf[2][KS];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        jk[u] = c0 + wave * 32 + u * 16 + slot;
        kvalid[u] = wave * 32 + u * 16 + slot < keys_in_tile;
        const int64_t tok = kvalid[u] ? (p.idx ? p.idx[jk[u]] : jk[u]) : 0;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            uint4 a = make_uint4(0, 0, 0, 0), c = make_uint4(0, 0, 0, 0);
            if (kvalid[u]) {
                a = *reinterpret_cast<const uint4*>(p.k_full + tok * Nkv + g * D + ks * 32 + qd * 8);
                c = *reinterpret_cast<const uint4*>(p.v_full + tok * Nkv + g * D + ks * 32 + qd * 8);
            }
            kf[u][ks] = __builtin_bit_cast(bf16x8_t, a);
            vf[u][ks] = __builtin_bit_cast(bf16x8_t, c);
        }
    }
    const float scale2 = p.scale * LOG2E;
    const int steps = (seq_end - c0 + 63) / 64;     // query tiles from the first key to the sequence end

    f32x4_t dk[2][NT], dv[2][NT];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) dk[u][nt] = dv[u][nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    const unsigned lds0 = __builtin_amdgcn_readfirstlane(lds_addr_of(smem));
    unsigned ra[KS], ta[NT];                        // per-lane offsets of the fragment reads inside a tile (see attn_dkv_kernel)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) ra[ks] = frag_rows_at<D>(lane, ks);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) ta[nt] = frag_tokens_at<D>(lane, nt);
    // global -> LDS as in attn_dkv_kernel; rows past the sequence end arrive as zeros
    constexpr int NCH = D / 8, RPL = 64 / NCH, NLD = 64 / RPL / 4, LPS = 2 * NLD + 2;
    unsigned voff[NLD];
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
        const int row = (4 * i + wv) * RPL + lane / NCH;
        voff[i] = (unsigned)row * (unsigned)(Nq * 2) + (unsigned)(((lane % NCH) ^ tile_swz<D>(row)) << 4);
    }

    bf16x8_t fa[2][2], fc[2][2];
    // s: 16 queries s / KS, 32 columns s % KS; part 0: of dO, part 1: of Q
    auto load_a = [&](unsigned sb, int hf, int s, int part) __attribute__((always_inline)) {
        fa[s & 1][part] = read_rows(reinterpret_cast<lds_u8_ptr>(sb + ra[s % KS]) + ((part == 0 ? TILE : 0) + (hf * 32 + 16 * (s / KS)) * (D * 2)));
    };
    auto load_c = [&](unsigned sb, int hf, int nt, int part) __attribute__((always_inline)) {
        fc[nt & 1][part] = read_tokens<D>(reinterpret_cast<lds_u8_ptr>(sb + ta[nt]) + ((part == 0 ? TILE : 0) + hf * 32 * (D * 2)));
    };
    // One step of 64 queries in the stage at sb, whose first query is compact row qrow0
    // (FINE: sb and ss, the rows and their statistics, and qrow0 begin at the wave's half)
    auto step = [&](auto MASKED_, const unsigned sb, const unsigned ss, const int qrow0) __attribute__((always_inline)) {
        constexpr bool masked = decltype(MASKED_)::value != 0;
        load_a(sb, 0, 0, 0);
        load_a(sb, 0, 0, 1);
#pragma unroll
        for (int hf = 0; hf < (FINE ? 1 : 2); ++hf) {
            f32x4_t st[2][2], dpt[2][2];            // [16 queries][16 keys]
            f32x4_t lq[2], nd[2];                   // log2(e)*LSE and -D of this lane's queries
            const lds_u8_ptr ps = reinterpret_cast<lds_u8_ptr>(ss + 16 * qd);
#pragma unroll
            for (int q = 0; q < 2; ++q) nd[q] = *reinterpret_cast<lds_f4_cptr>(ps + (64 + hf * 32 + 16 * q) * 4);
#pragma unroll
            for (int s = 0; s < 2 * KS; ++s) {
                const int q = s / KS, ks = s % KS, buf = s & 1;
                const f32x4_t z = {0.f, 0.f, 0.f, 0.f};
                if (s + 1 == 2 * KS)
#pragma unroll
                    for (int i = 0; i < 2; ++i) lq[i] = *reinterpret_cast<lds_f4_cptr>(ps + (hf * 32 + 16 * i) * 4);
#pragma unroll
                for (int m = 0; m < 4; ++m) {       // a fragment read ahead of each of the first two MFMAs
                    const int u = m & 1;
                    if (m < 2) {
                        if (s + 1 < 2 * KS) load_a(sb, hf, s + 1, m);
                        else load_c(sb, hf, 0, m);
                    }
                    CF_SCHED_FENCE();
                    if (m < 2) dpt[q][u] = mfma16(fa[buf][0], vf[u][ks], ks == 0 ? nd[q] : dpt[q][u]);
                    else st[q][u] = mfma16(fa[buf][1], kf[u][ks], ks == 0 ? z : st[q][u]);
                    CF_SCHED_FENCE();
                }
            }
            // P and dS: lane = key, register = query
            bf16x8_t ap[2], ads[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        float pr = __builtin_amdgcn_exp2f(st[q][u][e] * scale2 - lq[q][e]);
                        if (masked) {
                            const bool ok = kvalid[u] && (qrow0 + hf * 32 + 16 * q + 4 * qd + e >= jk[u]);
                            pr = ok ? pr : 0.f;
                        }
                        st[q][u][e] = pr;
                        dpt[q][u][e] *= pr;
                    }
                ap[u] = pack8(st[0][u], st[1][u]);
                ads[u] = pack8(dpt[0][u], dpt[1][u]);
            }
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const int u = m & 1;
                    if (m < 2) {
                        if (nt + 1 < NT) load_c(sb, hf, nt + 1, m);
                        else if (!FINE && hf == 0) load_a(sb, 1, 0, m);
                    }
                    CF_SCHED_FENCE();
                    if (m < 2) dv[u][nt] = mfma16(fc[nt & 1][0], ap[u], dv[u][nt]);
                    else dk[u][nt] = mfma16(fc[nt & 1][1], ads[u], dk[u][nt]);
                    CF_SCHED_FENCE();
                }
            }
        }
    };

    wait_vmcnt<0>();        // the K and V fragments: the counts below are those of the ring's loads alone
    const int masked_steps = keys_in_tile < KT ? steps : min(steps, KT / 64);
    for (int hi = 0; hi < HP; ++hi) {
        const int h = h0 + hi;
        const i32x4_t rsQ = make_rsrc(p.q_kept + (int64_t)c0 * Nq + h * D, ((int64_t)(seq_end - c0) * Nq - h * D) * 2);
        const i32x4_t rsO = make_rsrc(p.do_kept + (int64_t)c0 * Nq + h * D, ((int64_t)(seq_end - c0) * Nq - h * D) * 2);
        const i32x4_t rsL = make_rsrc(p.stat + (int64_t)h * p.n_kept + c0, (int64_t)(seq_end - c0) * 4);
        const i32x4_t rsD = make_rsrc(p.stat + (int64_t)(p.Hq + h) * p.n_kept + c0, (int64_t)(seq_end - c0) * 4);
        // every wave issues the same loads for every step, also past the end (zero fill), so a step is LPS loads of a wave
        auto issue_q = [&](int s, int stage) __attribute__((always_inline)) {
            const unsigned sq = lds0 + stage * STAGE;
            const unsigned base = (unsigned)(s * 64) * (unsigned)(Nq * 2);
#pragma unroll
            for (int i = 0; i < NLD; ++i) dma16(__builtin_amdgcn_readfirstlane(sq + (4 * i + wv) * 1024), rsQ, base + voff[i]);
#pragma unroll
            for (int i = 0; i < NLD; ++i) dma16(__builtin_amdgcn_readfirstlane(sq + TILE + (4 * i + wv) * 1024), rsO, base + voff[i]);
            const unsigned off = (unsigned)(s * 64 + lane) * 4u;
            dma4(sq + 2 * TILE, rsL, off);
            dma4(sq + 2 * TILE + 256, rsD, off);
        };
        if (hi > 0) lds_barrier();                  // every wave is done with the previous head's stages
        issue_q(0, 0);
        issue_q(1, 1);
        issue_q(2, 2);
        for (int s = 0; s < steps; ++s) {
            wait_vmcnt<2 * LPS>();                  // step s has landed; steps s+1 and s+2 may be in flight
            lds_barrier();                          // ... for every wave, and every wave is done with step s-1
            issue_q(s + 3, (s + 3) & 3);
            const unsigned st0 = lds0 + (unsigned)(s & 3) * STAGE, sb = st0 + qh * (32 * D * 2), ss = st0 + 2 * TILE + qh * 128;
            if (s < masked_steps) step(ic<1>{}, sb, ss, c0 + s * 64 + qh * 32);
            else step(ic<0>{}, sb, ss, c0 + s * 64 + qh * 32);
        }
        wait_vmcnt<0>();                            // the zero-fill loads of the steps past the end
    }

    if constexpr (FINE) {
        lds_barrier();                              // every wave is done with the stages
        f32x4_t* buf = reinterpret_cast<f32x4_t*>(smem) + wave * (4 * NT * 64) + lane;
        if (qh == 1) {
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    buf[(u * NT + nt) * 64] = dk[u][nt];
                    buf[((2 + u) * NT + nt) * 64] = dv[u][nt];
                }
        }
        lds_barrier();
        if (qh == 1) return;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                dk[u][nt] += buf[(u * NT + nt) * 64];
                dv[u][nt] += buf[((2 + u) * NT + nt) * 64];
            }
    }
    const bool whole = G == HP;
    const int64_t part = whole ? 0 : (int64_t)((h0 - g * G) / HP) * p.n_kept * Nkv;
#pragma unroll
    for (int u = 0; u < 2; ++u)
        if (kvalid[u]) store_dkv<D, ROPE>(p, whole, part + (int64_t)jk[u] * Nkv + g * D + 4 * qd, b, jk[u], qd, dk[u], dv[u]);
}

template <bool ROPE>
__global__ __launch_bounds__(256, 2) void attn_dkv64_kernel(AttnParams p) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int n_live = live_rows(p.n_kept, p.n_dev);
    if (attn_dkv_fine(p, n_live)) attn_dkv64_block<ROPE, true>(p, n_live, smem);
    else if (!p.dkv_both) attn_dkv64_block<ROPE, false>(p, n_live, smem);
}

// acc += part[0..3], part[half..half+3]
__device__ __forceinline__ void add4x2(const float* __restrict__ part, int half, float (&acc)[8]) {
    const float4 a = *reinterpret_cast<const float4*>(part), b = *reinterpret_cast<const float4*>(part + half);
    acc[0] += a.x; acc[1] += a.y; acc[2] += a.z; acc[3] += a.w;
    acc[4] += b.x; acc[5] += b.y; acc[6] += b.z; acc[7] += b.w;
}

// dk = scale * sum_g dk_part[g], dv = sum_g dv_part[g], and for a split dQ launch dq = scale * sum_z dq_part[z] (one launch
// for both: the smallest kernel costs 5 us), in a fixed order: deterministic.  Blocks below kv_blocks take dk and dv, the others dq.
// A thread sums columns c..c+3 and d/2+c..d/2+c+3 of a head: the pairs of the rotary embedding.
template <int D, bool ROPE>
__global__ __launch_bounds__(256) void attn_reduce_kernel(AttnParams p, int kv_blocks) {
    constexpr int half = D / 2;
    const int n_live = live_rows(p.n_kept, p.n_dev);
    const bool is_q = (int)blockIdx.x >= kv_blocks;
    const int heads = is_q ? p.Hq : p.Hkv;
    const int64_t stride = (int64_t)p.n_kept * heads * D;               // between two partials
    int parts;
    if (is_q) {
        parts = dq_ranges(attn_dq_fine(p, n_live) ? p.dq_limits_fine : p.dq_limits_coarse, n_live);
    } else {
        const int G = p.Hq / p.Hkv;
        parts = G / attn_heads_per_block(n_live, p.Hq, G, p.n_slots);
    }
    if (parts == 1) return;                                             // the dQ or dK/dV blocks wrote the results themselves
    const unsigned u = (blockIdx.x - (is_q ? kv_blocks : 0)) * 256u + threadIdx.x;
    const unsigned rh = u / (D / 8);                                    // row * heads + head
    if ((int64_t)rh >= (int64_t)n_live * heads) return;
    const int c = (int)(u % (D / 8)) * 4;
    const int64_t i = (int64_t)rh * D + c;
    float y[8], dv[8];                                                  // columns c + e, half + c + e
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] = dv[e] = 0.f;
    if (is_q) {
#pragma unroll 4
        for (int z = 0; z < parts; ++z) add4x2(p.dq_part + z * stride + i, half, y);
    } else {
#pragma unroll 2
        for (int z = 0; z < parts; ++z) {
            add4x2(p.dk_part + z * stride + i, half, y);
            add4x2(p.dv_part + z * stride + i, half, dv);
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] *= p.scale;
    if constexpr (ROPE) {
        const int row = (int)(rh / (unsigned)heads);
        const int64_t at = (int64_t)((p.idx ? p.idx[row] : row) % p.S) * half + c;
        const float4 co = *reinterpret_cast<const float4*>(p.rope_cos + at), si = *reinterpret_cast<const float4*>(p.rope_sin + at);
        const float cs[4] = {co.x, co.y, co.z, co.w}, sn[4] = {si.x, si.y, si.z, si.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float a = y[e], b = y[4 + e];
            y[e] = a * cs[e] + b * sn[e];
            y[4 + e] = b * cs[e] - a * sn[e];
        }
    }
    bf16_t* out = is_q ? p.dq_kept : p.dk_kept;
    *reinterpret_cast<uint2*>(out + i) = make_uint2(pack2(y[0], y[1]), pack2(y[2], y[3]));
    *reinterpret_cast<uint2*>(out + i + half) = make_uint2(pack2(y[4], y[5]), pack2(y[6], y[7]));
    if (is_q) return;
    *reinterpret_cast<uint2*>(p.dv_kept + i) = make_uint2(pack2(dv[0], dv[1]), pack2(dv[2], dv[3]));
    *reinterpret_cast<uint2*>(p.dv_kept + i + half) = make_uint2(pack2(dv[4], dv[5]), pack2(dv[6], dv[7]));
}

// stat[0][h][j] = log2(e) * LSE(b, h, position of kept row j); stat[1][h][j] = -D = -sum_c dO*O of
// (row j, head h): the row terms of the FlashAttention backward, laid out so that the 64 rows a
// dK/dV block needs per step are contiguous.  d/8 lanes share one (row, head).
// Only launched where the attention output and the queries are still stored full length (o_full, q_full, with idx):
// the pass reads their kept rows through idx and writes the compact copies o_out / q_out
// that the parameter-gradient GEMM of the output projection and the attention kernels' tile loads
// use (the gathers of the two tensors folded into this read).  In the dQ kernel, whose lanes hold 32-byte pieces of a
// row, the copies cost 35 us more where this pass takes 37 (4096 rows, 32 heads, d = 128).
// parts: dO may lie there; the pass then leaves it in do_kept, rounded.
template <int D>
__global__ __launch_bounds__(256, 8) void attn_stats_kernel(bf16_t* do_kept,
                                                         const float* __restrict__ lse_full,
                                                         const int32_t* __restrict__ idx, int n_max,
                                                         const int32_t* __restrict__ n_dev,
                                                         int Hq, int S, float* __restrict__ stat,
                                                         const bf16_t* __restrict__ o_full, bf16_t* __restrict__ o_out,
                                                         const bf16_t* __restrict__ q_full, bf16_t* __restrict__ q_out,
                                                         NtParts parts) {
    const int n_kept = live_rows(n_max, n_dev);
    constexpr int lanes = D / 8;
    const unsigned pair = (blockIdx.x * 256u + threadIdx.x) / lanes;    // (row, head); a matrix has less than 2^31 vectors
    const bool live = pair < (unsigned)n_kept * (unsigned)Hq;
    float s = 0.f;
    const unsigned j = pair / (unsigned)Hq, h = pair % (unsigned)Hq;
    int per;
    const int np = parts.count(n_kept, per);
    if (live) {
        const int part = (int)(threadIdx.x % lanes) * 8;
        const int64_t at = (int64_t)pair * D + part;
        float a[8], b[8];
        if (__builtin_expect(np > 1, 0)) {
            parts.load(n_kept, np, (int)j, (int)h * D + part, a);
            Vec<bf16_t>::store(do_kept + at, a);
        }
        Vec<bf16_t>::load(do_kept + at, a);
        const int64_t src = ((int64_t)idx[j] * Hq + h) * D + part;
        const uint4 ov = *reinterpret_cast<const uint4*>(o_full + src);
        *reinterpret_cast<uint4*>(o_out + at) = ov;
        *reinterpret_cast<uint4*>(q_out + at) = *reinterpret_cast<const uint4*>(q_full + src);
        const unsigned w[4] = {ov.x, ov.y, ov.z, ov.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            b[2 * i] = __uint_as_float(w[i] << 16);
            b[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) s += a[e] * b[e];
    }
#pragma unroll
    for (int o = lanes >> 1; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (live && threadIdx.x % lanes == 0) {
        const unsigned tok = (unsigned)idx[j], bb = tok / (unsigned)S, pos = tok - bb * (unsigned)S;
        stat[(int64_t)h * n_max + j] = lse_full[((int64_t)bb * Hq + h) * S + pos] * LOG2E;
        stat[(int64_t)(Hq + h) * n_max + j] = -s;
    }
}

bool attn_mfma_supported(const cf_layer_desc& L) {
    return L.dtype == CF_BF16 && (L.d == 64 || L.d == 128);
}

// bytes of fp32 partials behind the row statistics: dK and dV per head block (none for MHA), dQ per key range (split only)
static size_t attn_dkv_partial_bytes(const cf_layer_desc& L, int n_kept) {
    return L.Hq == L.Hkv ? 0 : align_up((size_t)2 * (size_t)(n_kept > 0 ? n_kept : 1) * L.Hq * L.d * sizeof(float), 256);
}
size_t attn_mfma_partial_bytes(const cf_layer_desc& L, int n_kept) {
    if (!attn_mfma_supported(L)) return 0;
    const int split = attn_dq_split(L);
    const size_t dq = split > 1 ? (size_t)split * (size_t)(n_kept > 0 ? n_kept : 1) * L.Hq * L.d * sizeof(float) : 0;
    return attn_dkv_partial_bytes(L, n_kept) + align_up(dq, 256);
}

// The largest attn_mfma_partial_bytes over all batch shapes that can hold n_kept rows.  A launch of `split` ranges has at most
// 4 * CUs / split query tiles, and those are at least Hq * n_kept / 128: split * n_kept * Hq <= 512 * CUs, and split <= 8.
size_t attn_mfma_partial_bound(const cf_layer_desc& L, int n_kept) {
    if (!attn_mfma_supported(L)) return 0;
    const size_t rows = (size_t)(n_kept > 0 ? n_kept : 1);
    size_t split_rows = DQ_MAX_RANGES * rows * L.Hq;
    const size_t most = (size_t)512 * compute_units();
    if (split_rows > most) split_rows = most;
    return attn_dkv_partial_bytes(L, n_kept) + align_up(split_rows * L.d * sizeof(float), 256);
}

template <int D, bool ROPE>
static hipError_t launch_t(AttnParams& p, int dq_cap, const bf16_t* o_full, bf16_t* o_out, const bf16_t* q_full, bf16_t* q_out,
                           const NtParts& do_parts, hipStream_t st) {
    constexpr int smem_dq = 2 * 2 * 64 * D * 2;
    constexpr int smem_dkv = 4 * (2 * 64 * D * 2 + 512);
    const int n_kept = p.n_kept;        // grids cover the upper bound of the row count
    const int max_per_seq = n_kept < p.S ? n_kept : p.S;
    const int tiles = ceil_div(max_per_seq, 128), n_cu = compute_units();
    // dK/dV kernel at d = 64.  Without a third block per CU to follow, the launch lasts as long as its longest chains, and a
    // block that shares its CU from the start walks through its own more slowly than the pipelined kernel does alone: whole call,
    // two per CU and pipelined, both on coarse tiles, [8192 rows, 8/8 heads, S = 8192: 512 blocks] 283 and 266 us, [3072, 16/16: 384] 100 and 91,
    // [2048, 4/4: 64] 57.9 and 54.4; just above the line [4593 rows, 16/16, S = 1531: 576] 76 and 83 us.  Chains of less than
    // 12 tiles are too short for that to make up for two full rounds ([4096, 16/16, S = 1024: 512] 52.2 and 52.7 us).  Over 534 calls on coarse tiles the
    // pipelined kernel is 1.04 times as fast on its side of the line (0.95 at worst), the plain one 1.08 on the other (0.95).
    // On a single tile the two take the same time (13 rows, 16/16: 10.0 and 9.9 us).
    // Only the plain kernel has the fine tiles that few live rows take (attn_dkv_fine_rows).  Both sum in the same order on coarse tiles and walk
    // through one head per block where chains decide, so the choice does not show.  With a device-side count either may be
    // needed: chains of 20 tiles and more launch both, and one of them leaves at once.  Layer calls (H = 64 * heads, F = 2H), the plain kernel alone and
    // both: [7296 of 7680 rows, 8/8 heads] 447 and 424 us, [4500 of 4736, 12/4] 367 and 357, on fine tiles [3840 of 7680] 254 and 256, [1600 of 3200,
    // 16/16] 207 and 210.  With fewer tiles the pipelined kernel gains no more than a launch costs ([1946 of 2048, 32/4] plain 213.4, pipelined 212.6,
    // with 32x32x16 MFMAs).
    const bool chains = (int64_t)p.Hq * p.B * tiles * 4 <= (int64_t)n_cu * (tiles < 12 ? 7 : 8);
    bool paired = D == 64;
    p.dkv_both = 0;
    if (D == 64 && chains && tiles > 1) {
        paired = p.n_dev == nullptr ? attn_dkv_fine(p, n_kept) : p.dkv_fine_rows > 0;
        p.dkv_both = p.n_dev != nullptr && paired && n_kept > p.dkv_coarse_above && tiles >= 20;
    }
    p.n_slots = n_cu * (paired && !p.dkv_both ? 2 : 1);
    static std::atomic<uint64_t> lds_ok_dq{0}, lds_ok_dkv{0}, lds_ok_paired{0};
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(&attn_dq_kernel<D, ROPE>), smem_dq, lds_ok_dq);
    if (e != hipSuccess) return e;
    if (paired) e = allow_dynamic_lds(reinterpret_cast<const void*>(&attn_dkv64_kernel<ROPE>), smem_dkv, lds_ok_paired);
    if (e == hipSuccess && (!paired || p.dkv_both))
        e = allow_dynamic_lds(reinterpret_cast<const void*>(&attn_dkv_kernel<D, ROPE>), smem_dkv, lds_ok_dkv);
    if (e != hipSuccess) return e;
    if (p.o_kept == nullptr) {
        const int64_t total = (int64_t)n_kept * p.Hq * (D / 8);
        attn_stats_kernel<D><<<(int)((total + 255) / 256), 256, 0, st>>>(const_cast<bf16_t*>(p.do_kept), p.lse_full, p.idx, n_kept,
                                                                     p.n_dev, p.Hq, p.S, p.stat, o_full, o_out, q_full, q_out,
                                                                     do_parts);
    }
    // Fine tiles in the grid only where they may be taken: what a block without work costs adds up ([3352 rows in eight sequences, S =
    // 933, 32/4 heads, d = 64]: 97 us with a row of blocks for every fine tile, 92 without).
    auto fine_tiles = [&](bool taken, int fine_rows) {
        return p.n_dev == nullptr && !taken ? 0 : ceil_div(std::min(max_per_seq, fine_rows), 64);
    };
    const int dq_tiles = std::max(tiles, fine_tiles(attn_dq_fine(p, n_kept), p.dq_fine_rows));
    attn_dq_kernel<D, ROPE><<<dim3(p.Hq * p.B, dq_tiles, dq_cap), 256, smem_dq, st>>>(p);
    if (paired) {
        const int dkv_tiles = std::max(p.dkv_both ? 1 : tiles, fine_tiles(attn_dkv_fine(p, n_kept), p.dkv_fine_rows));
        attn_dkv64_kernel<ROPE><<<dim3(p.Hq * p.B * dkv_tiles), 256, smem_dkv, st>>>(p);
    }
    if (!paired || p.dkv_both) attn_dkv_kernel<D, ROPE><<<dim3(p.Hq * p.B * tiles), 256, smem_dkv, st>>>(p);
    const int kv_blocks = p.Hq != p.Hkv ? ceil_div((int64_t)n_kept * p.Hkv * D / 8, 256) : 0;
    const int q_blocks = dq_cap > 1 ? ceil_div((int64_t)n_kept * p.Hq * D / 8, 256) : 0;
    if (kv_blocks + q_blocks > 0) attn_reduce_kernel<D, ROPE><<<kv_blocks + q_blocks, 256, 0, st>>>(p, kv_blocks);
    return hipGetLastError();
}

// o_full / q_full (null or both set, need idx): attention output and queries at full length; their kept
// rows are then copied to o_kept / q_kept (which must be writable buffers) by the row-statistics pass.
// rope_cos / rope_sin: null or the rotary tables, see AttnParams.  do_parts: with o_full, dO may lie there, and do_kept is written.
hipError_t launch_attn_bwd_mfma(const cf_layer_desc& L, float scale, const void* q_kept,
                                const void* k_full, const void* v_full, const void* o_kept,
                                const float* lse_full, const void* do_kept, float* stat,
                                const int32_t* idx, const int32_t* cu_kept, RowCount rows, void* dq_kept,
                                void* dk_kept, void* dv_kept, float* partials, hipStream_t st,
                                const void* o_full, const void* q_full, const float* rope_cos, const float* rope_sin,
                                const NtParts& do_parts) {
    AttnParams p;
    const int n_kept = rows.n;
    p.q_kept = (const bf16_t*)q_kept; p.k_full = (const bf16_t*)k_full; p.v_full = (const bf16_t*)v_full;
    p.do_kept = (const bf16_t*)do_kept; p.o_kept = o_full ? nullptr : (const bf16_t*)o_kept; p.lse_full = lse_full; p.stat = stat; p.idx = idx;
    p.cu_kept = cu_kept; p.dq_kept = (bf16_t*)dq_kept; p.dk_kept = (bf16_t*)dk_kept;
    p.dv_kept = (bf16_t*)dv_kept; p.B = L.B; p.S = L.S; p.Hq = L.Hq; p.Hkv = L.Hkv; p.scale = scale;
    p.rope_cos = rope_cos; p.rope_sin = rope_sin;
    p.n_kept = n_kept;
    p.n_dev = rows.dev;
    attn_dq_fine_rows(L, p);
    const int cap_fine = attn_dq_plan(L, rows, true, p.dq_limits_fine), cap_coarse = attn_dq_plan(L, rows, false, p.dq_limits_coarse);
    const int dq_cap = rows.dev ? std::max(cap_fine, cap_coarse) : (attn_dq_fine(p, n_kept) ? cap_fine : cap_coarse);
    attn_dkv_fine_rows(L, p);
    p.dq_part = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(partials) + attn_dkv_partial_bytes(L, n_kept));
    p.dk_part = partials;
    p.dv_part = partials ? partials + (size_t)n_kept * L.Hq * L.d : nullptr;
    bf16_t* o_out = (bf16_t*)const_cast<void*>(o_kept);
    bf16_t* q_out = (bf16_t*)const_cast<void*>(q_kept);
    if ((o_full != nullptr) != (q_full != nullptr) || (o_full != nullptr && idx == nullptr)) return hipErrorInvalidValue;
    const auto launch = L.d == 64 ? (rope_cos ? launch_t<64, true> : launch_t<64, false>)
                                  : (rope_cos ? launch_t<128, true> : launch_t<128, false>);
    return launch(p, dq_cap, (const bf16_t*)o_full, o_out, (const bf16_t*)q_full, q_out, do_parts, st);
}

}  // namespace cf
