// Dimension-reduced dense GEMMs (Sec. 3.2): next-node gradient dX = dY * W^T and
// parameter gradient dW = X^T * dY on kept rows only.
//
//   mode NT: C[M,N] = sum_seg A[M,K] * B[N,K]^T   (both operands contiguous along K)
//   mode TN: C[M,N] = sum_seg A[K,M]^T * B[K,N]   (both operands contiguous along M / N;
//                                                  K is the kept-token dimension)
// Up to six (A, B, K) segments accumulate into one output tile, which sums
// the gradients of a tensor consumed by several linears without rounding in
// between (e.g. d_gate*Wg^T + d_up*Wu^T).
//
// bf16 path: 16x16x32 bf16 MFMA, fp32 accumulators, 256 threads = 2x2 waves, one
// block per CU.  The block tile is (64*TM) x (64*TN) with wave tiles of
// (32*TM) x (32*TN); three shapes are compiled into one kernel: 256x256 (the
// wave tile with the fewest LDS bytes per MFMA), 256x128 and 128x128; the NT kernel
// also has 256x192, for outputs whose 256x256 tiles would leave CUs idle (a dX of
// 4096 x 3072 is 16 x 12 = 192 such tiles but 16 x 16 = 256 of the narrower ones).
//   * Why the small MFMA.  Under these kernels the chip is power-limited: the shader clock
//     settles at 1.5-1.9 GHz instead of 2.4, and 128 CUs deliver 75 % of what 256 do.
//     What counts is therefore energy per flop, not only cycles: 16x16x32 reads and writes
//     its accumulators half as often per flop as 32x32x16 does, runs at a 14 % higher
//     clock for the same work and gains 3-6 % on the large products, although its
//     16-cycle issue rhythm leaves less room for the other instructions (the matrix
//     cores are busy 72 % of the cycles instead of 77 %).  Fragment reads from LDS cost
//     no cycles any more but about 9 % of the clock.
//   * Tile scheduling.  A launch has as many blocks as CUs; a block walks through its
//     share of the output tiles.  The 256x256 tiles that fill whole rounds of the CUs
//     come first; the tiles of the last, partial round are cut into 2 or 4 sub-tiles
//     when that shortens the tail (a 3.5-round problem takes 3 rounds of full tiles
//     and one of half tiles instead of 4 rounds).  Within each group the 8 XCDs (block
//     id mod 8) take contiguous runs of a band-major tile order, so the blocks resident
//     on one XCD share operand panels in that XCD's L2.  Between two tiles of a block
//     the loads of the next tile's first K-steps are already in flight while the
//     finished tile leaves, and its stores drain under the next tile's MFMAs (the
//     write-out of a tile used to be 13 % of its time).
//   * Operand tiles move in K-steps of 32 through a ring of four 32 KB LDS stages (the 128x128
//     tile: eight of 16 KB, four pairs instead of two, three of them ahead),
//     filled by buffer_load ... lds (16 bytes per lane, no register hop).  K-steps are
//     handled in pairs (64 k: one whole 128-byte line of every NT operand row, eight such
//     lines per load); a pair is loaded two pairs ahead, into the two
//     stages that the barrier of the pair being computed has just retired; completion
//     is tracked with vmcnt.  Ragged edges come from the buffer descriptor's range
//     check, which returns zeros, so there are no branches around loads.
//   * One LDS barrier per 64 K.  A pair is 2*TM sub-steps: one 32-row block of the
//     wave's A rows against all its B columns for one K-step (16 MFMAs in a 128x128 wave
//     tile).  The A fragments of the next sub-step and a share of the B fragments of
//     the next K-step are read ahead of their use, and the instruction stream is laid
//     out by hand: a gap between two MFMAs carries at most one fragment read and one
//     instruction of a load (the write of M0 goes ahead of an MFMA, the load behind it).
//     The loop body is two pairs, which makes every stage a compile-time constant: an
//     LDS read is a loop-invariant per-lane base register plus an instruction offset, a
//     load takes its per-lane offset from a register that is fixed for the whole K
//     segment and its K position from the instruction's scalar offset, so the steady
//     state has no vector ALU instruction besides the MFMAs.
//   * The loads of a pair go out in groups spread over the sub-steps (four groups in
//     NT, three in TN; two cost 4 %): a CU sustains only so many bytes in flight, and a
//     burst of 64 KB stalls the stream.
//   * NT pair: [rows][64 k], 128-byte rows, the 16-byte chunk index of a row XOR-ed with a
//     function of the row chosen so that the 16 lanes that the LDS serves in one pass of a
//     ds_read_b128 hit distinct banks (see nt_swz); a lane of the loading wave picks the
//     global chunk that belongs in its (fixed) LDS slot.
//   * TN stage: [32 k][rows] exactly as in memory, with the 64-byte group index of a
//     k-row XOR-ed with k%4; fragments come out of LDS through the transpose read
//     (ds_read_b64_tr_b16), in the same register layout as the NT ones, so MFMA
//     order and epilogue are shared.  The four k-rows that a group of 16 lanes touches
//     in one transpose read land in four different 64-byte bank groups.
//   * The MFMA is issued with the operands swapped (D = B-frag x A-frag), so a lane
//     ends up with 4 adjacent output columns of one row; the epilogue packs them to
//     bf16 and sends them, 32 rows of the wave tile at a time, through 8 KB of LDS of
//     the wave's own (above the operand stages, which the next tile is filling by
//     then) to full-row 16-byte stores.
// fp32 path (check mode): plain LDS-tiled FMA kernel.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "mfma_util.h"

namespace cf {

static constexpr int MAX_SEG = 6;

struct GemmArgs {
    const void* A[MAX_SEG];
    const void* B[MAX_SEG];
    int K[MAX_SEG];
    int nseg;
    void* C;
    int M, N;
    float beta;
    float alpha;    // the product is scaled by alpha before beta*C is added
    int n_full;     // leading blocks that own a whole 256x256 tile
    int sub;        // the remaining tiles are cut into `sub` (1, 2 or 4) sub-tiles, one block each
    int tile_n;     // 256, or 192 (NT only): every tile is 256x192 and n_full, sub are unused
    // Kept-token count on the device (nullable).  When set, the kept-token dimension handed in by the
    // host (M in mode NT, K[0] in mode TN) is only an upper bound: every block reads the count, takes
    // min(count, bound) for that dimension and, in mode NT, plans the tiles itself (plan_launch).
    const int32_t* n_dev;
    // Mode NT, segment 0 (nullable): row m of A is row a_idx[m] of a matrix with a_rows rows (the
    // gather of the upstream gradient's kept rows, folded into the A-tile loads).
    const int32_t* a_idx;
    int64_t a_rows;
    NtParts parts;  // mode NT: the contraction cut into parts where the output has few tiles
};

// Mode TN: up to TN_MAX products C_j [M_j,N_j] = A_j^T * B_j over the same K rows (A, B, C, M and N above are unused).  Their
// tiles form one list, product by product; all the parameter gradients of a layer are one launch, whose tiles fill whole
// rounds of the CUs but for one remainder, where a launch per product has a remainder each: [8192 rows, H = 2048,
// F = 5632, 32/4 heads of 64] 176 + 352 + 64 + 80 tiles are 2.6 rounds instead of 1 + 2 + 1 + 1, into fp32 buffers 822 us in
// four launches and 750 in one; [841 rows, H = 4096, F = 1792, 4/1 heads of 128] 81 us in four, 60 in one.
struct TnArgs : GemmArgs {
    GemmTnProb p[TN_MAX];
    int end[TN_MAX];    // tiles of products 0..j
    int n_blocks;       // blocks that walk through the tiles; those behind them sum the gain gradients up
    GainGrads gain;
};

// How the tiles of the last, partial round are cut.  The cost of a round of sub-tiles
// relative to a round of 256x256 tiles is more than its share of the flops (smaller
// tiles move more operand bytes per flop); the figures are measured on MI355X at K = 4096.
// Returns the launch's length in rounds of 256x256 tiles.
// A round of 256x192 tiles costs 0.94 of a round of 256x256 tiles although it has 0.75 of the
// flops: the chip is power-limited under these kernels, so the 192 CUs that a 16 x 12 tile output
// occupies clock higher than all 256 do (measured: 412 GFLOP in 354 us on 192 CUs, 333 us on 256).
static constexpr double kCost192 = 0.94;
__host__ __device__ inline int cdiv(int a, int b) { return (a + b - 1) / b; }
__host__ __device__ inline double plan_tiles(int tiles, int n_cu, int& n_full, int& sub) {
    n_full = tiles / n_cu * n_cu;
    const int rem = tiles - n_full;
    sub = 1;
    if (rem == 0) return n_full / n_cu;
    double best = 1e30;
    for (int c = 0; c < 3; ++c) {
        const double cost = c == 0 ? 1.0 : (c == 1 ? 0.6 : 0.4);
        const int cut = 1 << c;
        const double t = (double)cdiv(rem * cut, n_cu) * cost;
        if (t < best - 1e-9) {
            best = t;
            sub = cut;
        }
    }
    return n_full / n_cu + best;
}

// Tile plan of an NT launch with n_cu blocks: sets n_full, sub, tile_n; returns the number of work
// items.  The host plans a launch whose sizes it knows; with a device-side count every block runs
// the same code on the count it read, so both give the same tiles for the same sizes.
__host__ __device__ inline int plan_launch(int M, int N, int n_cu, int& n_full, int& sub, int& tile_n) {
    const int tiles = cdiv(M, 256) * cdiv(N, 256);
    const double rounds = plan_tiles(tiles, n_cu, n_full, sub);
    int items = n_full + (tiles - n_full) * sub;
    tile_n = 256;
    // 256x192 tiles instead, when they fill the CUs better (an output of 16 x 12 tiles of
    // 256x256 leaves a quarter of the CUs idle; as 16 x 16 tiles of 256x192 it is one full round)
    const int tiles192 = cdiv(M, 256) * cdiv(N, 192);
    if (cdiv(tiles192, n_cu) * kCost192 < rounds - 1e-9) {
        tile_n = 192;
        items = tiles192;
    }
    return items;
}

typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4_t;
typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8_t;
typedef __attribute__((address_space(3))) s16x4_t* lds_s16x4_ptr;

static constexpr int GEMM_RING = 128 * 1024;        // the operand stages; their number and size depend on the tile (gemm_tiles)
static constexpr int GEMM_SMEM = 160 * 1024;    // the whole LDS of a CU: the ring and the bf16 write-out's staging above it

// Position l of a block in the logical order of its group of n blocks: XCD x (block id
// mod 8) takes the x-th contiguous share of the order.
__device__ __forceinline__ int xcd_order(int pid, int n) {
    const int xcd = pid & 7, local = pid >> 3;
    const int base = n >> 3, rem = n & 7;
    return xcd * base + (xcd < rem ? xcd : rem) + local;
}

// Logical tile l -> tile coordinates: bands of GROUP_M tile rows walked column by column.
__device__ __forceinline__ void tile_coords(int l, int tiles_m, int tiles_n, int& bm, int& bn) {
    constexpr int GROUP_M = 8;
    const int band = l / (GROUP_M * tiles_n);
    const int first_m = band * GROUP_M;
    const int gsize = min(GROUP_M, tiles_m - first_m);
    const int r = l - band * GROUP_M * tiles_n;
    bm = first_m + r % gsize;
    bn = r / gsize;
}

template <typename P>
__device__ __forceinline__ P* uniform_ptr(P* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<P*>(((uint64_t)hi << 32) | lo);
}

// Swizzle of a K-contiguous operand's rows in LDS (128 bytes, 64 k): the 16-byte chunk index of row r is XOR-ed with
// (r / 2) % 8.  The LDS serves a ds_read_b128 in four passes of 16 lanes, and the passes are not runs of consecutive lanes:
// {0-3, 12-15, 20-27}, {4-11, 16-19, 28-31} and the same plus 32 (measured).  A fragment read has lane l at row l % 16,
// chunk l / 16 of a K-step, so a pass mixes chunk c of rows 0-3 and 12-15 with chunk c + 1 of rows 4-11 (or the other way
// round); with this function its 16 lanes fall into 16 different 16-byte bank groups.
__device__ __forceinline__ int nt_swz(int row) { return (row >> 1) & 7; }

// Of D loads spread over the N MFMAs of a sub-step (D <= N), the one that goes with MFMA q, or -1.
constexpr int load_in_gap(int q, int D, int N) {
    for (int d = 0; d < D; ++d)
        if ((d * N) / D == q) return d;
    return -1;
}

// One output tile: its origin, and the operands (of segment 0), output matrix and its sizes that it belongs to.
struct TileRef {
    int m0, n0, M, N;
    const void *A0, *B0;
    void* C;
};

// The block's output tiles of (64*TM) x (64*TN), one after the other: `first`, then whatever
// next_tile(TileRef&) hands out until it returns false.  The loads of the next
// tile's first K-steps are in flight while the finished tile leaves through a staging area of its
// own, and its stores drain under the next tile's MFMAs.  SPLIT: the block contracts only the pairs of K-steps
// [pbeg, pend) of the segments' sequence and stores its fp32 accumulators, unscaled, to `part_out`
// ([BM, BN] fp32, the rows below M); whoever needs the product adds the parts up.
// K0x: the live value of g.K[0] (it differs from the launch argument when the kept-token count is read on the device).
template <int MODE, int TM, int TN, bool SPLIT, bool CF32, typename Next>
__device__ __forceinline__ void gemm_tiles(const GemmArgs& g, const int K0x, const TileRef first,
                                           Next next_tile, unsigned char* smem,
                                           const int pbeg = 0, const int pend = 0, float* part_out = nullptr) {
    // Ring of operand stages: four of 32 KB, i.e. two pairs of K-steps, or for the 128x128 tile eight of 16 KB = four
    // pairs.  A pair of the small tile is 32 MFMAs (0.22 us) per wave, and with one pair of lookahead a block waited
    // out most of a load's latency per pair; three pairs of lookahead cover it.
    constexpr bool DEEP = TM == 2 && TN == 2;
    constexpr int BM = 64 * TM, BN = 64 * TN, KB = 32, STAGE = DEEP ? 16384 : 32768;
    constexpr int NSTG = GEMM_RING / STAGE, NPR = NSTG / 2;     // stages and pairs in the ring
    constexpr int PAIR = 2 * STAGE, PWIN = 65536 / PAIR;    // bytes of a pair, pairs within reach of one LDS base register
    // MODE 0 (NT): both operands lie with K contiguous in memory; 1 (TN): both K-major; 2 (NN): A K-contiguous, B K-major
    constexpr bool AK = MODE != 1, BK = MODE == 0;
    constexpr int A_BYTES = BM * KB * 2, B_BYTES = BN * KB * 2;     // of one K-step; a pair holds A's two K-steps, then B's
    constexpr int NU = TM + TN;                         // 1 KB wave-loads per wave per K-step: TM for A, TN for B
    constexpr int FM = 2 * TM, FN = 2 * TN;             // 16-row fragments of the wave tile along M and N
    constexpr int NQ = 2 * FN;                          // MFMAs per sub-step: one 32-row block of A x all of B
    // groups that the wave-loads of a pair are issued in (measured: 2 groups cost 4 %; NT is best
    // with 4 to 6, TN with 3)
    constexpr int NG = TM == 2 ? 2 : (MODE == 0 ? 4 : 3);
    static_assert(A_BYTES + B_BYTES <= STAGE, "tile shape");

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int l16 = lane & 15, g4 = lane >> 4;

    f32x4_t acc[FM][FN];
    TileRef ld = first;             // the tile whose operands are being loaded

    // ---- global -> LDS -----------------------------------------------------------
    // (seg, k0): the K-step that the next loads fetch.  Past the last segment Kseg = 0, so
    // every load is out of range (zero fill into a stage whose contents are never used):
    // the number of loads per K-step never changes, which keeps the vmcnt bookkeeping constant.
    int seg = 0, k0 = 0, Kseg = 0;
    i32x4_t rsA, rsB;
    unsigned ldA = 0, ldB = 0;
    // Per-lane byte offsets of the pair's wave-loads at k = 0 of the current segment (out of range for rows / columns beyond the
    // matrix edge); the K position of a pair is added as the load's scalar offset, so the steady-state loop spends no vector
    // instruction on addresses.
    constexpr unsigned OOB_FAST = 0x80000000u;          // stays out of range when the scalar offset is added
    unsigned vo[NU][2];
    auto open_segment = [&](int s) __attribute__((always_inline)) {
        const bool live = (unsigned)s < (unsigned)g.nseg;
        const int m0 = ld.m0, n0 = ld.n0, Mx = ld.M;
        const int sa = live ? s : 0;
        const bf16_t* A = static_cast<const bf16_t*>(ld.A0);
        const bf16_t* B = static_cast<const bf16_t*>(ld.B0);
        int Kraw = K0x;
        if (sa != 0) {      // a branch: the first segment's operands, which open every tile, do not wait for a load
            A = static_cast<const bf16_t*>(g.A[sa]);
            B = static_cast<const bf16_t*>(g.B[sa]);
            Kraw = g.K[sa];
        }
        Kseg = live ? Kraw : 0;
        const int64_t K = Kraw;
        const bool gatherA = MODE == 0 && s == 0 && g.a_idx != nullptr;
        if (AK) {
            // gathered A: the descriptor spans the whole source matrix and a lane's offset starts at its source row
            rsA = gatherA ? make_rsrc(A, g.a_rows * K * 2) : make_rsrc(A + (int64_t)m0 * K, ((int64_t)Mx - m0) * K * 2);
            ldA = (unsigned)K * 2u;
        } else {
            rsA = make_rsrc(A + m0, (K * Mx - m0) * 2);
            ldA = (unsigned)Mx * 2u;
        }
        if (BK) {
            rsB = make_rsrc(B + (int64_t)n0 * K, ((int64_t)ld.N - n0) * K * 2);
            ldB = (unsigned)K * 2u;
        } else {
            rsB = make_rsrc(B + n0, (K * ld.N - n0) * 2);
            ldB = (unsigned)ld.N * 2u;
        }
        // The per-lane parts below never change, but they are cheap to rebuild and registers are
        // scarce while a finished tile is still in the accumulators: keep the compiler from carrying
        // them across the main loop (and spilling them) by hiding where the lane number comes from.
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const unsigned lc_nt = (unsigned)((ln & 7) ^ nt_swz(wave * 8 + (ln >> 3)));
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const bool isA = u < TM;
            const int i = isA ? u : u - TM;
            if (isA ? AK : BK) {
#pragma unroll
                for (int sec = 0; sec < 2; ++sec) {
                    const unsigned row = (4 * (2 * i + sec) + wave) * 8 + (ln >> 3);
                    vo[u][sec] = row * (isA ? ldA : ldB) + lc_nt * 16u;
                    if (isA && gatherA) {   // rows past M carry an out-of-range offset; the index is read for live rows only
                        const int m = m0 + (int)row;
                        vo[u][sec] = m < Mx ? (unsigned)g.a_idx[m] * ldA + lc_nt * 16u : OOB_FAST;
                    }
                }
            } else {
                const int cpr = (isA ? BM : BN) / 8;
                const int qq = (4 * i + wave) * 64 + ln;
                const int kr = qq / cpr;
                const int c = (qq % cpr) ^ ((kr & 3) << 2);
                const bool ok = (isA ? m0 : n0) + c * 8 < (isA ? Mx : ld.N);
                vo[u][0] = vo[u][1] = ok ? (unsigned)kr * (isA ? ldA : ldB) + c * 16u : OOB_FAST;
            }
        }
    };
    // scalar K offsets of the pair at (seg, k0); in the last pair of a segment (and past the last segment, where Kseg = 0) the lanes
    // whose k falls past its end go out of range
    unsigned ka0 = 0, kb0 = 0, ka1 = 0, kb1 = 0;
    auto prepare_pair = [&]() __attribute__((always_inline)) {
        if (k0 + 2 * KB > Kseg) {
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                const bool isA = u < TM;
                const int i = isA ? u : u - TM;
#pragma unroll
                for (int sec = 0; sec < 2; ++sec) {         // first k of the lane's chunk within the pair
                    const int kpos = (isA ? AK : BK) ? (int)((lane & 7) ^ nt_swz(wave * 8 + (lane >> 3))) * 8
                                                     : sec * KB + ((4 * i + wave) * 64 + lane) / ((isA ? BM : BN) / 8);
                    if (k0 + kpos >= Kseg) vo[u][sec] = OOB_FAST;
                }
            }
        }
        if (AK) ka0 = (unsigned)k0 * 2u;
        else { ka0 = (unsigned)k0 * ldA; ka1 = (unsigned)(k0 + KB) * ldA; }
        if (BK) kb0 = (unsigned)k0 * 2u;
        else { kb0 = (unsigned)k0 * ldB; kb1 = (unsigned)(k0 + KB) * ldB; }
    };
    // A pair of K-steps never straddles a segment boundary: the part of a segment's last pair past Kseg is zeros.
    int left = SPLIT ? pend - pbeg : 0;         // pairs of the part whose loads are not all out yet
    auto advance_pair = [&]() __attribute__((always_inline)) {
        if (SPLIT && --left <= 0) {             // nothing of the part is left: the loads behind it are out of range
            Kseg = 0;
            return;
        }
        k0 += 2 * KB;
        if (k0 >= Kseg) {
            k0 = 0;
            ++seg;
            if (!DEEP || (unsigned)seg < (unsigned)g.nseg) open_segment(seg);
            else Kseg = 0;      // past the last segment: only the range of k matters any more
        }
    };

    const unsigned lds0 = __builtin_amdgcn_readfirstlane(lds_addr_of(smem) + wave * 1024);
    // Wave-load (U, SEC) of the pair at (seg, k0) into pair P of the ring: U < TM -> A tile, else B tile.  K-contiguous: 8 rows of
    // 64 k, whole 128-byte lines, and the chunk a lane fetches undoes the XOR swizzle of its LDS slot.  (Loads of 16 rows x 32 k,
    // with the other half of the lines in the next instruction, cost a third more of the time that a CU needs to take in its
    // operands: 0.46 us per pair of a 128x128 tile without MFMAs against 0.35; [4096, 4096], K = 14336, 328 us and 319,
    // [300, 4096], K = 14336, 90 and 82, [841, 1792], K = 4096, 30.8 and 29.0.)  K-major: 1024 / (2*rows) k-rows of K-step SEC.
    auto load_dst = [](int p, int u, int sec) constexpr {
        const bool isA = u < TM;
        const int i = isA ? u : u - TM, op0 = p * PAIR + (isA ? 0 : 2 * A_BYTES);
        return op0 + ((isA ? AK : BK) ? (2 * i + sec) * 4096 : sec * (isA ? A_BYTES : B_BYTES) + i * 4096);
    };
    auto dma_one = [&](auto P, auto U, auto SEC) __attribute__((always_inline)) {
        constexpr int p = decltype(P)::value, u = decltype(U)::value, sec = decltype(SEC)::value;
        constexpr bool isA = u < TM, kc = isA ? AK : BK;
        dma16i<load_dst(p, u, sec), 0>(lds0, isA ? rsA : rsB, vo[u][sec],
                                       isA ? (!kc && sec ? ka1 : ka0) : (!kc && sec ? kb1 : kb0));
    };
    // the same load wrapped around the MFMA acc += a x b (inside the MFMA stream)
    auto mma_dma_one = [&](f32x4_t& c, const bf16x8_t a, const bf16x8_t b, auto P, auto U, auto SEC) __attribute__((always_inline)) {
        constexpr int p = decltype(P)::value, u = decltype(U)::value, sec = decltype(SEC)::value;
        constexpr bool isA = u < TM, kc = isA ? AK : BK;
        mfma16_dma16i<load_dst(p, u, sec), 0>(c, a, b, lds0, isA ? rsA : rsB, vo[u][sec],
                                              isA ? (!kc && sec ? ka1 : ka0) : (!kc && sec ? kb1 : kb0));
    };

    // ---- LDS -> fragments.  A fragment is 16 rows x 32 k (one K-step): lane l holds row l%16,
    // k = 8*(l/16) .. +7.  An LDS address is a per-lane base register that never changes plus a
    // compile-time constant (stage, fragment) in the instruction's 16-bit offset field; the upper half of
    // the ring lies past that field's reach from the base of stage 0 and has base registers of its own.
    typedef __attribute__((address_space(3))) unsigned char* lds_u8_ptr;
    typedef const __attribute__((address_space(3))) u32x4_t* lds_u32x4_cptr;
    // base registers: one per K-step for a K-contiguous operand (the swizzle mixes the K-step's chunk bit in), one per 32-row block
    // for a K-major one (it mixes the block in)
    constexpr int NBA = AK ? 2 : TM, NBASE = NBA + (BK ? 2 : TN);
    unsigned fbase[NBASE][2];
    {
        const unsigned s0 = lds_addr_of(smem);
#pragma unroll
        for (int u = 0; u < NBASE; ++u) {
            const bool isA = u < NBA;
            const int i = isA ? u : u - NBA;
            const unsigned op0 = s0 + (isA ? 0 : 2 * A_BYTES);
            unsigned v;
            if (isA ? AK : BK) {
                const int wrow = isA ? wm * (32 * TM) : wn * (32 * TN);
                v = op0 + (wrow + l16) * 128 + (((4 * i + g4) ^ nt_swz(l16)) << 4);
            } else {
                const int W2 = (isA ? BM : BN) * 2;                 // bytes per k-row
                const int row0 = isA ? wm * (32 * TM) + i * 32 : wn * (32 * TN) + i * 32;
                const int kl = 8 * g4 + (l16 >> 2);                 // k within the K-step (and kl + 4)
                const int lc = row0 / 8 + ((lane & 3) >> 1);
                const int sw = (kl & 3) << 2;                       // the same for k and k + 4
                v = op0 + kl * W2 + ((lc ^ sw) << 4) + (lane & 1) * 8;
            }
            fbase[u][0] = v;
            fbase[u][1] = v + 65536;
        }
    }
    bf16x8_t fa[2][2], fb[2][FN];
    // fragment F (16 rows; F < FM: of the wave's A rows, else of its B rows) of K-step KS of pair P of the ring
    // into fa[BUF][F % 2] or fb[BUF][F - FM]
    auto frag_one = [&](auto P, auto KS, auto F, auto BUF) __attribute__((always_inline)) {
        constexpr int p = decltype(P)::value, ks = decltype(KS)::value, fr = decltype(F)::value, buf = decltype(BUF)::value;
        constexpr bool isA = fr < FM;
        constexpr int f = isA ? fr : fr - FM;
        constexpr int win = p / PWIN, poff = (p % PWIN) * PAIR;
        bf16x8_t v;
        if constexpr (isA ? AK : BK) {
            const lds_u8_ptr q = reinterpret_cast<lds_u8_ptr>(fbase[(isA ? 0 : NBA) + ks][win]);
            v = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<lds_u32x4_cptr>(q + (poff + f * 2048)));
        } else {
            constexpr int W2 = (isA ? BM : BN) * 2, off = poff + ks * (isA ? A_BYTES : B_BYTES) + (f & 1) * 32;
            const lds_u8_ptr q = reinterpret_cast<lds_u8_ptr>(fbase[(isA ? 0 : NBA) + f / 2][win]);
            const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(q + off));
            const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(q + (off + 4 * W2)));
            v = __builtin_bit_cast(bf16x8_t, (s16x8_t)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        }
        if constexpr (isA) fa[buf][f & 1] = v;
        else fb[buf][f] = v;
    };
    // Sub-step T of pair P of the ring (T = KS*TM + A): the MFMAs of K-step KS for the 32-row
    // block A of the wave's rows against all its columns.  D = Bfrag x Afrag: lane l holds row l%16 of
    // the fragment and 4 adjacent output columns.  Spread between the MFMAs:
    //   * the two A fragments of the next sub-step (the next block of the same K-step, or block 0 of
    //     the next K-step);
    //   * the B fragments of the next K-step: during K-step 0 of the pair a share of those of K-step 1
    //     per sub-step; K-step 0 of the next pair is published by the barrier ahead of the pair's last
    //     sub-step, which therefore reads all of them;
    //   * a share of the wave-loads: the pair at (seg, k0) is loaded in NG groups, group 0 in the last
    //     sub-step of a pair (into the pair of stages its barrier has just retired), groups 1.. in the first
    //     sub-steps of the next pair.
    constexpr bool BACK = !DEEP;        // the order of a sub-step's MFMAs, see there
    auto substep = [&](auto P, auto T) __attribute__((always_inline)) {
        constexpr int p = decltype(P)::value, t = decltype(T)::value;
        constexpr int ks = t / TM, a = t % TM;
        constexpr int nxt = ks == 0 ? p : (p + 1) % NPR;            // pair of the next K-step
        constexpr bool last = t == 2 * TM - 1;
        constexpr int a_pair = a + 1 < TM ? p : nxt, a_ks = a + 1 < TM ? ks : ks ^ 1, a_blk = a + 1 < TM ? a + 1 : 0;
        // reads of this sub-step, in the order their first users come: A fragments, B fragments (BACK) or A fragment 0, B
        // fragments, A fragment 1
        constexpr int NB = ks == 0 ? 0 : (last ? FN : 0);           // all B fragments at once
        constexpr int b_lo = ks == 0 ? (a * FN) / TM : 0, b_hi = ks == 0 ? ((a + 1) * FN) / TM : NB;
        constexpr int NR = 2 + (b_hi - b_lo);
        // wave-loads of this sub-step: group 0 (last sub-step) or group t + 1 (t < TM - 1)
        constexpr int grp = last ? 0 : (t < NG - 1 ? t + 1 : -1);
        constexpr int e_lo = grp < 0 ? 0 : ((grp * NU) / NG) * 2, e_hi = grp < 0 ? 0 : (((grp + 1) * NU) / NG) * 2;
        constexpr int dp = last ? p : (p + NPR - 1) % NPR;          // where they go: this pair, or the one before
        static_for<NQ>([&](auto Q) __attribute__((always_inline)) {
            constexpr int q = decltype(Q)::value;
            static_for<NR>([&](auto R) __attribute__((always_inline)) {
                constexpr int r = decltype(R)::value;
                if constexpr ((r * NQ) / NR == q) {
                    constexpr int f = BACK ? (r < 2 ? r : -1) : (r == 0 ? 0 : (r == NR - 1 ? 1 : -1));
                    if constexpr (f >= 0) frag_one(ic<a_pair>{}, ic<a_ks>{}, ic<2 * a_blk + f>{}, ic<((a + 1) & 1)>{});
                    else frag_one(ic<nxt>{}, ic<(ks ^ 1)>{}, ic<FM + b_lo + r - (BACK ? 2 : 1)>{}, ic<(ks ^ 1)>{});
                }
            });
            CF_SCHED_FENCE();
            {
                // Inline assembly pins the accumulators to the AGPR file: with the builtin the register
                // allocator keeps part of the 64 four-register accumulators of a 128x128 wave tile in
                // VGPRs and copies them to and fro around every MFMA.  An accumulator is touched once
                // per K-step, so two MFMAs on the same registers are never back to back.
                // Both A fragments per B fragment, back and forth: an MFMA shares an operand with the one before it and the other
                // with the one after, which costs less power than eight B fragments in a row for one A fragment (a register-resident
                // loop 2060 and 2107 TFLOP/s; X^T*dY and dY*W^T of [4096, 4096 -> 14336] 694 and 688 us, the layer step with
                // these sizes 3265 and 3230).  The small tile, which waits for its operands, runs the other way: there A fragment 1 has
                // half a sub-step longer to arrive ([841, 4096], K = 3584 out of HBM: 40 us back and forth, 36).
                constexpr int j = BACK ? q >> 1 : q % FN, h = BACK ? (q & 1) ^ (j & 1) : q / FN, i = 2 * a + h;
                constexpr int dsel = load_in_gap(q, e_hi - e_lo, NQ);       // the wave-load that goes with this MFMA
                if constexpr (dsel >= 0) {
                    constexpr int e = dsel + e_lo;
                    mma_dma_one(acc[i][j], fb[ks][j], fa[a & 1][h], ic<dp>{}, ic<(e >> 1)>{}, ic<(e & 1)>{});
                } else {
                    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[i][j]) : "v"(fb[ks][j]), "v"(fa[a & 1][h]));
                }
            }
            CF_SCHED_FENCE();
        });
    };
    // loads of the pair at (seg, k0) outside the MFMA stream (prologue): all of them, or group 0 only
    auto issue_pair = [&](auto P, auto FIRST_GROUP) __attribute__((always_inline)) {
        prepare_pair();
        static_for<(decltype(FIRST_GROUP)::value ? (NU / NG) * 2 : 2 * NU)>([&](auto E) __attribute__((always_inline)) {
            constexpr int e = decltype(E)::value;
            dma_one(P, ic<(e >> 1)>{}, ic<(e & 1)>{});
        });
    };
    // One pair of K-steps in pair P of the ring; the next NPR - 1 pairs lie in the
    // others, and the loads of the pair after those go back into P once the barrier
    // has retired it.  The loop body is NPR pairs, so every LDS place is a compile-time constant.
    // The loads of a pair are issued in NG groups, the first right after the barrier that frees their
    // place, which keeps the burst that the load path sees short; the last group still has more
    // than half a pair to land before the next barrier.
    auto pair_body = [&](auto P) __attribute__((always_inline)) {
        static_for<2 * TM>([&](auto T) __attribute__((always_inline)) {
            constexpr int t = decltype(T)::value;
            if constexpr (t == 2 * TM - 1) {
                prepare_pair();
                wait_vmcnt<(NPR - 2) * 2 * NU>();       // the next pair has landed; later pairs (loads only) may be in flight
                lds_barrier();          // ... and every wave is done with pair P
            }
            substep(P, T);
            if constexpr (t == NG - 2) advance_pair();      // the last group of the pair has been issued
        });
    };

    // pairs of K-steps; the last one of a segment may be a part of one
    int npairs = SPLIT ? pend - pbeg : (K0x + 2 * KB - 1) / (2 * KB);
    if (!SPLIT)
        for (int s = 1; s < g.nseg; ++s) npairs += (g.K[s] + 2 * KB - 1) / (2 * KB);
    // prologue of tile ld: the first NPR - 1 pairs and the first group of the loads of the pair behind them
    auto start_tile = [&]() __attribute__((always_inline)) {
        seg = 0;
        k0 = 0;
        if (SPLIT) {                    // the part's first pair
            int p = pbeg;
            for (int n = (K0x + 2 * KB - 1) / (2 * KB); seg + 1 < g.nseg && p >= n; n = (g.K[seg] + 2 * KB - 1) / (2 * KB)) {
                p -= n;
                ++seg;
            }
            k0 = p * 2 * KB;
        }
        open_segment(seg);
        static_for<NPR - 1>([&](auto P) __attribute__((always_inline)) {
            constexpr int p = decltype(P)::value;
            issue_pair(ic<p>{}, ic<0>{});
            advance_pair();
        });
        issue_pair(ic<NPR - 1>{}, ic<1>{});        // the loop's first sub-steps issue the other groups
    };
    constexpr bool OVERLAP = !SPLIT;        // the epilogue leaves the operand stages alone
    if (npairs > 0) start_tile();
    for (bool first_tile = true;; first_tile = false) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.f;
        if (npairs > 0) {
            // K-steps 0 and 1 have landed.  The counter covers loads and stores, which retire out of order with respect
            // to each other, but a bound on what is outstanding is one on the outstanding loads, and those retire in order:
            // a partial count is safe with a previous call's stores in flight too.  Between two tiles of a call
            // everything is waited for: the tile's stores, issued behind these loads, are in flight then and a partial
            // count would be met little earlier.
            if (DEEP && first_tile) wait_vmcnt<(NPR - 2) * 2 * NU + (NU / NG) * 2>();
            else wait_vmcnt<0>();
            lds_barrier();
            frag_one(ic<0>{}, ic<0>{}, ic<0>{}, ic<0>{});
            static_for<FN>([&](auto J) __attribute__((always_inline)) { frag_one(ic<0>{}, ic<0>{}, ic<FM + decltype(J)::value>{}, ic<0>{}); });
            frag_one(ic<0>{}, ic<0>{}, ic<1>{}, ic<0>{});
            // NPR pairs per iteration.  The small tile, where short contractions are the rule, leaves after the last
            // pair; the others run an odd count's extra pair on zeros (loads past the last segment return them)
            if constexpr (DEEP) {
                for (int p = npairs;;) {
                    pair_body(ic<0>{});
                    if (--p <= 0) break;
                    pair_body(ic<1>{});
                    if (--p <= 0) break;
                    pair_body(ic<2>{});
                    if (--p <= 0) break;
                    pair_body(ic<3>{});
                    if (--p <= 0) break;
                }
            } else {
                for (int p = 0; p < npairs; p += 2) {
                    pair_body(ic<0>{});
                    pair_body(ic<1>{});
                }
            }
            wait_vmcnt<0>();
            // The MFMAs are inline assembly (see substep), so the compiler does not know that their
            // results are still on the way when the next vector instruction wants to read them: the
            // wait states between a 4-pass MFMA and a reader of its destination are spent here.
            asm volatile("s_nop 15\n\ts_nop 15");
        }
        const TileRef ep = ld;          // the tile that leaves
        const bool has_next = next_tile(ld);
        if (OVERLAP) {
            lds_barrier();              // every wave has read its last fragments: the stages are free
            if (has_next && npairs > 0) start_tile();
        }
        const int m0 = ep.m0, n0 = ep.n0, Mx = ep.M;

    if (SPLIT) {
        // ---- split-K epilogue: the tile's fp32 accumulators, unscaled, straight to the item's own slot (columns past the
        // matrix are zeros in it, rows past it are not written)
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const int r = wm * (32 * TM) + i * 16 + l16;
            if (m0 + r < Mx) {
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    float4 o;
                    o.x = acc[i][j][0]; o.y = acc[i][j][1]; o.z = acc[i][j][2]; o.w = acc[i][j][3];
                    *reinterpret_cast<float4*>(part_out + r * BN + wn * (32 * TN) + j * 16 + 4 * g4) = o;
                }
            }
        }
        break;
    }
    const float alpha = g.alpha;
    if constexpr (CF32) {
        // ---- fp32 epilogue: C += the tile, straight from the accumulators: a lane's 4 adjacent columns are 16 bytes of a row, and
        // the four lanes of a row cover half a line, whose other half is the next column fragment.  The old values of the
        // next 16 rows are on their way while these are added.  No LDS, so the next tile's operands are loaded meanwhile, as in
        // the bf16 epilogue.  (Through LDS in two halves of the tile, to whole rows, with nothing else in flight:
        // [5632, 2048] += , K = 8192, 238 us, now 223.)
        // Descriptor over this wave's rows: an offset stays below 2^31 for every N that the launcher accepts.
        const int mw = m0 + wm * (32 * TM), rows = min(Mx - mw, 32 * TM);
        const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(
            static_cast<float*>(ep.C) + (int64_t)mw * ep.N, 0, rows > 0 ? (int)((unsigned)rows * (unsigned)ep.N * 4u) : 0, 0x00020000);
        int ln = lane;                                      // as in open_segment: rebuilt per tile, not carried
        asm volatile("" : "+v"(ln));
        const unsigned row_bytes = (unsigned)ep.N * 4u;
        const int n = n0 + wn * (32 * TN) + 4 * (ln >> 4);
        const unsigned voff = (unsigned)(ln & 15) * row_bytes + (unsigned)n * 4u;
        u32x4_t old[2][FN];
        auto fetch = [&](int i) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < FN; ++j)                    // N is a multiple of 8
                old[i & 1][j] = __builtin_amdgcn_raw_buffer_load_b128(
                    rc, n + j * 16 < ep.N ? voff + (unsigned)(i * 16) * row_bytes + j * 64u : OOB_FAST, 0, 0);
        };
        fetch(0);
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            if (i + 1 < FM) fetch(i + 1);
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                u32x4_t o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = __float_as_uint(acc[i][j][e] * alpha + __uint_as_float(old[i & 1][j][e]));
                __builtin_amdgcn_raw_buffer_store_b128(
                    o, rc, n + j * 16 < ep.N ? voff + (unsigned)(i * 16) * row_bytes + j * 64u : OOB_FAST, 0, 0);
            }
        }
        if (!has_next) break;
        continue;
    }
    // ---- epilogue: 32 rows of the wave tile at a time: acc -> bf16 -> the wave's own 8 KB above the
    // four stages -> global with 16-byte stores, whole rows per group of lanes.  The 16-byte chunks
    // of a staged row are XOR-ed with the row number, which keeps both the column-wise writes (a
    // lane holds 4 adjacent columns of one row) and the row-wise reads spread over the banks.  No
    // block barrier: the area is private to the wave and its LDS operations execute in order.
    // The stores go through a buffer descriptor over the whole output matrix, so there is no
    // branch in the stream: rows past M fall outside its range and lanes whose columns lie past
    // N carry an out-of-range offset.
    {
        // bytes of a staged row: 32*TN columns, padded to a power of two of 16-byte chunks (TN = 3:
        // the lanes of the four pad chunks store nothing)
        constexpr int RBY = 64 * (TN == 3 ? 4 : TN);
        constexpr int CPR = RBY / 16, RPP = 64 / CPR;       // 16-byte chunks per row, rows per pass of the wave
        constexpr int NP = 32 / RPP, NV = CPR / RPP;        // passes per 32 rows; distinct swizzle phases
        unsigned char* stg = smem + GEMM_RING + wave * 8192;
        const __amdgpu_buffer_rsrc_t rc =
            __builtin_amdgcn_make_buffer_rsrc(ep.C, 0, (int)((int64_t)Mx * ep.N * 2), 0x00020000);
        const float beta = g.beta;
        int ln = lane;                                      // as in open_segment: rebuilt per tile, not carried
        asm volatile("" : "+v"(ln));
        const int c = ln % CPR, rl = ln / CPR;
        const int l16 = ln & 15, g4 = ln >> 4;
        const int n = n0 + wn * (32 * TN) + c * 8;
        const unsigned row_bytes = (unsigned)ep.N * 2u;
        // N is a multiple of 8, so a 16-byte chunk lies inside a row or outside it
        const unsigned voff = (n < ep.N && c < 4 * TN)
                                  ? (unsigned)(m0 + wm * (32 * TM) + rl) * row_bytes + (unsigned)n * 2u : OOB_FAST;
        const unsigned char* rd[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) rd[v] = stg + rl * RBY + ((c ^ ((rl + RPP * v) & (CPR - 1))) << 4);
        // a lane's 4 columns of fragment column j are half of the 16-byte chunk 2*j + g4/2 of its row
        unsigned char* const wr = stg + l16 * RBY + (g4 & 1) * 8;
        const int wsw = l16 & (CPR - 1);                    // staged row 16*h + l16, and CPR divides 16
        const int wch = g4 >> 1;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    uint2 o;
                    o.x = pack_bf16x2(acc[2 * i + h][j][0] * alpha, acc[2 * i + h][j][1] * alpha);
                    o.y = pack_bf16x2(acc[2 * i + h][j][2] * alpha, acc[2 * i + h][j][3] * alpha);
                    *reinterpret_cast<uint2*>(wr + h * 16 * RBY + (((2 * j + wch) ^ wsw) << 4)) = o;
                }
            u32x4_t val[NP];
#pragma unroll
            for (int q = 0; q < NP; ++q)
                val[q] = *reinterpret_cast<const u32x4_t*>(rd[q % NV] + q * RPP * RBY);
            if (MODE == 1 && beta != 0.f) {
#pragma unroll
                for (int q = 0; q < NP; ++q) {
                    const u32x4_t old = __builtin_amdgcn_raw_buffer_load_b128(
                        rc, voff + (unsigned)(i * 32 + q * RPP) * row_bytes, 0, 0);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float lo = __uint_as_float(val[q][e] << 16) + beta * __uint_as_float(old[e] << 16);
                        const float hi = __uint_as_float(val[q][e] & 0xFFFF0000u) +
                                         beta * __uint_as_float(old[e] & 0xFFFF0000u);
                        val[q][e] = pack_bf16x2(lo, hi);
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < NP; ++q)
                __builtin_amdgcn_raw_buffer_store_b128(val[q], rc, voff + (unsigned)(i * 32 + q * RPP) * row_bytes, 0, 0);
        }
    }
    if (!has_next) break;
    }   // tile loop
}

// The work items of a launch: the n_full whole tiles first, then the sub-tiles of the remaining
// tiles.  Block b takes items b, b + stride, ...: with as many blocks as CUs every block runs
// its share of the whole tiles back to back and then at most a few sub-tiles, and the items of
// one block stay on one XCD (item id mod 8 = block id mod 8).
// locate(l, t, bm, bn): logical tile l of the launch -> the product it belongs to (t without its origin) and its tile coordinates.
template <int MODE, bool CF32, typename Locate>
__device__ __forceinline__ void gemm_items(const GemmArgs& g, const int K0x, const int tiles, const int n_full, const int sub,
                                           const int stride, Locate locate, unsigned char* smem) {
    const int n_items = n_full + (tiles - n_full) * sub;
    // item -> tile; false when a sub-tile lies outside the matrix
    auto decode = [&](int w, TileRef& t) __attribute__((always_inline)) {
        int bm, bn, m0, n0;
        if (w < n_full) {
            locate(xcd_order(w, n_full), t, bm, bn);
            m0 = bm * 256;
            n0 = bn * 256;
        } else {
            const int cut = sub;
            const int j = xcd_order(w - n_full, n_items - n_full);
            const int part = j % cut;
            locate(n_full + j / cut, t, bm, bn);
            m0 = bm * 256 + (cut == 4 ? (part >> 1) * 128 : 0);
            n0 = bn * 256 + (cut == 4 ? (part & 1) * 128 : (cut == 2 ? part * 128 : 0));
            if (m0 >= t.M || n0 >= t.N) return false;
        }
        // every field is the same in all lanes: say so, which keeps the address arithmetic of the
        // tile's prologue on the scalar unit
        t.m0 = __builtin_amdgcn_readfirstlane(m0);
        t.n0 = __builtin_amdgcn_readfirstlane(n0);
        t.M = __builtin_amdgcn_readfirstlane(t.M);
        t.N = __builtin_amdgcn_readfirstlane(t.N);
        t.A0 = uniform_ptr(t.A0);
        t.B0 = uniform_ptr(t.B0);
        t.C = uniform_ptr(t.C);
        return true;
    };
    int w = (int)blockIdx.x;
    TileRef t;
    // the next item of this block below `end` that is a tile
    auto advance = [&](int end) __attribute__((always_inline)) {
        for (w += stride; w < end; w += stride)
            if (decode(w, t)) return true;
        return false;
    };
    if (w < n_full) {         // whole tiles
        decode(w, t);
        gemm_tiles<MODE, 4, 4, false, CF32>(g, K0x, t, [&](TileRef& nx) __attribute__((always_inline)) {
            if (!advance(n_full)) return false;
            nx = t;
            return true;
        }, smem);
    }
    // sub-tiles: w is now this block's first item at or past n_full
    bool have = false;
    for (; w < n_items; w += stride)
        if (decode(w, t)) { have = true; break; }
    if (!have) return;
    auto next_sub = [&](TileRef& nx) __attribute__((always_inline)) {
        if (!advance(n_items)) return false;
        nx = t;
        return true;
    };
    if (sub == 1) gemm_tiles<MODE, 4, 4, false, CF32>(g, K0x, t, next_sub, smem);
    else if (sub == 2) gemm_tiles<MODE, 4, 2, false, CF32>(g, K0x, t, next_sub, smem);
    else gemm_tiles<MODE, 2, 2, false, CF32>(g, K0x, t, next_sub, smem);
}

__global__ __launch_bounds__(256) void gemm_nt_kernel(GemmArgs g) {
    extern __shared__ __align__(16) unsigned char smem[];
    int Mx = g.M, n_full = g.n_full, sub = g.sub, tile_n = g.tile_n;
    if (g.n_dev != nullptr) {
        // the kept-token count is a device value: clamp the rows to it and plan the tiles here, as the host does for sizes it
        // knows (the output shape depends on it)
        int n = *g.n_dev;
        n = __builtin_amdgcn_readfirstlane(n < 0 ? 0 : n);
        Mx = n < Mx ? n : Mx;
        plan_launch(Mx, g.N, (int)gridDim.x, n_full, sub, tile_n);
        n_full = __builtin_amdgcn_readfirstlane(n_full);
        sub = __builtin_amdgcn_readfirstlane(sub);
        tile_n = __builtin_amdgcn_readfirstlane(tile_n);
    }
    const TileRef whole{0, 0, Mx, g.N, g.A[0], g.B[0], g.C};
    int per = 0;
    const int parts = g.parts.count(Mx, per);
    if (__builtin_expect(parts > 1, 0)) {
        // An item is a part of a 128x128 tile.  The items of one part come together, column of tiles by column: an XCD's share
        // of them reads the same rows of A and B.
        const int tm = (Mx + 127) / 128, tiles = tm * ((g.N + 127) / 128), items = tiles * parts;
        if ((int)blockIdx.x >= items) return;
        const int w = xcd_order((int)blockIdx.x, items);
        const int part = __builtin_amdgcn_readfirstlane(w / tiles), tile = __builtin_amdgcn_readfirstlane(w % tiles);
        TileRef t = whole;
        t.m0 = __builtin_amdgcn_readfirstlane((tile % tm) * 128);
        t.n0 = __builtin_amdgcn_readfirstlane((tile / tm) * 128);
        per = __builtin_amdgcn_readfirstlane(per);
        gemm_tiles<0, 2, 2, true, false>(g, g.K[0], t, [](TileRef&) { return false; }, smem, part * per,
                                         min(g.parts.pairs, part * per + per), g.parts.slots + ((int64_t)tile * parts + part) * (128 * 128));
        return;
    }
    const int tiles_m = (Mx + 255) / 256, tiles_n = (g.N + 255) / 256;
    if (tile_n == 192) {
        // tiles of 256x192, all of one kind: block b takes tiles b, b + gridDim.x, ...
        const int tiles_n192 = (g.N + 191) / 192, n_items = tiles_m * tiles_n192;
        int w = (int)blockIdx.x;
        // with a device-side count there are as many blocks as CUs, whatever the number of tiles: a block
        // past the last tile would compute another block's tile a second time
        if (w >= n_items) return;
        auto tile = [&](int w, TileRef& t) __attribute__((always_inline)) {
            int bm, bn;
            tile_coords(xcd_order(w, n_items), tiles_m, tiles_n192, bm, bn);
            t = whole;
            t.m0 = __builtin_amdgcn_readfirstlane(bm * 256);
            t.n0 = __builtin_amdgcn_readfirstlane(bn * 192);
        };
        TileRef t;
        tile(w, t);
        gemm_tiles<0, 4, 3, false, false>(g, g.K[0], t, [&](TileRef& nx) __attribute__((always_inline)) {
            w += (int)gridDim.x;
            if (w >= n_items) return false;
            tile(w, nx);
            return true;
        }, smem);
        return;
    }
    gemm_items<0, false>(g, g.K[0], tiles_m * tiles_n, n_full, sub, (int)gridDim.x, [&](int l, TileRef& t, int& bm, int& bn) __attribute__((always_inline)) {
        t = whole;
        tile_coords(l, tiles_m, tiles_n, bm, bn);
    }, smem);
}

// CF32: C is fp32 (main-gradient buffers) and the products are added to it without rounding.
template <bool CF32>
__global__ __launch_bounds__(256) void gemm_tn_kernel(TnArgs g) {
    extern __shared__ __align__(16) unsigned char smem[];
    // Blocks behind those of the tiles sum the gain gradients up: where a CU has no tile left in the last, partial round they cost
    // nothing, where a launch of their own is 5 us ([841 of 2103 rows, H = 4096, F = 1792, 4/1 heads] layer call 231.0 and 226.3 us).
    if ((int)blockIdx.x >= g.n_blocks) {
        using T = std::conditional_t<CF32, float, bf16_t>;
        gain_grads_block<T, CF32>(g.gain, (int)blockIdx.x - g.n_blocks, reinterpret_cast<float (*)[33]>(smem));
        return;
    }
    int K0x = g.K[0];
    if (g.n_dev != nullptr) {           // the contraction is over the kept tokens: only its length depends on the count
        int n = *g.n_dev;
        n = __builtin_amdgcn_readfirstlane(n < 0 ? 0 : n);
        K0x = n < K0x ? n : K0x;
    }
    gemm_items<1, CF32>(g, K0x, g.end[TN_MAX - 1], g.n_full, g.sub, g.n_blocks, [&](int l, TileRef& t, int& bm, int& bn) __attribute__((always_inline)) {
        int j = 0, first = 0;
#pragma unroll
        for (int q = 0; q + 1 < TN_MAX; ++q) {
            const int e = g.end[q];
            j = l >= e ? q + 1 : j;
            first = l >= e ? e : first;
        }
        j = __builtin_amdgcn_readfirstlane(j);
        const GemmTnProb& p = g.p[j];
        t.M = p.M; t.N = p.N; t.A0 = p.A; t.B0 = p.B; t.C = p.C;
        tile_coords(l - first, (t.M + 255) / 256, (t.N + 255) / 256, bm, bn);
    }, smem);
}

// ---------------------------------------------------------------------------
// Grouped launch: up to GROUP_MAX independent products with 128x128 tiles, their contractions cut into parts when the
// tiles alone leave CUs idle.  For the products with a rank-r adapter matrix (an output of r columns or r rows with a long
// contraction: 2 to 32 tiles each) and for layers with few kept tokens: what they cost one by one is launches (5 us
// for the smallest kernel), blocks that wait for loads on a few CUs (a CU takes in about 60 B/ns whatever the number
// of active CUs), and a reduction each.  A launch has a fixed cost, though (scale * dY*b^T of 4096 rows, rank 64, K = 3072, six
// steps of 64 k in every block: 16 us and 6 us for the sum), so a single product of medium size gains nothing here.
// An item is one (tile, part); a part of a split tile leaves its fp32 accumulators in a 64 KB slot of its own and
// gemm_group_reduce_kernel adds the slots of a tile up in the order of the parts.  Blocks and reduction make the same plan
// from the live kept-token count, so the result is the same whether the count was known to the host or not.
// ---------------------------------------------------------------------------
struct GroupArgs {
    GemmGroupProb p[GROUP_MAX];
    int np;
    int n_cu;               // items that may be split over (and slots)
    const int32_t* n_dev;   // nullable: the live kept-token count (M in modes 0 and 2, K in mode 1), at most the one in p
    int gain;               // steps of 64 that parts have to take off the longest contraction
    float* slots;           // nullable: no splitting; n_cu slots and, behind them, the plan (one int)
    __host__ __device__ int32_t* plan() const { return reinterpret_cast<int32_t*>(slots + (size_t)n_cu * (128 * 128)); }
};

__host__ __device__ inline void group_sizes(const GemmGroupProb& p, int n_live, int& M, int& K) {
    M = p.mode != 1 && n_live < p.M ? n_live : p.M;
    K = p.mode == 1 && n_live < p.K ? n_live : p.K;
}
// Part sizes are numbered q = 2, 3, 4, 5, ...: 2, 3, 4, 6, 8, 12, ... steps of 64.
__host__ __device__ inline int group_step(int q) { return q & 1 ? 3 << ((q >> 1) - 1) : 1 << (q >> 1); }
// parts of a contraction of K, at least one
__host__ __device__ inline int group_parts(int K, int q) {
    const int k64 = (K + 63) >> 6, up = k64 + group_step(q) - 1;
    if (k64 <= 0) return 1;
    return q & 1 ? (up / 3) >> ((q >> 1) - 1) : up >> (q >> 1);
}
// Part size number of a launch: the smallest (at least 128 k: two steps) with which the items of all products fit one
// round of the CUs; -1, nothing is split, when even the whole tiles do not, or without slots.
static constexpr int GROUP_Q = 40;
// ... or when the longest contraction gets shorter by fewer than g.gain steps: a step is 0.35 to 0.5 us, against the launch that sums
// the parts up and their slots (GROUP_GAIN; GROUP_GAIN_ONE for a single product, whose sum is smaller).  Four products
// [4096, 64] of 48 and 16 steps, 128 tiles: 24 + 13 us in two parts, 33 whole; three of 48 steps, 96 tiles: 23 + 10 and 28; one, 32
// tiles: 16 + 6 in eight parts, 28 whole.  Contractions of up to 32 steps are faster whole whatever the rows (layer calls: H = 840, 215 rows 149
// and 172 us, H = 2048, 150 rows 167 and 172).  Those of 48 steps would be faster in four parts and more, which a batch of up to 1900 rows
// allows (H = 3072: 100 rows 202 and 210, 900 443 and 452, 1900 809 and 817), but with the count on the device their sums would have
// to be launched for longer batches too, where nothing is cut ([4096, 3072] 1216 and 1210, [4096 of 8192 in one sequence] 1436 and 1428).
__host__ __device__ inline int group_steps(const GroupArgs& g, int n_live) {        // of the longest contraction
    int most = 0;
#pragma unroll
    for (int j = 0; j < GROUP_MAX; ++j) {
        int M, K;
        group_sizes(g.p[j], n_live, M, K);
        const int k64 = (K + 63) >> 6;
        most = j < g.np && k64 > most ? k64 : most;
    }
    return most;
}
__host__ __device__ inline bool group_fits(const GroupArgs& g, int n_live, int q, bool& split) {
    int items = 0;
    split = false;
#pragma unroll
    for (int j = 0; j < GROUP_MAX; ++j) {
        int M, K;
        group_sizes(g.p[j], n_live, M, K);
        const int parts = group_parts(K, q);
        const bool used = j < g.np;
        items += used ? cdiv(M, 128) * cdiv(g.p[j].N, 128) * parts : 0;
        split |= used && parts > 1;
    }
    return items <= g.n_cu;
}
inline int group_plan_host(const GroupArgs& g, int n_live) {
    if (g.slots == nullptr) return -1;
    for (int q = 2; q < GROUP_Q; ++q) {
        bool split;
        const bool fits = group_fits(g, n_live, q, split);
        if (fits || !split) return split && group_steps(g, n_live) - group_step(q) >= g.gain ? q : -1;
    }
    return -1;
}
// The same with a candidate per lane: one after the other they cost every block several microseconds.
__device__ __forceinline__ int group_plan(const GroupArgs& g, int n_live) {
    if (g.slots == nullptr) return -1;
    const int q = 2 + (int)(threadIdx.x & 63);
    bool split = false;
    const bool fits = group_fits(g, n_live, q < GROUP_Q ? q : GROUP_Q - 1, split);
    const uint64_t done = __ballot(q < GROUP_Q && (fits || !split)), cut = __ballot(split);
    if (done == 0) return -1;
    const int first = __ffsll((unsigned long long)done) - 1;
    return ((cut >> first) & 1) && group_steps(g, n_live) - group_step(first + 2) >= g.gain ? first + 2 : -1;
}

// item -> product, tile and part; false past the last item
struct GroupItem {
    int j, M, K, m0, n0, parts, part;
};
__device__ __forceinline__ bool group_item(const GroupArgs& g, int n_live, int plan, int w, GroupItem& it) {
    it.j = -1;
    int tm_j = 1;
#pragma unroll
    for (int j = 0; j < GROUP_MAX; ++j) {
        int M, K;
        group_sizes(g.p[j], n_live, M, K);
        const int tm = cdiv(M, 128), parts = plan < 0 ? 1 : group_parts(K, plan);
        const int n = j < g.np ? tm * cdiv(g.p[j].N, 128) * parts : 0;
        if (it.j < 0 && w < n) { it.j = j; it.M = M; it.K = K; it.parts = parts; it.part = w; tm_j = tm; }
        w -= n;
    }
    if (it.j < 0) return false;
    const int t = it.part / it.parts;
    it.part -= t * it.parts;
    it.m0 = (t % tm_j) * 128;
    it.n0 = (t / tm_j) * 128;
    return true;
}

template <int MODE>
__device__ __forceinline__ void group_tile(const GroupArgs& ga, const GroupItem& it, int plan, int w, unsigned char* smem) {
    const GemmGroupProb& p = ga.p[it.j];
    GemmArgs g;
    g.A[0] = uniform_ptr(p.A); g.B[0] = uniform_ptr(p.B); g.K[0] = it.K; g.nseg = 1;
    g.C = uniform_ptr(p.C); g.M = it.M; g.N = p.N; g.beta = 0.f; g.alpha = p.alpha;
    g.n_dev = nullptr; g.a_idx = nullptr; g.a_rows = 0;
    const TileRef t{it.m0, it.n0, it.M, p.N, g.A[0], g.B[0], g.C};
    auto none = [](TileRef&) { return false; };
    if (it.parts > 1) {
        const int c = group_step(plan), pbeg = it.part * c, pend = min((it.K + 63) >> 6, pbeg + c);
        gemm_tiles<MODE, 2, 2, true, false>(g, it.K, t, none, smem, pbeg, pend, ga.slots + (int64_t)w * (128 * 128));
    } else {
        gemm_tiles<MODE, 2, 2, false, false>(g, it.K, t, none, smem);
    }
}

__global__ __launch_bounds__(256) void gemm_group_kernel(GroupArgs g) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int n_live = g.n_dev != nullptr ? __builtin_amdgcn_readfirstlane(max(*g.n_dev, 0)) : INT32_MAX;
    const int plan = __builtin_amdgcn_readfirstlane(group_plan(g, n_live));
    // for the reduction: made by every one of its blocks, the plan would cost it more than the sums (12 us for 4096 blocks)
    if (blockIdx.x == 0 && threadIdx.x == 0 && g.slots != nullptr) *g.plan() = plan;
    for (int w = blockIdx.x;; w += gridDim.x) {
        GroupItem it;
        if (!group_item(g, n_live, plan, w, it)) return;
        it.j = __builtin_amdgcn_readfirstlane(it.j);
        it.m0 = __builtin_amdgcn_readfirstlane(it.m0);
        it.n0 = __builtin_amdgcn_readfirstlane(it.n0);
        const int mode = g.p[it.j].mode;
        if (mode == 0) group_tile<0>(g, it, plan, w, smem);
        else if (mode == 1) group_tile<1>(g, it, plan, w, smem);
        else group_tile<2>(g, it, plan, w, smem);
        wait_vmcnt<0>();
        lds_barrier();          // the stages are free for the block's next item
    }
}

// C tile = alpha * (sum of its parts); tiles that were not split have been written already.  A block sums 8 rows of a
// tile, 4 columns per thread, eight parts in flight.  The grid has 16 blocks for every tile that the plan may hold.
__global__ __launch_bounds__(256) void gemm_group_reduce_kernel(GroupArgs g) {
    const int n_live = g.n_dev != nullptr ? max(*g.n_dev, 0) : INT32_MAX;
    const int plan = *g.plan();
    if (plan < 0) return;
    int t = (int)blockIdx.x >> 4, w0 = 0, jj = -1, Mj = 0, parts_j = 1, tm_j = 1, t_j = 0, w_j = 0;
#pragma unroll
    for (int j = 0; j < GROUP_MAX; ++j) {
        int M, K;
        group_sizes(g.p[j], n_live, M, K);
        const int tm = cdiv(M, 128), tiles = j < g.np ? tm * cdiv(g.p[j].N, 128) : 0;
        const int parts = group_parts(K, plan);
        if (jj < 0 && t < tiles) { jj = j; Mj = M; parts_j = parts; tm_j = tm; t_j = t; w_j = w0; }
        t -= tiles;
        w0 += tiles * parts;
    }
    if (jj < 0 || parts_j == 1) return;
    const GemmGroupProb& p = g.p[jj];
    const int row = ((int)blockIdx.x & 15) * 8 + ((int)threadIdx.x >> 5), col = ((int)threadIdx.x & 31) * 4;
    const int m = (t_j % tm_j) * 128 + row, n = (t_j / tm_j) * 128 + col;
    if (m >= Mj || n >= p.N) return;            // N is a multiple of 8
    const float* src = g.slots + (int64_t)(w_j + t_j * parts_j) * (128 * 128) + row * 128 + col;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 8
    for (int k = 0; k < parts_j; ++k) {
        const float4 v = *reinterpret_cast<const float4*>(src + (int64_t)k * (128 * 128));
        s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    uint2 o;
    o.x = pack_bf16x2(p.alpha * s.x, p.alpha * s.y);
    o.y = pack_bf16x2(p.alpha * s.z, p.alpha * s.w);
    *reinterpret_cast<uint2*>(static_cast<bf16_t*>(p.C) + (int64_t)m * p.N + n) = o;
}

// ---------------------------------------------------------------------------
// fp32 check-mode GEMM: 64x64 tile, 16-wide K step, 4x4 outputs per thread
// ---------------------------------------------------------------------------
template <int MODE>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmArgs g) {
    __shared__ float As[16][64 + 4];
    __shared__ float Bs[16][64 + 4];
    const int tid = threadIdx.x;
    const int tiles_m = (g.M + 63) / 64;        // of the upper bound: the grid was sized for it
    const int m0 = (blockIdx.x % tiles_m) * 64, n0 = (blockIdx.x / tiles_m) * 64;
    if (g.n_dev != nullptr) {
        const int n = live_rows(MODE != 1 ? g.M : g.K[0], g.n_dev);
        if (MODE != 1) g.M = n;
        else g.K[0] = n;
        if (m0 >= g.M) return;
    }
    const int tx = tid & 15, ty = tid >> 4;
    float acc[4][4] = {};
    for (int s = 0; s < g.nseg; ++s) {
        const float* A = static_cast<const float*>(g.A[s]);
        const float* B = static_cast<const float*>(g.B[s]);
        const int K = g.K[s];
        for (int k0 = 0; k0 < K; k0 += 16) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int e = tid + 256 * i;      // 0..1023
                int kk, r;
                if (MODE != 1) { kk = e & 15; r = e >> 4; } else { r = e & 63; kk = e >> 6; }
                const bool ka = k0 + kk < K;
                float av = 0.f, bv = 0.f;
                if (ka && m0 + r < g.M) {
                    const int64_t arow = (MODE == 0 && s == 0 && g.a_idx != nullptr) ? g.a_idx[m0 + r] : m0 + r;
                    av = MODE != 1 ? A[arow * K + k0 + kk] : A[(int64_t)(k0 + kk) * g.M + m0 + r];
                }
                if (ka && n0 + r < g.N)
                    bv = MODE == 0 ? B[(int64_t)(n0 + r) * K + k0 + kk] : B[(int64_t)(k0 + kk) * g.N + n0 + r];
                As[kk][r] = av;
                Bs[kk][r] = bv;
            }
            __syncthreads();
#pragma unroll
            for (int kk = 0; kk < 16; ++kk) {
                float a[4], b[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) { a[i] = As[kk][ty * 4 + i]; b[i] = Bs[kk][tx * 4 + i]; }
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc[i][j] += a[i] * b[j];
            }
            __syncthreads();
        }
    }
    float* C = static_cast<float*>(g.C);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int m = m0 + ty * 4 + i;
        if (m >= g.M) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int n = n0 + tx * 4 + j;
            if (n >= g.N) continue;
            float* p = C + (int64_t)m * g.N + n;
            *p = (g.beta != 0.f) ? g.alpha * acc[i][j] + g.beta * *p : g.alpha * acc[i][j];
        }
    }
}


// per-lane load and store offsets are 32-bit with the upper half reserved for "out of range"
static bool offsets_fit(int64_t M, int64_t N, int64_t K) {
    const int64_t lim = (int64_t)1 << 31;
    return M * K * 2 < lim && N * K * 2 < lim && (M + 256) * N * 2 < lim;
}

// C = the sum of the parts of a product that was cut into some
__global__ __launch_bounds__(256) void gemm_nt_sum_kernel(NtParts pt, int M, bf16_t* __restrict__ C) {
    int per;
    const int parts = pt.count(M, per), vpr = pt.N / 8;
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v >= (int64_t)M * vpr) return;
    const int j = (int)(v / vpr), c = (int)(v % vpr) * 8;
    float o[8];
    pt.load(M, parts, j, c, o);
    Vec<bf16_t>::store(C + (int64_t)j * pt.N + c, o);
}

hipError_t launch_gemm_nt_sum(const NtParts& parts, int M, void* C, hipStream_t st) {
    int per;
    if (M <= 0 || parts.count(M, per) == 1) return hipSuccess;
    gemm_nt_sum_kernel<<<ceil_div((int64_t)M * parts.N, 256 * 8), 256, 0, st>>>(parts, M, (bf16_t*)C);
    return hipGetLastError();
}

NtParts gemm_nt_parts(int dtype, const GemmSeg* segs, int nseg, int N, float* slots) {
    NtParts p{slots, N, 0, compute_units(), 0};
    if (dtype != CF_BF16 || slots == nullptr) return p;
    for (int s = 0; s < nseg; ++s) p.pairs += ceil_div(segs[s].K, 64);
    // the more tiles, the fewer parts: the last number of tile rows with more than one
    const int tn = ceil_div(N, 128);
    int per;
    for (int tm = 1; 2 * tm * tn <= p.n_cu; ++tm) {
        p.max_rows = tm * 128;
        if (p.count(tm * 128, per) == 1) {
            p.max_rows = (tm - 1) * 128;
            break;
        }
    }
    return p;
}

hipError_t launch_gemm_nt(int dtype, const GemmSeg* segs, int nseg, void* C, int M, int N, hipStream_t st, const int32_t* n_dev,
                          const int32_t* a_idx, int64_t a_rows, const NtParts* parts) {
    if (M <= 0 || N <= 0) return hipSuccess;
    if (a_idx != nullptr && a_rows <= 0) return hipErrorInvalidValue;
    if (nseg > MAX_SEG) return hipErrorInvalidValue;
    GemmArgs g{};
    for (int s = 0; s < nseg; ++s) {
        if (segs[s].K <= 0) return hipErrorInvalidValue;
        g.A[s] = segs[s].A;
        g.B[s] = segs[s].B;
        g.K[s] = segs[s].K;
        if (dtype == CF_BF16 && !offsets_fit(M, N, segs[s].K)) return hipErrorInvalidValue;
    }
    g.nseg = nseg;
    g.C = C; g.M = M; g.N = N; g.alpha = 1.f; g.sub = 1; g.tile_n = 256;
    g.n_dev = n_dev; g.a_idx = a_idx; g.a_rows = a_rows;
    if (dtype == CF_F32) {
        gemm_f32_kernel<0><<<ceil_div(M, 64) * ceil_div(N, 64), 256, 0, st>>>(g);
        return hipGetLastError();
    }
    if (a_idx != nullptr && a_rows * g.K[0] * 2 >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    static std::atomic<uint64_t> lds_ok{0};
    const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(&gemm_nt_kernel), GEMM_SMEM, lds_ok);
    if (e != hipSuccess) return e;
    if (parts != nullptr) g.parts = *parts;
    int per, items = plan_launch(M, N, compute_units(), g.n_full, g.sub, g.tile_n);
    const int np = g.parts.count(M, per);
    if (np > 1) items = ceil_div(M, 128) * ceil_div(N, 128) * np;
    // a block walks through its items; with a device-side count the blocks plan for themselves (for
    // as many blocks as CUs) and those without an item leave at once
    const int grid = n_dev != nullptr ? compute_units() : std::min(items, compute_units());
    gemm_nt_kernel<<<grid, 256, GEMM_SMEM, st>>>(g);
    return hipGetLastError();
}

hipError_t launch_gemm_tn(int dtype, const GemmTnProb* probs, int np, int K, float beta, hipStream_t st, bool c_f32,
                          const int32_t* n_dev, const GainGrads* gains) {
    if (np < 1 || np > TN_MAX) return hipErrorInvalidValue;
    if (c_f32 && dtype == CF_BF16 && beta != 1.f) return hipErrorInvalidValue;
    if (gains != nullptr && (K <= 0 || dtype == CF_F32)) {
        const hipError_t e = launch_gain_grads(dtype, *gains, c_f32, st);
        if (e != hipSuccess) return e;
    }
    if (K <= 0) {           // empty contraction: C = beta*C; only beta in {0,1} is supported by the API
        for (int j = 0; j < np && beta == 0.f; ++j) {
            const hipError_t e = launch_fill_zero(probs[j].C, (size_t)probs[j].M * probs[j].N * dtype_size(dtype), st);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    TnArgs g{};
    g.K[0] = K; g.nseg = 1; g.beta = beta; g.alpha = 1.f; g.n_dev = n_dev;
    if (dtype == CF_F32) {
        for (int j = 0; j < np; ++j) {
            g.A[0] = probs[j].A; g.B[0] = probs[j].B; g.C = probs[j].C; g.M = probs[j].M; g.N = probs[j].N;
            gemm_f32_kernel<1><<<ceil_div(g.M, 64) * ceil_div(g.N, 64), 256, 0, st>>>(g);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    int tiles = 0;
    for (int j = 0; j < TN_MAX; ++j) {
        if (j < np) {
            const GemmTnProb& p = probs[j];
            if (p.M <= 0 || p.N <= 0 || !offsets_fit(p.M, p.N, K)) return hipErrorInvalidValue;
            g.p[j] = p;
            tiles += ceil_div(p.M, 256) * ceil_div(p.N, 256);
        }
        g.end[j] = tiles;       // behind the last product: no tile there
    }
    static std::atomic<uint64_t> lds_ok{0}, lds_ok_f32{0};
    void (*const kernel)(TnArgs) = c_f32 ? gemm_tn_kernel<true> : gemm_tn_kernel<false>;
    const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kernel), GEMM_SMEM, c_f32 ? lds_ok_f32 : lds_ok);
    if (e != hipSuccess) return e;
    plan_tiles(tiles, compute_units(), g.n_full, g.sub);
    g.n_blocks = std::min(g.n_full + (tiles - g.n_full) * g.sub, compute_units());
    int more = 0;
    if (gains != nullptr && tiles > compute_units()) {
        g.gain = *gains;
        more = gain_grad_units(gains->H);
    } else if (gains != nullptr) {
        // Up to one round a launch of their own, as the number of launches of such a call has always been, which test_gpu_routes.py
        // holds to.  Not for speed: beside the products 94 layer calls of 7 to 228 tiles are 1.03 times as fast (1.01 to 1.07, 1 to 7 us).
        const hipError_t eg = launch_gain_grads(dtype, *gains, c_f32, st);
        if (eg != hipSuccess) return eg;
    }
    kernel<<<g.n_blocks + more, 256, GEMM_SMEM, st>>>(g);
    return hipGetLastError();
}

size_t gemm_group_slot_bytes() { return (size_t)compute_units() * 128 * 128 * sizeof(float) + 256; }

hipError_t launch_gemm_group(int dtype, const GemmGroupProb* probs, int np, hipStream_t st, float* slots,
                             const int32_t* n_dev) {
    if (np < 1 || np > GROUP_MAX) return hipErrorInvalidValue;
    if (dtype == CF_F32) {
        for (int j = 0; j < np; ++j) {
            const GemmGroupProb& p = probs[j];
            GemmArgs g{};
            g.A[0] = p.A; g.B[0] = p.B; g.K[0] = p.K; g.nseg = 1; g.C = p.C; g.M = p.M; g.N = p.N; g.alpha = p.alpha;
            g.n_dev = n_dev;
            const int grid = ceil_div(p.M, 64) * ceil_div(p.N, 64);
            if (p.mode == 0) gemm_f32_kernel<0><<<grid, 256, 0, st>>>(g);
            else if (p.mode == 1) gemm_f32_kernel<1><<<grid, 256, 0, st>>>(g);
            else gemm_f32_kernel<2><<<grid, 256, 0, st>>>(g);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    GroupArgs g{};
    int64_t tiles = 0;
    bool all_tn = true;
    for (int j = 0; j < np; ++j) {
        const GemmGroupProb& p = probs[j];
        if (p.M <= 0 || p.N <= 0 || p.K <= 0) return hipErrorInvalidValue;
        if (!offsets_fit(p.M, p.N, p.K)) return hipErrorInvalidValue;
        g.p[j] = p;
        tiles += (int64_t)ceil_div(p.M, 128) * ceil_div(p.N, 128);
        all_tn = all_tn && p.mode == 1;
    }
    g.np = np; g.n_cu = compute_units(); g.n_dev = n_dev; g.slots = slots; g.gain = np == 1 ? GROUP_GAIN_ONE : GROUP_GAIN;
    // no live count can lead to parts: their sum is not launched (products over the kept tokens have the same tiles whatever the count, and
    // are cut alike)
    if (group_steps(g, INT32_MAX) - group_step(2) < g.gain || (all_tn && 2 * tiles > g.n_cu)) g.slots = slots = nullptr;
    static std::atomic<uint64_t> lds_ok{0};
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(&gemm_group_kernel), GEMM_SMEM, lds_ok);
    if (e != hipSuccess) return e;
    // a live count below the bound may be split although the bound is not: the launches are sized for either
    const bool may_split = slots != nullptr && (n_dev != nullptr || group_plan_host(g, INT32_MAX) >= 0);
    const int grid = (int)(may_split ? g.n_cu : std::min<int64_t>(tiles, g.n_cu));
    gemm_group_kernel<<<grid, 256, GEMM_SMEM, st>>>(g);
    e = hipGetLastError();
    if (e != hipSuccess || !may_split) return e;
    // a plan with parts has at most n_cu items, so at most n_cu / 2 of its tiles are split; whole ones count too
    const int rtiles = (int)std::min<int64_t>(tiles, g.n_cu);
    gemm_group_reduce_kernel<<<16 * rtiles, 256, 0, st>>>(g);
    return hipGetLastError();
}

}  // namespace cf
