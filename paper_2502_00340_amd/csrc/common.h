// Internal helpers shared by the HIP translation units of the library (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "centrifuge.h"

namespace cf {

typedef unsigned short bf16_t;   // raw bfloat16 bits

__device__ __forceinline__ float bf16_to_f32(bf16_t h) {
    return __uint_as_float(((unsigned)h) << 16);
}

// round-to-nearest-even; inputs are finite in every use here
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
    unsigned u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}

// two fp32 -> packed bf16 pair (round-to-nearest-even in hardware: v_cvt_pk_bf16_f32)
__device__ __forceinline__ unsigned pack_bf16x2(float lo, float hi) {
    typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_hw;
    bf16x2_hw v;
    v[0] = (__bf16)lo;
    v[1] = (__bf16)hi;
    return __builtin_bit_cast(unsigned, v);
}

// 16-byte vector access of VN elements, widened to fp32
template <typename T> struct Vec;

template <> struct Vec<float> {
    static constexpr int N = 4;
    __device__ static __forceinline__ void load(const float* p, float (&o)[4]) {
        float4 v = *reinterpret_cast<const float4*>(p);
        o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
    }
    __device__ static __forceinline__ void store(float* p, const float (&i)[4]) {
        *reinterpret_cast<float4*>(p) = make_float4(i[0], i[1], i[2], i[3]);
    }
};

template <> struct Vec<bf16_t> {
    static constexpr int N = 8;
    __device__ static __forceinline__ void load(const bf16_t* p, float (&o)[8]) {
        uint4 v = *reinterpret_cast<const uint4*>(p);
        unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            o[2 * i] = __uint_as_float(w[i] << 16);
            o[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
        }
    }
    __device__ static __forceinline__ void store(bf16_t* p, const float (&i)[8]) {
        uint4 v;
        v.x = pack_bf16x2(i[0], i[1]);
        v.y = pack_bf16x2(i[2], i[3]);
        v.z = pack_bf16x2(i[4], i[5]);
        v.w = pack_bf16x2(i[6], i[7]);
        *reinterpret_cast<uint4*>(p) = v;
    }
};

template <typename T> __device__ __forceinline__ float to_f32(T v);
template <> __device__ __forceinline__ float to_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ float to_f32<bf16_t>(bf16_t v) { return bf16_to_f32(v); }
template <typename T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float v) { return f32_to_bf16(v); }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Raises a kernel's dynamic LDS limit once per device (the attribute belongs to the device's
// copy of the kernel); `done` holds one bit per device ordinal.  Safe from several host threads:
// a second thread at worst sets the attribute again.
static inline hipError_t allow_dynamic_lds(const void* kernel, int bytes, std::atomic<uint64_t>& done) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = 1ull << (dev & 63);
    if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess) done.fetch_or(bit, std::memory_order_release);
    return e;
}

static inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
static inline int ceil_div(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }
static inline size_t dtype_size(int dtype) { return dtype == CF_F32 ? 4 : 2; }

// Number of live rows of a launch (kept tokens).  dev == nullptr: exactly n, known to the host.
// Otherwise the count lives on the device (the index build earlier on the same stream wrote it) and
// n is only its upper bound: it sizes grids and buffer strides, and every kernel works on
// min(*dev, n) rows, so no launch has to wait for the host to learn the count.
struct RowCount {
    int n;
    const int32_t* dev;
};
__device__ __forceinline__ int live_rows(int n, const int32_t* dev) {
    if (dev == nullptr) return n;
    const int v = *dev;
    return v < 0 ? 0 : (v < n ? v : n);
}

// ---- internal launchers (one per translation unit) --------------------------

// index.hip
size_t index_ws_bytes(int64_t n_tokens);
hipError_t launch_keep_index(const uint8_t* mask, int B, int S, int32_t* idx, int32_t* cu_kept,
                             int32_t* n_kept_dev, void* ws, hipStream_t st);
// the same with the per-block counts in a device array of the library's own (no workspace, no
// allocation); at most IDX_STATIC_MAX_TOKENS tokens
static constexpr int64_t IDX_STATIC_MAX_TOKENS = (int64_t)1 << 24;
hipError_t launch_keep_index_static(const uint8_t* mask, int B, int S, int32_t* idx, int32_t* cu_kept,
                                    int32_t* n_kept_dev, hipStream_t st);
hipError_t launch_gather(const void* src, int64_t cols_bytes, const int32_t* idx, RowCount rows,
                         void* dst, hipStream_t st);

// gemm.hip
struct GemmSeg {
    const void* A;
    const void* B;
    int K;
};
// C [M,N] = sum_seg A_seg [M,K] * B_seg [N,K]^T, up to six segments; all matrices dense row-major.
// n_dev (nullable): the kept-token count on the device; then M is only an upper bound and the kernel uses
// min(*n_dev, M) rows.  a_idx (nullable, segment 0): row m of A is row a_idx[m] of a longer
// matrix (the gather of the upstream gradient folded into the A-tile loads); a_rows = rows of that matrix.
// parts (nullable): where the product may be left in parts instead of in C.
struct NtParts;
hipError_t launch_gemm_nt(int dtype, const GemmSeg* segs, int nseg, void* C, int M, int N, hipStream_t st,
                          const int32_t* n_dev = nullptr, const int32_t* a_idx = nullptr, int64_t a_rows = 0,
                          const NtParts* parts = nullptr);

// An NT product with few output tiles and a long contraction may leave its result in parts: fp32 [128,128] slots, tile by tile
// (column of tiles by column), a tile's parts one after the other, for the kernel that reads the product to add up (or
// launch_gemm_nt_sum).  A CU takes in the operands of a 128x128 tile at 0.35 us per 64 k whatever the others do, so that few
// tiles are a long chain on few CUs.  A function of the live rows: launch and readers agree on it, and the result does not
// depend on who knows the count.
struct NtParts {
    float* slots;       // null: never in parts
    int N, pairs;       // columns; 64-wide steps of all segments
    int n_cu;           // slots
    int max_rows;       // more rows than this are one part: a kernel that is not concerned finds out with a compare
    // Parts of a contraction for M rows, `per` steps each.  The items fit one round of the CUs, a part has eight steps or more (three
    // microseconds; the ring's prologue is another two) and a reader sixteen parts at most; less than 16 steps saved do
    // not pay for the fp32 slots.  [100, 4096], K = 28672: 268 -> 74 us (its reader 8 -> 15), [841, 512], K = 4096: 27.5 -> 12.0 (4.9 -> 6.2),
    // [841, 1792], K = 4096, 98 tiles in two parts: 31.6 -> 22.7 (6.4 -> 7.6).
    __host__ __device__ int count(int M, int& per) const {
        per = pairs;
        if (M <= 0 || M > max_rows) return 1;
        const int tiles = ((M + 127) / 128) * ((N + 127) / 128);
        int parts = n_cu / tiles;
        if (parts > pairs / 8) parts = pairs / 8;
        if (parts > 16) parts = 16;
        if (parts < 2) return 1;
        per = (pairs + parts - 1) / parts;
        if (pairs - per < 16) { per = pairs; return 1; }
        return (pairs + per - 1) / per;
    }
    // columns c .. c+VN-1 of row j of M
    template <int VN>
    __device__ __forceinline__ void load(int M, int parts, int j, int c, float (&o)[VN]) const {
        const float* p = slots + (int64_t)((c >> 7) * ((M + 127) >> 7) + (j >> 7)) * parts * (128 * 128) + (j & 127) * 128 + (c & 127);
#pragma unroll
        for (int e = 0; e < VN; ++e) o[e] = 0.f;
#pragma unroll 4
        for (int k = 0; k < parts; ++k, p += 128 * 128) {
#pragma unroll
            for (int q = 0; q < VN / 4; ++q) {
                const float4 a = reinterpret_cast<const float4*>(p)[q];
                o[4 * q] += a.x; o[4 * q + 1] += a.y; o[4 * q + 2] += a.z; o[4 * q + 3] += a.w;
            }
        }
    }
};
NtParts gemm_nt_parts(int dtype, const GemmSeg* segs, int nseg, int N, float* slots);
hipError_t launch_gemm_nt_sum(const NtParts& parts, int M, void* C, hipStream_t st);    // M: the live rows, known to the host

// One launch for up to TN_MAX products over the same K rows: C_j [M,N] = beta*C_j + A_j [K,M]^T * B_j [K,N].  c_f32 (bf16
// dtype, beta = 1): the C_j are fp32 (main-gradient buffers) and the accumulators are added to them without rounding to
// bf16.  No product may read another one's result.  n_dev (nullable): the kept-token count, which bounds K.
static constexpr int TN_MAX = 7;
struct GemmTnProb {
    const void *A, *B;
    void* C;
    int M, N;
};
// gains (nullable): the gain gradients, too, c_f32 as their acc_f32; no product may read them.
struct GainGrads;
hipError_t launch_gemm_tn(int dtype, const GemmTnProb* probs, int np, int K, float beta, hipStream_t st, bool c_f32 = false,
                          const int32_t* n_dev = nullptr, const GainGrads* gains = nullptr);

// One launch for up to GROUP_MAX independent products C [M,N] = alpha * op(A) * op(B) with few output tiles:
//   mode 0 ("NT"): A [M,K], B [N,K]    1 ("TN"): A [K,M], B [K,N]    2 ("NN"): A [M,K], B [K,N]
// No product may read another one's result.  slots (nullable, gemm_group_slot_bytes(), 16-byte aligned): scratch that
// lets the contractions be split over idle CUs.  n_dev (nullable): the live kept-token count, which bounds M in
// modes 0 and 2 and K in mode 1.
static constexpr int GROUP_MAX = 8;
static constexpr int GROUP_GAIN = 47, GROUP_GAIN_ONE = 36;      // steps of 64 that parts have to save (see gemm.hip)
struct GemmGroupProb {
    const void *A, *B;
    void* C;
    int M, N, K;
    int mode;
    float alpha;
};
size_t gemm_group_slot_bytes();
hipError_t launch_gemm_group(int dtype, const GemmGroupProb* probs, int np, hipStream_t st, float* slots = nullptr,
                             const int32_t* n_dev = nullptr);

// rowlocal.hip
// act (nullable) also receives silu(gate)*up; d_gate may alias d_act.  parts: d_act may lie there; it is then summed
// up into d_act first.  copy_src (nullable):
// a [.., copy_cols] tensor whose rows copy_idx (null: the first n_rows) the same launch copies to copy_dst
// [n_rows, copy_cols] (the compact upstream gradient that the parameter-gradient GEMM contracts over).
hipError_t launch_swiglu_bwd(int dtype, void* d_act, const void* gate, const void* up,
                             const int32_t* idx, RowCount rows, int F, void* d_gate, void* d_up,
                             void* act, hipStream_t st, const NtParts& parts, const void* copy_src = nullptr, int copy_cols = 0,
                             void* copy_dst = nullptr, const int32_t* copy_idx = nullptr);
// dx_out = res + rmsnorm_bwd(dh; x, g); dg_partial (nullable: the gains are frozen) receives the gain gradient's
// [rmsnorm_bwd_blocks(n_rows), H] fp32 partials for launch_gain_grads.
// h_out (nullable, [n_rows, H], may be dh): also receives the normalised rows rmsnorm(x)*g.  parts: dh may lie
// there; it is then summed up into dh first.
int rmsnorm_bwd_blocks(int n_rows);
hipError_t launch_rmsnorm_bwd(int dtype, void* dh, const void* x, const void* g,
                              const int32_t* idx, const void* res, RowCount rows, int H, float eps,
                              void* dx_out, float* dg_partial, hipStream_t st, const NtParts& parts, void* h_out = nullptr);
// The gain gradients of both norms from their partials: gain_grads_block in launches of their own or with a launch_gemm_tn.
struct GainGrads {
    const float *partial1, *partial2;   // of the norm whose gain gradient dg1 / dg2 is
    void *dg1, *dg2;                    // [H]; fp32 and added to (acc_f32), or of the dtype and written
    int H, n_rows;
    const int32_t* n_dev;
};
hipError_t launch_gain_grads(int dtype, const GainGrads& g, bool acc_f32, hipStream_t st);
// fp32 gq [n_rows, hq*d] and gk [n_rows, hk*d], in place: transposed rotary rotation at position idx[j] % S
// (idx null: j % S); cos, sin are [S, d/2] fp32
hipError_t launch_rope_bwd_f32(void* gq, int hq, void* gk, int hk, const int32_t* idx, RowCount rows, int d, int S,
                               const float* cos, const float* sin, hipStream_t st);
// D[j,h] = sum_c da[j,h*d+c] * a[row,h*d+c], row = a_idx ? a_idx[j] : j; with a_idx the same launch also
// writes the compact copies a_out[j,:] = a[row,:] and (q_src non-null) q_out[j,:] = q_src[row,:]
hipError_t launch_attn_rowdot(int dtype, const void* da, const void* a, RowCount rows, int Hq, int d,
                              float* D, hipStream_t st, const int32_t* a_idx = nullptr, void* a_out = nullptr,
                              const void* q_src = nullptr, void* q_out = nullptr);
hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t st);
// CUs of the current device (cached per device ordinal; 256 if the query fails)
inline int compute_units() {
    static std::atomic<int> cache[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 256;
    std::atomic<int>& c = cache[dev & 63];
    int n = c.load(std::memory_order_relaxed);
    if (n == 0) {
        int v = 0;
        n = (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0) ? v : 256;
        c.store(n, std::memory_order_relaxed);
    }
    return n;
}

// Blocks that the rmsnorm backward deals its live rows out to, two rows per iteration, and so the partials of a gain gradient.
__host__ __device__ inline int rmsnorm_bwd_nblk(int n_rows) {
    const int pairs = (n_rows + 1) / 2;
    return pairs < 512 ? pairs : 512;
}

// Block `unit` of gain_grad_units(H), of 256 threads: out[c] = sum_b partial[b,c] for 32 columns of one norm (8 lanes x 4 columns), 32 row groups
// stride through the partials with 16-byte loads, many in flight; H is a multiple of 4.
// The order of the additions is fixed, so the result is reproducible.  ACC: out is fp32 and the
// sum is added to it (main-gradient accumulation).  red: LDS.
__host__ __device__ inline int gain_grad_units(int H) { return 2 * ((H + 31) / 32); }
template <typename T, bool ACC>
__device__ __forceinline__ void gain_grads_block(const GainGrads& g, int unit, float (*red)[33]) {
    const int H = g.H, norm = unit & 1, c0 = (unit >> 1) * 32;
    const float* partial = norm == 0 ? g.partial1 : g.partial2;
    T* out = (T*)(norm == 0 ? g.dg1 : g.dg2);
    const int nblk = rmsnorm_bwd_nblk(live_rows(g.n_rows, g.n_dev));     // the partials that the backward kernel wrote
    const int cq = threadIdx.x & 7, rg = threadIdx.x >> 3;
    const int c = c0 + cq * 4;
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    if (c < H) {
#pragma unroll 8
        for (int b = rg; b < nblk; b += 32) {
            const float4 v = *reinterpret_cast<const float4*>(partial + (int64_t)b * H + c);
            s[0] += v.x; s[1] += v.y; s[2] += v.z; s[3] += v.w;
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) red[rg][cq * 4 + e] = s[e];
    __syncthreads();
    if (threadIdx.x < 32 && c0 + (int)threadIdx.x < H) {
        float t = 0.f;
#pragma unroll
        for (int r = 0; r < 32; ++r) t += red[r][threadIdx.x];
        if (ACC) out[c0 + threadIdx.x] += from_f32<T>(t);
        else out[c0 + threadIdx.x] = from_f32<T>(t);
    }
}

}  // namespace cf
