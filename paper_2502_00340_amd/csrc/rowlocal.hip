// Row-local backward operators on kept rows (Sec. 3.2: element-wise products
// of a row-sparse gradient inherit its row sparsity).  Every kernel takes an
// optional kept-row index for tensors that are still stored full length, so
// the gather of those tensors is folded into the read.  Arithmetic is fp32;
// storage is fp32 or bf16.  All of them are HBM-bound streaming kernels.
#include <type_traits>

#include "common.h"

namespace cf {

__device__ __forceinline__ float sigmoidf_(float z) { return 1.0f / (1.0f + __expf(-z)); }

// d_gate = d_act * up * s(1 + gate(1-s)), d_up = d_act * gate * s,  s = sigmoid(gate);
// act (nullable) = gate * s * up, the SwiGLU product rebuilt in the same pass.
// d_gate may alias d_act (every element is read before it is written, by the same thread).
// copy_src (nullable): after its share of the SwiGLU elements every thread also copies its share of
// copy_dst[j, :] = copy_src[copy_idx[j], :] (copy_idx null: row j; copy_cols columns, a multiple of VN): the kept rows of the
// upstream gradient, which the down projection's parameter-gradient GEMM contracts over; folding the
// copy in here saves the launch of a gather kernel.
template <typename T>
__global__ __launch_bounds__(256) void swiglu_bwd_kernel(T* d_act,
                                                         const T* __restrict__ gate,
                                                         const T* __restrict__ up,
                                                         const int32_t* __restrict__ idx,
                                                         int n_max, const int32_t* __restrict__ n_dev, int F, T* d_gate,
                                                         T* __restrict__ d_up, T* __restrict__ act,
                                                         const T* __restrict__ copy_src, int copy_cols,
                                                         T* __restrict__ copy_dst, const int32_t* __restrict__ copy_idx,
                                                         NtParts parts) {
    constexpr int VN = Vec<T>::N;
    // vectors are counted in 32 bits where every matrix is below 2 GiB (the bf16 layers); a 64-bit division per vector
    // is a tenth of the pass
    typedef typename std::conditional<VN == 8, unsigned, uint64_t>::type Count;
    const int n_rows = live_rows(n_max, n_dev);
    if (copy_src != nullptr) {
        const Count cvpr = copy_cols / VN;
        const Count ctotal = (Count)n_rows * cvpr;
        for (Count v = (Count)blockIdx.x * 256 + threadIdx.x; v < ctotal; v += gridDim.x * 256) {
            const int j = (int)(v / cvpr);
            const int c = (int)(v % cvpr) * VN;
            *reinterpret_cast<uint4*>(copy_dst + (int64_t)j * copy_cols + c) =
                *reinterpret_cast<const uint4*>(copy_src + (int64_t)(copy_idx ? copy_idx[j] : j) * copy_cols + c);
        }
    }
    const Count vpr = F / VN;
    const Count total = (Count)n_rows * vpr;
    // In parts: every thread first sums up what it is going to read.  (A second loop with the sum in the load's place, let
    // alone a branch there, costs the calls without parts a microsecond or two a pass.)
    if constexpr (VN == 8) {
        int per;
        const int np = parts.count(n_rows, per);
        if (__builtin_expect(np > 1, 0))
            for (Count v = (Count)blockIdx.x * 256 + threadIdx.x; v < total; v += gridDim.x * 256) {
                const int j = (int)(v / vpr), c = (int)(v % vpr) * VN;
                float da[VN];
                parts.load(n_rows, np, j, c, da);
                Vec<T>::store(d_act + (int64_t)j * F + c, da);
            }
    }
    for (Count v = (Count)blockIdx.x * 256 + threadIdx.x; v < total; v += gridDim.x * 256) {
        const int j = (int)(v / vpr);
        const int c = (int)(v % vpr) * VN;
        const int64_t row = idx ? idx[j] : j;
        float g[VN], u[VN], da[VN], dg[VN], du[VN], a[VN];
        Vec<T>::load(gate + row * F + c, g);
        Vec<T>::load(up + row * F + c, u);
        Vec<T>::load(d_act + (int64_t)j * F + c, da);
#pragma unroll
        for (int e = 0; e < VN; ++e) {
            const float s = sigmoidf_(g[e]);
            dg[e] = da[e] * u[e] * s * (1.0f + g[e] * (1.0f - s));
            du[e] = da[e] * g[e] * s;
            a[e] = g[e] * s * u[e];
        }
        Vec<T>::store(d_gate + (int64_t)j * F + c, dg);
        Vec<T>::store(d_up + (int64_t)j * F + c, du);
        if (act) Vec<T>::store(act + (int64_t)j * F + c, a);
    }
}

// dx_out[j,:] = res[j,:] + rstd*(u - n*mean(u*n)),  n = x*rstd, u = dh*g
// dg_partial[block,:] = sum over the block's rows of dh*n
// h_out (nullable, may be dh: every element is read before it is written, by the same thread): h_out[j,:] = n*g, the normalised row itself: the parameter-gradient GEMMs of the linears behind
// this norm need it as an operand, and the row and its rstd are in registers here anyway.
// A block owns one row at a time, NV 16-byte vectors per thread, and works on two rows per
// iteration so that the loads of the second row overlap the reduction of the first; every
// load of an iteration (x, dh, res of both rows) is issued before the first reduction.
// The rows are dealt out to rmsnorm_bwd_nblk(live rows) blocks whatever the grid is (a grid sized for
// an upper bound of the row count leaves the blocks past that number idle), so the partial sums, and
// with them the rounding of the gain gradient, depend on the number of live rows alone.
template <typename T, int NV>
__global__ __launch_bounds__(256) void rmsnorm_bwd_kernel(T* dh,
                                                          const T* __restrict__ x,
                                                          const T* __restrict__ g,
                                                          const int32_t* __restrict__ idx,
                                                          const T* __restrict__ res, int n_max,
                                                          const int32_t* __restrict__ n_dev,
                                                          int H, float eps, T* __restrict__ dx_out,
                                                          float* __restrict__ dg_partial, T* h_out, NtParts parts) {
    constexpr int VN = Vec<T>::N;
    __shared__ float red[16];
    const int n_rows = live_rows(n_max, n_dev);
    const int nblk = rmsnorm_bwd_nblk(n_rows);
    if ((int)blockIdx.x >= nblk) return;
    const int vpr = H / VN;
    float gv[NV][VN], dgacc[NV][VN];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int v = threadIdx.x + i * 256;
#pragma unroll
        for (int e = 0; e < VN; ++e) { dgacc[i][e] = 0.f; gv[i][e] = 0.f; }
        if (v < vpr) Vec<T>::load(g + v * VN, gv[i]);
    }
    const int wave = threadIdx.x >> 6;
    if constexpr (VN == 8) {        // in parts: as in the SwiGLU pass
        int per;
        const int np = parts.count(n_rows, per);
        if (__builtin_expect(np > 1, 0))
            for (int j0 = blockIdx.x * 2; j0 < n_rows; j0 += nblk * 2)
                for (int j = j0; j < min(j0 + 2, n_rows); ++j)
                    for (int v = threadIdx.x; v < vpr; v += 256) {
                        float o[VN];
                        parts.load(n_rows, np, j, v * VN, o);
                        Vec<T>::store(dh + (int64_t)j * H + v * VN, o);
                    }
    }
    for (int j0 = blockIdx.x * 2; j0 < n_rows; j0 += nblk * 2) {
        float xv[2][NV][VN], dv[2][NV][VN], rv[2][NV][VN];
        float ss[2] = {0.f, 0.f}, sd[2] = {0.f, 0.f};
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int j = j0 + r;
            const bool live = j < n_rows;
            const int64_t row = live ? (idx ? idx[j] : j) : 0;
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const int v = threadIdx.x + i * 256;
                if (live && v < vpr) {
                    Vec<T>::load(x + row * H + v * VN, xv[r][i]);
                    Vec<T>::load(dh + (int64_t)j * H + v * VN, dv[r][i]);
                    Vec<T>::load(res + (int64_t)j * H + v * VN, rv[r][i]);
                } else {
#pragma unroll
                    for (int e = 0; e < VN; ++e) { xv[r][i][e] = 0.f; dv[r][i][e] = 0.f; rv[r][i][e] = 0.f; }
                }
            }
        }
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int i = 0; i < NV; ++i)
#pragma unroll
                for (int e = 0; e < VN; ++e) {
                    ss[r] += xv[r][i][e] * xv[r][i][e];
                    sd[r] += dv[r][i][e] * gv[i][e] * xv[r][i][e];
                }
#pragma unroll
        for (int r = 0; r < 2; ++r) { ss[r] = wave_sum(ss[r]); sd[r] = wave_sum(sd[r]); }
        __syncthreads();
        if ((threadIdx.x & 63) == 0) {
            red[wave] = ss[0]; red[4 + wave] = sd[0]; red[8 + wave] = ss[1]; red[12 + wave] = sd[1];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int j = j0 + r;
            if (j >= n_rows) break;
            const float ssr = red[8 * r] + red[8 * r + 1] + red[8 * r + 2] + red[8 * r + 3];
            const float sdr = red[8 * r + 4] + red[8 * r + 5] + red[8 * r + 6] + red[8 * r + 7];
            const float rstd = rsqrtf(ssr / (float)H + eps);
            const float c = sdr * rstd / (float)H;          // mean(u*n)
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const int v = threadIdx.x + i * 256;
                if (v < vpr) {
                    float o[VN];
#pragma unroll
                    for (int e = 0; e < VN; ++e) {
                        const float n = xv[r][i][e] * rstd;
                        o[e] = rv[r][i][e] + rstd * (dv[r][i][e] * gv[i][e] - n * c);
                        dgacc[i][e] += dv[r][i][e] * n;
                    }
                    Vec<T>::store(dx_out + (int64_t)j * H + v * VN, o);
                    if (h_out != nullptr) {
#pragma unroll
                        for (int e = 0; e < VN; ++e) o[e] = xv[r][i][e] * rstd * gv[i][e];
                        Vec<T>::store(h_out + (int64_t)j * H + v * VN, o);
                    }
                }
            }
        }
    }
    if (dg_partial == nullptr) return;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int v = threadIdx.x + i * 256;
        if (v < vpr) {
#pragma unroll
            for (int e = 0; e < VN; ++e) dg_partial[(int64_t)blockIdx.x * H + v * VN + e] = dgacc[i][e];
        }
    }
}

template <typename T, bool ACC = false>
__global__ __launch_bounds__(256) void colsum_finish_kernel(GainGrads g) {
    __shared__ float red[32][33];
    gain_grads_block<T, ACC>(g, blockIdx.x, red);
}

// D[j,h] = sum_c da[j,h*d+c] * a[row,h*d+c]   (the FlashAttention-backward row term), row = a_idx ?
// a_idx[j] : j.  With a_idx the pass also writes the compact copies a_out[j,:] = a[row,:] and, when
// q_src is given, q_out[j,:] = q_src[row,:] (the gathers of attn_out and q folded into this read).
template <typename T>
__global__ __launch_bounds__(256) void attn_rowdot_kernel(const T* __restrict__ da,
                                                          const T* __restrict__ a, int n_max,
                                                          const int32_t* __restrict__ n_dev,
                                                          int Hq, int d, float* __restrict__ D,
                                                          const int32_t* __restrict__ a_idx, T* __restrict__ a_out,
                                                          const T* __restrict__ q_src, T* __restrict__ q_out) {
    constexpr int VN = Vec<T>::N;
    const int n_rows = live_rows(n_max, n_dev);
    const int lanes = d / VN;                    // lanes per (row, head): power of two <= 64
    const int64_t total = (int64_t)n_rows * Hq * lanes;
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    float s = 0.f;
    int64_t pair = gid / lanes;
    if (gid < total) {
        const int part = (int)(gid % lanes);
        int64_t src = pair;
        if (a_idx != nullptr) src = (int64_t)a_idx[pair / Hq] * Hq + pair % Hq;
        float p[VN], q[VN];
        Vec<T>::load(da + pair * d + part * VN, p);
        Vec<T>::load(a + src * d + part * VN, q);
#pragma unroll
        for (int e = 0; e < VN; ++e) s += p[e] * q[e];
        if (a_idx != nullptr) {
            Vec<T>::store(a_out + pair * d + part * VN, q);        // widening and rounding back is exact
            if (q_src != nullptr)
                *reinterpret_cast<uint4*>(q_out + pair * d + part * VN) =
                    *reinterpret_cast<const uint4*>(q_src + src * d + part * VN);
        }
    }
    for (int o = lanes >> 1; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (gid < total && (gid % lanes) == 0) D[pair] = s;
}

// Transposed rotary rotation, in place: for i < d/2 and c = cos[pos,i], s = sin[pos,i]
//   dx[i] = dy[i]*c + dy[i+d/2]*s,   dx[i+d/2] = dy[i+d/2]*c - dy[i]*s
// of the hq heads of a row of gq and the hk heads of a row of gk (one launch: the smallest kernel costs 5 us).
// One thread per vector of VN frequencies of one (row, head); d/2 is a multiple of VN.
// fp32 check mode only: the matrix-core attention kernels rotate where they write dq and dk.
__global__ __launch_bounds__(256) void rope_bwd_f32_kernel(float* __restrict__ gq, int hq, float* __restrict__ gk, int hk,
                                                           const int32_t* __restrict__ idx,
                                                           int n_max, const int32_t* __restrict__ n_dev, int d, int S,
                                                           const float* __restrict__ cs,
                                                           const float* __restrict__ sn) {
    typedef float T;
    constexpr int VN = Vec<T>::N;
    const int n_rows = live_rows(n_max, n_dev);
    const int half = d / 2, vph = half / VN, heads = hq + hk;           // vph: vectors per head half
    const int64_t total = (int64_t)n_rows * heads * vph;
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < total; t += (int64_t)gridDim.x * 256) {
        const int iv = (int)(t % vph);
        const int64_t rh = t / vph;
        const int h = (int)(rh % heads);
        const int64_t j = rh / heads;
        const int pos = (int)((idx ? (int64_t)idx[j] : j) % S);
        T* p = (h < hq ? gq + (j * hq + h) * d : gk + (j * hk + (h - hq)) * d) + iv * VN;
        float lo[VN], hi[VN], olo[VN], ohi[VN], c[VN], s[VN];
        Vec<T>::load(p, lo);
        Vec<T>::load(p + half, hi);
        const float* pc = cs + (int64_t)pos * half + iv * VN;
        const float* ps = sn + (int64_t)pos * half + iv * VN;
#pragma unroll
        for (int e = 0; e < VN; ++e) { c[e] = pc[e]; s[e] = ps[e]; }
#pragma unroll
        for (int e = 0; e < VN; ++e) {
            olo[e] = lo[e] * c[e] + hi[e] * s[e];
            ohi[e] = hi[e] * c[e] - lo[e] * s[e];
        }
        Vec<T>::store(p, olo);
        Vec<T>::store(p + half, ohi);
    }
}

// ---------------------------------------------------------------------------

static int stream_grid(int64_t vec_total) {
    int64_t g = (vec_total + 255) / 256;
    if (g > 256 * 32) g = 256 * 32;
    if (g < 1) g = 1;
    return (int)g;
}

hipError_t launch_swiglu_bwd(int dtype, void* d_act, const void* gate, const void* up,
                             const int32_t* idx, RowCount rows, int F, void* d_gate, void* d_up,
                             void* act, hipStream_t st, const NtParts& parts, const void* copy_src, int copy_cols, void* copy_dst,
                             const int32_t* copy_idx) {
    const int n_rows = rows.n;
    if (n_rows <= 0) return hipSuccess;
    if (dtype == CF_F32)
        swiglu_bwd_kernel<float><<<stream_grid((int64_t)n_rows * F / 4), 256, 0, st>>>(
            (float*)d_act, (const float*)gate, (const float*)up, idx, n_rows, rows.dev, F,
            (float*)d_gate, (float*)d_up, (float*)act, (const float*)copy_src, copy_cols, (float*)copy_dst, copy_idx, parts);
    else
        swiglu_bwd_kernel<bf16_t><<<stream_grid((int64_t)n_rows * F / 8), 256, 0, st>>>(
            (bf16_t*)d_act, (const bf16_t*)gate, (const bf16_t*)up, idx, n_rows, rows.dev, F,
            (bf16_t*)d_gate, (bf16_t*)d_up, (bf16_t*)act, (const bf16_t*)copy_src, copy_cols, (bf16_t*)copy_dst, copy_idx,
            parts);
    return hipGetLastError();
}

int rmsnorm_bwd_blocks(int n_rows) {
    return n_rows < 1 ? 1 : rmsnorm_bwd_nblk(n_rows);
}

template <typename T>
static void rmsnorm_bwd_dispatch(int nv, int nblk, hipStream_t st, void* dh, const void* x, const void* g,
                                 const int32_t* idx, const void* res, RowCount rows, int H, float eps,
                                 void* dx_out, float* dg_partial, void* h_out, const NtParts& parts) {
#define CF_RMS_BWD(NV)                                                                               \
    rmsnorm_bwd_kernel<T, NV><<<nblk, 256, 0, st>>>((T*)dh, (const T*)x, (const T*)g, idx,      \
                                                    (const T*)res, rows.n, rows.dev, H, eps, (T*)dx_out, dg_partial, (T*)h_out, parts)
    if (nv <= 1) CF_RMS_BWD(1);
    else if (nv <= 2) CF_RMS_BWD(2);
    else if (nv <= 4) CF_RMS_BWD(4);
    else CF_RMS_BWD(8);
#undef CF_RMS_BWD
}

hipError_t launch_rmsnorm_bwd(int dtype, void* dh, const void* x, const void* g,
                              const int32_t* idx, const void* res, RowCount rows, int H, float eps,
                              void* dx_out, float* dg_partial, hipStream_t st, const NtParts& parts, void* h_out) {
    const int n_rows = rows.n;
    if (n_rows <= 0) return hipSuccess;
    const int nblk = rmsnorm_bwd_blocks(n_rows);
    const int vn = dtype == CF_F32 ? 4 : 8;
    const int nv = ceil_div(H / vn, 256);           // 16-byte vectors per thread (at most 8, checked by the API)
    if (dtype == CF_F32) rmsnorm_bwd_dispatch<float>(nv, nblk, st, dh, x, g, idx, res, rows, H, eps, dx_out, dg_partial, h_out, parts);
    else rmsnorm_bwd_dispatch<bf16_t>(nv, nblk, st, dh, x, g, idx, res, rows, H, eps, dx_out, dg_partial, h_out, parts);
    return hipGetLastError();
}

hipError_t launch_gain_grads(int dtype, const GainGrads& g, bool acc_f32, hipStream_t st) {
    const int grid = gain_grad_units(g.H);
    if (acc_f32) colsum_finish_kernel<float, true><<<grid, 256, 0, st>>>(g);
    else if (dtype == CF_F32) colsum_finish_kernel<float><<<grid, 256, 0, st>>>(g);
    else colsum_finish_kernel<bf16_t><<<grid, 256, 0, st>>>(g);
    return hipGetLastError();
}

hipError_t launch_rope_bwd_f32(void* gq, int hq, void* gk, int hk, const int32_t* idx, RowCount rows, int d, int S,
                               const float* cos, const float* sin, hipStream_t st) {
    const int n_rows = rows.n, vn = Vec<float>::N;
    if (n_rows <= 0) return hipSuccess;
    if ((d / 2) % vn != 0) return hipErrorInvalidValue;
    const int grid = stream_grid((int64_t)n_rows * (hq + hk) * (d / 2 / vn));
    rope_bwd_f32_kernel<<<grid, 256, 0, st>>>((float*)gq, hq, (float*)gk, hk, idx, n_rows, rows.dev, d, S, cos, sin);
    return hipGetLastError();
}

hipError_t launch_attn_rowdot(int dtype, const void* da, const void* a, RowCount rows, int Hq, int d,
                              float* D, hipStream_t st, const int32_t* a_idx, void* a_out, const void* q_src,
                              void* q_out) {
    const int n_rows = rows.n;
    if (n_rows <= 0) return hipSuccess;
    const int vn = dtype == CF_F32 ? 4 : 8;
    const int64_t total = (int64_t)n_rows * Hq * (d / vn);
    const int grid = (int)((total + 255) / 256);
    if (dtype == CF_F32)
        attn_rowdot_kernel<float><<<grid, 256, 0, st>>>((const float*)da, (const float*)a, n_rows, rows.dev, Hq, d, D,
                                                        a_idx, (float*)a_out, (const float*)q_src, (float*)q_out);
    else
        attn_rowdot_kernel<bf16_t><<<grid, 256, 0, st>>>((const bf16_t*)da, (const bf16_t*)a, n_rows, rows.dev, Hq, d, D,
                                                         a_idx, (bf16_t*)a_out, (const bf16_t*)q_src, (bf16_t*)q_out);
    return hipGetLastError();
}

}  // namespace cf
