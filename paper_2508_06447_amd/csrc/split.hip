// Second half of the split projections (few rows): the float partial sums that split_gemm_kernel (gemm.hip) leaves are
// added in split order and finished the way the fused epilogues of the large projections do.
#include "slim_common.h"
#include <math.h>

namespace slim {

// out[m, :] = R[m, :] + sum over the splits (out may be R).  Reads splits * 4 + 2 bytes per element, mostly from the caches
// that the partial sums have just been written through: 4 splits of 512 x 4096 in 9 us (launch included).  n % 8 == 0.
__global__ void __launch_bounds__(256) split_residual_kernel(const float* __restrict__ partial, int splits, size_t split_stride,
                                                             size_t chunks, const bf16_t* R, bf16_t* out) {
    const size_t c = ((size_t)blockIdx.x * 256 + threadIdx.x) * 8;
    if (c >= chunks * 8) return;
    f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int s = 0; s < splits; ++s) {
        const float* p = partial + s * split_stride + c;
        lo += *reinterpret_cast<const f32x4*>(p);
        hi += *reinterpret_cast<const f32x4*>(p + 4);
    }
    float f[8];
    Elem<bf16_t>::unpack(*reinterpret_cast<const uint4*>(R + c), f);
#pragma unroll
    for (int i = 0; i < 4; ++i) { f[i] += lo[i]; f[4 + i] += hi[i]; }
    *reinterpret_cast<uint4*>(out + c) = Elem<bf16_t>::pack(f);
}

int launch_split_residual(const float* partial, int splits, int m, int n, const void* residual, void* out, hipStream_t st) {
    const size_t chunks = (size_t)m * n / 8;
    hipLaunchKernelGGL(split_residual_kernel, dim3((unsigned)((chunks + 255) / 256)), dim3(256), 0, st, partial, splits, (size_t)m * n,
                       chunks, (const bf16_t*)residual, (bf16_t*)out);
    return check_launch();
}

// The same for rows that a norm follows, one per workgroup: also 1 / rms of the finished row, or with a gain the normalised row (from registers; n <= 8192).  2 splits
// of 512 x 4096 read 17 MB, mostly from the caches.
template <bool NORM>
__global__ void __launch_bounds__(256) split_residual_rows_kernel(const float* __restrict__ partial, int splits, size_t split_stride, int n, const bf16_t* R,
                                                                  bf16_t* out, float eps, const bf16_t* __restrict__ gain, bf16_t* __restrict__ normed,
                                                                  float* __restrict__ rstd) {
    __shared__ float part[4];
    const size_t row = (size_t)blockIdx.x * n;
    uint4 y[4];
    float ss = 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int c = (u * 256 + threadIdx.x) * 8;
        if (c >= n) break;
        f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
        for (int s = 0; s < splits; ++s) {
            const float* p = partial + s * split_stride + row + c;
            lo += *reinterpret_cast<const f32x4*>(p);
            hi += *reinterpret_cast<const f32x4*>(p + 4);
        }
        float f[8];
        Elem<bf16_t>::unpack(*reinterpret_cast<const uint4*>(R + row + c), f);
#pragma unroll
        for (int i = 0; i < 4; ++i) { f[i] += lo[i]; f[4 + i] += hi[i]; }
        y[u] = Elem<bf16_t>::pack(f);
        *reinterpret_cast<uint4*>(out + row + c) = y[u];
        Elem<bf16_t>::unpack(y[u], f);
#pragma unroll
        for (int i = 0; i < 8; ++i) ss += f[i] * f[i];
    }
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
    __syncthreads();
    const float inv = 1.0f / sqrtf((part[0] + part[1] + part[2] + part[3]) / (float)n + eps);
    if (!NORM) {
        if (threadIdx.x == 0) rstd[blockIdx.x] = inv;
        return;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int c = (u * 256 + threadIdx.x) * 8;
        if (c >= n) break;
        float f[8], g[8];
        Elem<bf16_t>::unpack(y[u], f);
        Elem<bf16_t>::unpack(*reinterpret_cast<const uint4*>(gain + c), g);
#pragma unroll
        for (int i = 0; i < 8; ++i) f[i] = g[i] * (f[i] * inv);
        *reinterpret_cast<uint4*>(normed + row + c) = Elem<bf16_t>::pack(f);
    }
}

int launch_split_residual_rows(const float* partial, int splits, int m, int n, const void* residual, void* out, float eps, const void* gain, void* normed,
                               float* rstd, hipStream_t st) {
    hipLaunchKernelGGL(gain ? split_residual_rows_kernel<true> : split_residual_rows_kernel<false>, dim3(m), dim3(256), 0, st, partial, splits, (size_t)m * n, n,
                       (const bf16_t*)residual, (bf16_t*)out, eps, (const bf16_t*)gain, (bf16_t*)normed, rstd);
    return check_launch();
}

// Query / Key / Value states of one token row per workgroup: scale (1/rms), bias, rotation of the heads of 128 and one
// rounding; with a window query the per-(token, kv head) dots of the rounded keys with it.  A thread takes features
// 8 u .. 8 u + 7 of a head and the eight 64 above them, so rotation partners meet in one thread and the dot of a head in
// eight neighbouring lanes.
struct SplitHeads {
    bf16_t* out[3];
    const bf16_t* bias[3];
    int heads[3];                        // 0: no such matrix
    int rope[3];
    int score;                           // matrix whose heads are dotted with qt, -1: none
};
struct SplitFreq { double inv_freq[64]; };

__global__ void __launch_bounds__(384) split_heads_kernel(const float* __restrict__ partial, int splits, size_t split_stride, int n,
                                                          SplitHeads o, const float* __restrict__ rstd,
                                                          const int* __restrict__ pos, SplitFreq fr,
                                                          const float* __restrict__ qt, float* __restrict__ token_scores) {
    __shared__ __align__(16) float cs[64], sn[64];
    const int m = blockIdx.x, tid = threadIdx.x;
    const float* row = partial + (size_t)m * n;
    if (tid < 64) {
        double s, c;
        sincos((double)(pos ? pos[m] : m) * fr.inv_freq[tid], &s, &c);
        cs[tid] = (float)c;
        sn[tid] = (float)s;
    }
    const float sc = rstd ? rstd[m] : 1.f;
    __syncthreads();
    const int units = n / 16;
    for (int q = tid; q < units; q += blockDim.x) {
        int head = q >> 3;
        const int u = (q & 7) * 8;
        float lo[8], hi[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) lo[i] = hi[i] = 0.f;
        const float* p = row + head * 128 + u;
#pragma unroll 4
        for (int s = 0; s < splits; ++s) {
            const f32x4 a0 = *reinterpret_cast<const f32x4*>(p + s * split_stride), a1 = *reinterpret_cast<const f32x4*>(p + s * split_stride + 4);
            const f32x4 b0 = *reinterpret_cast<const f32x4*>(p + s * split_stride + 64), b1 = *reinterpret_cast<const f32x4*>(p + s * split_stride + 68);
#pragma unroll
            for (int i = 0; i < 4; ++i) { lo[i] += a0[i]; lo[4 + i] += a1[i]; hi[i] += b0[i]; hi[4 + i] += b1[i]; }
        }
        int mat = 0;
        if (head >= o.heads[0]) { head -= o.heads[0]; mat = 1; }
        if (mat == 1 && head >= o.heads[1]) { head -= o.heads[1]; mat = 2; }
        const bf16_t* bias = mat == 0 ? o.bias[0] : mat == 1 ? o.bias[1] : o.bias[2];
        bf16_t* out = mat == 0 ? o.out[0] : mat == 1 ? o.out[1] : o.out[2];
        const int heads = mat == 0 ? o.heads[0] : mat == 1 ? o.heads[1] : o.heads[2];
        const int rope = mat == 0 ? o.rope[0] : mat == 1 ? o.rope[1] : o.rope[2];
        float bl[8] = {}, bh[8] = {};
        if (bias) {
            Elem<bf16_t>::unpack(*reinterpret_cast<const uint4*>(bias + head * 128 + u), bl);
            Elem<bf16_t>::unpack(*reinterpret_cast<const uint4*>(bias + head * 128 + 64 + u), bh);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float x1 = lo[i] * sc + bl[i], x2 = hi[i] * sc + bh[i];
            lo[i] = rope ? x1 * cs[u + i] - x2 * sn[u + i] : x1;
            hi[i] = rope ? x2 * cs[u + i] + x1 * sn[u + i] : x2;
        }
        const uint4 pl = Elem<bf16_t>::pack(lo), ph = Elem<bf16_t>::pack(hi);
        bf16_t* dst = out + ((size_t)m * heads + head) * 128 + u;
        *reinterpret_cast<uint4*>(dst) = pl;
        *reinterpret_cast<uint4*>(dst + 64) = ph;
        if (mat == o.score) {                                // uniform over the eight lanes of a head
            Elem<bf16_t>::unpack(pl, lo);
            Elem<bf16_t>::unpack(ph, hi);
            float dot = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) dot += lo[i] * qt[head * 128 + u + i] + hi[i] * qt[head * 128 + 64 + u + i];
            dot += __shfl_xor(dot, 1, 64);
            dot += __shfl_xor(dot, 2, 64);
            dot += __shfl_xor(dot, 4, 64);
            if ((q & 7) == 0) token_scores[(size_t)m * heads + head] = dot;
        }
    }
}

int launch_split_heads(const float* partial, int splits, int m, const SplitHeadsArgs& a, const float* rstd, const int* pos, float theta,
                       const float* qt, float* token_scores, hipStream_t st) {
    SplitHeads o;
    int n = 0;
    for (int i = 0; i < 3; ++i) {
        o.out[i] = (bf16_t*)a.out[i];
        o.bias[i] = (const bf16_t*)a.bias[i];
        o.heads[i] = a.heads[i];
        o.rope[i] = a.rope[i];
        n += a.heads[i] * 128;
    }
    o.score = qt ? a.score : -1;
    SplitFreq fr;
    for (int i = 0; i < 64; ++i) fr.inv_freq[i] = pow((double)theta, -2.0 * (double)i / 128.0);
    const int threads = n / 16 < 384 ? (n / 16 + 63) / 64 * 64 : 384;
    hipLaunchKernelGGL(split_heads_kernel, dim3(m), dim3(threads), 0, st, partial, splits, (size_t)m * n, n, o, rstd, pos, fr, qt,
                       token_scores);
    return check_launch();
}

}  // namespace slim
