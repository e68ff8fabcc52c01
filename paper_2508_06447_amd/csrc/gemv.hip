// Projections of ONE token (decoding phase of Fig. 2: "QKV Generation" and "FFN" for the newly decoded token):
//   out[n] = s * (w[n, :] . x) (+ bias[n]) (+ residual[n]),   or   silu(s * w0[n, :] . x) * (s * w1[n, :] . x),
// s = the token's 1/rms (fused RMSNorm with a folded gain: formed by every workgroup from the token, or read from
// *scale) or 1.  HBM-bound: every weight is read once, 16 bytes per lane, with a non-temporal hint (nothing will find it in
// a cache again before the next token).
//
// A workgroup owns four weight rows (four features, or the gate and up rows of two) and its four waves deal their 1 KB
// pieces out among themselves (short rows: each wave owns four): a row piece meets the token's piece in registers, so no load waits for a
// barrier, and U pieces of each row (32 to 112 registers per lane, 8 to 28 for the token's) are requested before the first is used.  With a wave per four rows, the token
// staged in LDS and two pieces in flight, a launch of 4096 x 4096 was one round of workgroups that spent half its time on
// latency.  Weights from HBM, us before -> now (bf16): 6144 x 4096 12.0 -> 9.2, 4096 x 4096 9.9 -> 7.1, 28672 x 4096 42.8 ->
// 33.9 (6.9 TB/s), 4096 x 14336 27.3 -> 18.4; without the hint 9.9 / 7.4 / 37.4 / 20.3.
//
// Up to three matrices with their own bias and output share one launch (the Query, Key and Value projections), and a
// segment can ask for RoPE at the token's position: its workgroups then own the features {i, i+1, i+64, i+65} of a 128-wide head,
// so that the rotate-half partners meet in one workgroup.
#include "slim_common.h"
#include <math.h>

namespace slim {

struct GemvSeg {
    const void* w;
    const void* bias;        // null: none
    void* out;
    int n;                   // output features (a multiple of 4 except in the last segment; of 128 with rope)
    int rope;                // != 0: rotate heads of 128 features
};
struct GemvArgs {
    GemvSeg seg[3];
    int n_seg;
    const void* w_up;        // SwiGLU: second matrix of segment 0 (n_seg == 1)
    const void* x;
    const float* scale;      // null: 1 (or the in-kernel statistic when norm_eps >= 0)
    float norm_eps;          // >= 0: s = 1 / sqrt(mean(x^2) + norm_eps) computed here
    const void* residual;    // segment 0 only
    int k;
    int position;            // RoPE position of the token
    double inv_freq[64];
};

constexpr int kGemvRows = 4; // weight rows per workgroup
constexpr int kGemvGrid = 1 << 22;                       // workgroups per row of the grid (work items per dimension stay below 2^32)

// KW: waves that share the rows (4, or 1: each of the four waves has four rows of its own).
template <typename T, bool SWIGLU, int U, int KW>
__global__ void __launch_bounds__(256) gemv_kernel(GemvArgs a) {
    constexpr int V = Elem<T>::kVec, R = kGemvRows, FPW = SWIGLU ? R / 2 : R;   // features of four rows
    __shared__ float red[4][R + 1];                      // per wave: its share of the rows' sums and of the token's sum of squares
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), tid = KW == 1 ? lane : threadIdx.x;
    const int K = a.k, nchunk = K / V;
    long long j = blockIdx.x + (long long)blockIdx.y * kGemvGrid;
    if (KW == 1) j = j * 4 + wave;
    int s = 0;                                           // the segment of these four rows, j: their place in it
    while (s < a.n_seg - 1 && j >= (a.seg[s].n + FPW - 1) / FPW) { j -= (a.seg[s].n + FPW - 1) / FPW; ++s; }
    const GemvSeg sg = a.seg[s];
    const int N = sg.n;
    if (j * FPW >= N) return;                            // (the last row of the grid is not full)
    const int n0 = (int)(sg.rope ? (j >> 5) * 128 + (j & 31) * 2 : j * FPW);
    auto feature = [&](int r) { return sg.rope ? n0 + (r & 1) + (r >> 1) * 64 : n0 + r; };
    const T* rows[R];
#pragma unroll
    for (int r = 0; r < R; ++r)                          // features past the end repeat the last one
        rows[r] = (SWIGLU && r >= FPW ? (const T*)a.w_up : (const T*)sg.w) + (size_t)min(feature(SWIGLU ? r % FPW : r), N - 1) * K;
    const T* x = (const T*)a.x;
    uint4 raw[U][R], xr[U];
    auto load = [&](int c0) {                            // pieces past the end: the token's values are zeros there
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = c0 + u * 64 * KW, cc = min(c, nchunk - 1);
            xr[u] = c < nchunk ? *reinterpret_cast<const uint4*>(x + (size_t)cc * V) : make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < R; ++r) raw[u][r] = load_stream16(rows[r] + (size_t)cc * V);
        }
    };
    load(tid);
    float cs = 1.f, sn = 0.f;                            // of the thread's rotation index, while the weights are on their way
    if (sg.rope && tid < R) {
        const double ang = (double)a.position * a.inv_freq[(n0 + (tid & 1)) & 63];
        const double kk = rint(ang * 0.15915494309189535);
        sincosf((float)fma(-kk, 2.4492935982947064e-16, fma(-kk, 6.283185307179586, ang)), &sn, &cs);
    }
    float acc[R], ss = 0.f;
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = 0.f;
    for (int c = tid; c - lane < nchunk; c += 64 * KW * U) { // (wave-uniform bound)
        if (c != tid) load(c);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float xf[V];
            Elem<T>::unpack(xr[u], xf);
#pragma unroll
            for (int i = 0; i < V; ++i) ss += xf[i] * xf[i];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                float f[V];
                Elem<T>::unpack(raw[u][r], f);
                if (c + u * 64 * KW >= nchunk) continue;     // (a repeated piece may hold an infinity: 0 times it is not 0)
#pragma unroll
                for (int i = 0; i < V; ++i) acc[r] += f[i] * xf[i];
            }
        }
    }
    // The four sums in one butterfly: after the first two exchanges a lane carries one row, row lane / 16.
#pragma unroll
    for (int h = R / 2, o = 32; h >= 1; h >>= 1, o >>= 1) {
        const bool up = lane & o;
#pragma unroll
        for (int i = 0; i < h; ++i) {
            const float keep = up ? acc[i + h] : acc[i], give = up ? acc[i] : acc[i + h];
            acc[i] = keep + __shfl_xor(give, o, 64);
        }
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) acc[0] += __shfl_xor(acc[0], o, 64);
    if (KW == 1) {
        if (a.norm_eps >= 0.f) ss = wave_sum(ss);
    } else {
        if ((lane & 15) == 0) red[wave][lane >> 4] = acc[0];
        if (a.norm_eps >= 0.f) {
            ss = wave_sum(ss);
            if (lane == 0) red[wave][R] = ss;
        }
        __syncthreads();
    }
    float own[R];                                        // KW 1: the rows' sums, in every lane
    if (KW == 1) {
#pragma unroll
        for (int r = 0; r < R; ++r) own[r] = __shfl(acc[0], r * 16, 64);
    }
    if (tid >= FPW) return;
    auto row_sum = [&](int r) {
        if (KW == 1) return r == 0 ? own[0] : r == 1 ? own[1] : r == 2 ? own[2] : own[3];
        return red[0][r] + red[1][r] + red[2][r] + red[3][r];
    };
    const int n = feature(tid);
    if (n >= N) return;
    float sc = a.scale ? *a.scale : 1.0f;
    if (a.norm_eps >= 0.f) sc = 1.0f / sqrtf((KW == 1 ? ss : row_sum(R)) / (float)K + a.norm_eps);
    float val = row_sum(tid) * sc;
    if (SWIGLU) val = val / (1.0f + __expf(-val)) * (row_sum(FPW + tid) * sc);
    const T* bias = (const T*)sg.bias;
    if (bias) val += Elem<T>::ld(bias + n);
    if (sg.rope) {                                       // partner: the row 64 features away, with scale and bias applied
        float other = row_sum(tid ^ 2) * sc;
        if (bias) other += Elem<T>::ld(bias + (n ^ 64));
        val = (n & 64) ? val * cs + other * sn : val * cs - other * sn;
    }
    if (s == 0 && a.residual) val += Elem<T>::ld((const T*)a.residual + n);
    Elem<T>::st((T*)sg.out + n, val);
}

// Rows of up to 192 pieces of 16 bytes are a wave's own: dealt to four waves they leave some without any (128256 rows of bf16, us dealt / own: k_in 256
// 38.5 / 15.6, 512 42.8 / 20.0, 1024 50.6 / 37.7, 1280 56.0 / 46.5).  Pieces in flight per row: all of a wave's share where that is 7 or fewer (7 beats 4 by 3 % at k_in 14336 although fewer
// waves fit: one wait instead of two).
constexpr int kGemvOwnPieces = 192;

template <typename T, bool S>
static void launch_gemv_u(const GemvArgs& a, dim3 grid, hipStream_t st) {
    const int pieces = (a.k / Elem<T>::kVec + 255) / 256;
#define SLIM_GEMV(U, KW) hipLaunchKernelGGL((gemv_kernel<T, S, U, KW>), grid, dim3(256), 0, st, a)
    if (a.k / Elem<T>::kVec <= 128) SLIM_GEMV(2, 1);
    else if (a.k / Elem<T>::kVec <= kGemvOwnPieces) SLIM_GEMV(3, 1);
    else if (pieces <= 2) SLIM_GEMV(2, 4);
    else if (pieces > 4 && pieces <= 7) SLIM_GEMV(7, 4);
    else SLIM_GEMV(4, 4);
#undef SLIM_GEMV
}

static int launch_gemv_args(const GemvArgs& a, int dtype, hipStream_t st) {
    const int per = a.w_up ? kGemvRows / 2 : kGemvRows;
    long long wgs = 0;
    for (int s = 0; s < a.n_seg; ++s) wgs += ((long long)a.seg[s].n + per - 1) / per;
    if (a.k / (dtype == SLIM_BF16 ? Elem<bf16_t>::kVec : Elem<float>::kVec) <= kGemvOwnPieces) wgs = (wgs + 3) / 4;
    const dim3 grid((unsigned)(wgs < kGemvGrid ? wgs : kGemvGrid), (unsigned)((wgs + kGemvGrid - 1) / kGemvGrid));
    if (dtype == SLIM_BF16) { if (a.w_up) launch_gemv_u<bf16_t, true>(a, grid, st); else launch_gemv_u<bf16_t, false>(a, grid, st); }
    else                    { if (a.w_up) launch_gemv_u<float, true>(a, grid, st);  else launch_gemv_u<float, false>(a, grid, st); }
    return check_launch();
}

// One matrix (or gate/up pair).  k_in a multiple of 8 (bf16) or 4 (fp32), x and the weights 16-byte aligned
// (checked by the caller).  norm_eps >= 0 computes the scale from x itself.
int launch_gemv(const void* w0, const void* w1, const void* x, const float* scale, float norm_eps, const void* bias,
                const void* residual, int n_out, int k_in, int dtype, void* out, hipStream_t st) {
    GemvArgs a{};
    a.seg[0] = GemvSeg{w0, bias, out, n_out, 0};
    a.n_seg = 1;
    a.w_up = w1;
    a.x = x;
    a.scale = scale;
    a.norm_eps = norm_eps;
    a.residual = residual;
    a.k = k_in;
    return launch_gemv_args(a, dtype, st);
}

// Query, Key and Value projections of one token in one launch: RMSNorm statistic in the kernel when norm_eps >= 0
// (x = the raw residual row), biases or null, RoPE on q and k at `position` (heads of 128).
int launch_gemv_qkv(const void* wq, const void* wk, const void* wv, const void* bq, const void* bk, const void* bv,
                    const void* x, float norm_eps, int n_q, int n_kv, int k_in, int position, float theta, int dtype,
                    void* q, void* k, void* v, hipStream_t st) {
    GemvArgs a{};
    a.seg[0] = GemvSeg{wq, bq, q, n_q, 1};
    a.seg[1] = GemvSeg{wk, bk, k, n_kv, 1};
    a.seg[2] = GemvSeg{wv, bv, v, n_kv, 0};
    a.n_seg = 3;
    a.x = x;
    a.norm_eps = norm_eps;
    a.k = k_in;
    a.position = position;
    for (int i = 0; i < 64; ++i) a.inv_freq[i] = pow((double)theta, -2.0 * (double)i / 128.0);
    return launch_gemv_args(a, dtype, st);
}

}  // namespace slim
