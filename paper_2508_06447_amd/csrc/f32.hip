// The float32 layer's projections and attention (bf16 has its own kernels in gemm.hip and attn.hip).  Everything is float
// in, float accumulated and float out: v_mfma_f32_16x16x4_f32, whose products and sums are those of a float fma chain.
#include "slim_common.h"
#include <math.h>
#include <algorithm>

namespace slim {

// Four floats at any 4-byte aligned address: global_load_dwordx4 needs no more, and these entry points ask for no more.
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

// p[0..3], elements at and past `left` read as zero and are not touched.
__device__ __forceinline__ f32x4 load4(const float* p, int left) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (left >= 4) {
        v = *reinterpret_cast<const f32x4_any*>(p);
    } else if (left > 0) {
        v[0] = p[0];
        if (left > 1) v[1] = p[1];
        if (left > 2) v[2] = p[2];
    }
    return v;
}

// p[0..N-1] = v, of which only `left` are there.
template <int N> __device__ __forceinline__ void store_some(float* p, const float (&v)[N], int left) {
    typedef float any __attribute__((ext_vector_type(N == 1 ? 2 : N), aligned(4)));
    if (N > 1 && left >= N) {
        any x;
#pragma unroll
        for (int e = 0; e < N; ++e) x[e] = v[e];
        *reinterpret_cast<any*>(p) = x;
    } else {
#pragma unroll
        for (int e = 0; e < N; ++e)
            if (e < left) p[e] = v[e];
    }
}

// -------------------------------------------------------------------------------------------------
// Projections.  The float workload is small (512 rows, 128 to 688 features): what a launch costs is the chain load -> sum
// -> store of one workgroup, not the rate of the chip, so a workgroup takes 32 rows x 32 features only and its eight waves
// an eighth of the reduction each; a wave requests two 16-deep chunks (8 KB) before it waits.  The operands go from
// global memory into the registers that the matrix instruction reads: with so small tiles nothing would be read twice
// from LDS.  Which 4 of a chunk's 16 reduction elements an instruction takes is free as long as both operands agree,
// so a lane reads 16 contiguous bytes and element j of them belongs to instruction j.
//
// A tile's 32 features are two groups of 16 whose partners meet in one thread: neighbours (plain), the two halves of a
// rotation pair (rope), or the gate and up features of the same 16 outputs (SwiGLU).  RMSNorm runs inside: the rows are
// scaled by the gain on their way in, their sums of squares are taken from the same registers and 1/rms is applied to the
// finished sums.  Up to three projections share a launch.
//
// 512 rows x 256 features, k_in 256: 40.9 -> 6.2 us (688 features in: 127 -> 9.4), with tiles of 16 rows 5.3 (6.1); the
// whole layer of 512 tokens, 18 launches before and 9 now, 523 -> 50 us (four waves and four chunks 64, eight and four 71: most
// of a wave's share is then loads past its end).
// -------------------------------------------------------------------------------------------------
struct F32LinearArgs {
    F32Seg seg[3];
    int tiles_m[3], tile_end[3];         // row tiles of the segment, first tile id behind it
    int k;
    const float* gain;                   // not null: RMSNorm of the rows of a, [k]
    float eps;
    int head_dim;
    double inv_freq[64];
};

// MT groups of 16 rows, NW waves that the reduction is dealt to, G chunks of it in flight per wave.  ONCE: they are all that a wave has.
template <int MT, int NW, int G, bool ONCE = false>
__global__ void __launch_bounds__(64 * NW) f32_linear_kernel(F32LinearArgs p) {
    constexpr int MG = MT > 1 ? 2 : 1;                   // row groups that the waves take side by side behind the sum
    constexpr int EPT = 4 * MG >= NW ? 4 * MG / NW : 1;  // and elements of a tile group per thread
    __shared__ f32x4 red[NW][2 * MT][64];                // [wave][feature group * MT + row group][lane], 32 KB (MT = 1: 16)
    __shared__ float red_ss[NW][16 * MT];
    const int id = blockIdx.x, s = (id >= p.tile_end[0]) + (id >= p.tile_end[1]);
    // In the smallest launches all three segments are requested with the tile ids: an index would make theirs a second trip to the arguments.
    auto pick = [&](auto x0, auto x1, auto x2) { return s == 0 ? x0 : s == 1 ? x1 : x2; };
#define SLIM_SEG(f) (MT == 1 ? pick(p.seg[0].f, p.seg[1].f, p.seg[2].f) : p.seg[s].f)
    const F32Seg sg{SLIM_SEG(a), SLIM_SEG(lda), SLIM_SEG(m), SLIM_SEG(w0), SLIM_SEG(w1), SLIM_SEG(bias), SLIM_SEG(residual), SLIM_SEG(out),
                    SLIM_SEG(ldo), SLIM_SEG(n), SLIM_SEG(mode), SLIM_SEG(pos), SLIM_SEG(pos0)};
#undef SLIM_SEG
    const int t = MT == 1 ? id - pick(0, p.tile_end[0], p.tile_end[1]) : s ? id - p.tile_end[s - 1] : id;
    const int tiles_m = MT == 1 ? pick(p.tiles_m[0], p.tiles_m[1], p.tiles_m[2]) : p.tiles_m[s];
    const int tm = t % tiles_m, tn = t / tiles_m;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, q = lane >> 4;
    const int m0 = tm * 16 * MT, K = p.k;

    int f0, f1;                                          // first feature of the two groups
    const float* w1 = sg.w0;
    if (sg.mode == F32_ROPE) {
        const int per = p.head_dim / 32, head = tn / per;
        f0 = head * p.head_dim + (tn - head * per) * 16;
        f1 = f0 + p.head_dim / 2;
    } else if (sg.mode == F32_SWIGLU) {
        f0 = f1 = tn * 16;
        w1 = sg.w1;
    } else {
        f0 = tn * 32;
        f1 = f0 + 16;
    }
    // rows and features past the end repeat the last one: computed and never stored
    const float* pw[2] = {sg.w0 + (size_t)min(f0 + l16, sg.n - 1) * K + q * 4, w1 + (size_t)min(f1 + l16, sg.n - 1) * K + q * 4};
    const float* pa[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) pa[m] = sg.a + (size_t)min(m0 + m * 16 + l16, sg.m - 1) * sg.lda + q * 4;
    const float* pg = p.gain ? p.gain + q * 4 : nullptr;

    const int n_chunks = (K + 15) / 16, lo = (int)((long long)n_chunks * wave / NW), hi = (int)((long long)n_chunks * (wave + 1) / NW);
    const int k_end = min(K, hi * 16) - q * 4;           // elements from chunk c's on: k_end - 16 c
    f32x4 acc[2][MT];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[i][m] = f32x4{0.f, 0.f, 0.f, 0.f};
    float ss[MT] = {};
    f32x4 w[G][2], a[G][MT], g[G];
    auto load = [&](int c0) {
#pragma unroll
        for (int u = 0; u < G; ++u) {
            const int k = (c0 + u) * 16, left = k_end - k;
#pragma unroll
            for (int i = 0; i < 2; ++i) w[u][i] = load4(pw[i] + k, left);
#pragma unroll
            for (int m = 0; m < MT; ++m) a[u][m] = load4(pa[m] + k, left);
            if (pg) g[u] = load4(pg + k, left);
        }
    };
    auto multiply = [&](f32x4 (&cw)[G][2], f32x4 (&ca)[G][MT], f32x4 (&cg)[G]) {
        if (pg) {
#pragma unroll
            for (int u = 0; u < G; ++u)
#pragma unroll
                for (int m = 0; m < MT; ++m)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        ss[m] += ca[u][m][j] * ca[u][m][j];
                        ca[u][m][j] *= cg[u][j];
                    }
        }
#pragma unroll
        for (int u = 0; u < G; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int m = 0; m < MT; ++m)
                        acc[i][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(cw[u][i][j], ca[u][m][j], acc[i][m], 0, 0, 0);
    };
    if (lo < hi) load(lo);
    if (ONCE) {
        if (lo < hi) multiply(w, a, g);
    } else {
        for (int c = lo; c < hi; c += G) {
            f32x4 cw[G][2], ca[G][MT], cg[G];
#pragma unroll
            for (int u = 0; u < G; ++u) {
#pragma unroll
                for (int i = 0; i < 2; ++i) cw[u][i] = w[u][i];
#pragma unroll
                for (int m = 0; m < MT; ++m) ca[u][m] = a[u][m];
                cg[u] = g[u];
            }
            if (c + G < hi) load(c + G); // the next group flies under this one's matrix instructions
            multiply(cw, ca, cg);
        }
    }
    // Accumulator element e of lane (l16, q) in tile (i, m): feature f_i + q * 4 + e, row m0 + m * 16 + l16.
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int m = 0; m < MT; ++m) red[wave][i * MT + m][lane] = acc[i][m];
    if (pg) {
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            ss[m] += __shfl_xor(ss[m], 16, 64);
            ss[m] += __shfl_xor(ss[m], 32, 64);
            if (q == 0) red_ss[wave][m * 16 + l16] = ss[m];
        }
    }
    __syncthreads();
    // Wave v adds all waves' sums of the row groups v % MG, v % MG + MG, .., EPT elements from EPT (v / MG) on of both feature groups.
    const int e0 = wave / MG * EPT, c = q * 4 + e0;      // the thread's places in a group of 16 features
    if (NW > 4 * MG && e0 >= 4) return;                  // (said to the compiler where no wave is left over: a test that never holds costs 0.15 us)
#pragma unroll
    for (int m = wave % MG; m < MT; m += MG) {
        const int row = m0 + m * 16 + l16;
        if (row >= sg.m) continue;
        float v[2][EPT] = {};
#pragma unroll
        for (int x = 0; x < NW; ++x)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const float* part = reinterpret_cast<const float*>(&red[x][i * MT + m][lane]) + e0;
#pragma unroll
                for (int e = 0; e < EPT; ++e) v[i][e] += part[e];
            }
        if (pg) {
            float tot = 0.f;
#pragma unroll
            for (int x = 0; x < NW; ++x) tot += red_ss[x][m * 16 + l16];
            const float inv = 1.0f / sqrtf(tot / (float)K + p.eps);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int e = 0; e < EPT; ++e) v[i][e] *= inv;
        }
        float* out = sg.out + (size_t)row * sg.ldo;
        if (sg.mode == F32_SWIGLU) {
#pragma unroll
            for (int e = 0; e < EPT; ++e) v[0][e] = v[0][e] / (1.0f + expf(-v[0][e])) * v[1][e];
            store_some<EPT>(out + f0 + c, v[0], sg.n - f0 - c);
            continue;
        }
        if (sg.bias) {
#pragma unroll
            for (int e = 0; e < EPT; ++e) {
                v[0][e] += sg.bias[min(f0 + c + e, sg.n - 1)];
                v[1][e] += sg.bias[min(f1 + c + e, sg.n - 1)];
            }
        }
        if (sg.mode == F32_ROPE) {
            const double ps = (double)(sg.pos ? sg.pos[row] : sg.pos0 + row);
            const int r = f0 % p.head_dim + c;           // rotation index of e = 0
#pragma unroll
            for (int e = 0; e < EPT; ++e) {
                double sn, cs;
                sincos(ps * p.inv_freq[r + e], &sn, &cs);
                const float x1 = v[0][e], x2 = v[1][e];
                v[0][e] = x1 * (float)cs - x2 * (float)sn;
                v[1][e] = x2 * (float)cs + x1 * (float)sn;
            }
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int f = (i ? f1 : f0) + c;
            if (sg.residual) {
#pragma unroll
                for (int e = 0; e < EPT; ++e)
                    if (f + e < sg.n) v[i][e] += sg.residual[(size_t)row * sg.ldo + f + e];
            }
            store_some<EPT>(out + f, v[i], sg.n - f);
        }
    }
}

// Work items of a launch stay below 2^32: what is larger goes one segment, and then so many features and so many rows, at a time.
constexpr long long kF32TilesMax = 1ll << 23;
constexpr int kF32FeaturesMax = 1 << 27;                 // (2^23 tiles of 16; whole heads)
// From how many tiles of 32 rows on tiles of 64 are taken (of more than 32 rows): twice the flops per byte read, half the workgroups (us, tall
// and not: 2048 x 2048 from 2048 features 241 / 293, 2048 x 1024 from 512, 2048 tiles, 45 / 53; 1024 tiles fill the chip with 32 rows only).
// Four waves there: with eight the sums of 64 rows do not fit the LDS.
// Reductions of up to 64 (tall: 32) go to four (two) waves of one chunk each; more have none (us, before and so: 100000 x 16 from 16 16.6 / 5.9, 8192 x 512 from
// 64 23 / 13, 2000 x 1024 from 64 17.8 / 8.5; 16 x 100000 from 64, which were tall, 30 / 9.9).
constexpr long long kF32TallTiles = 2048;
// Up to how many tiles of 32 rows tiles of 16 are taken: a CU's four matrix pipes take 13 ns for a 16-deep chunk of 32 x 32, and half of the chip's CUs have no
// tile (us: 256 x 256 from 256 5.6 -> 5.0, from 688 8.6 -> 6.0; 100 x 1000 from 1000 11.0 -> 8.0; the layer of 512 tokens 56.6 -> 49.5).
constexpr long long kF32LowTiles = 128;

int launch_f32_linear(const F32Seg* segs, int count, int k_in, const float* gain, float eps, int head_dim, float theta, hipStream_t st) {
    F32LinearArgs p{};
    auto tiles_n = [](const F32Seg& g) { return g.mode == F32_SWIGLU ? (g.n + 15ll) / 16 : (g.n + 31ll) / 32; };
    long long small = 0, tiles = 0;
    int m_most = 0;
    for (int s = 0; s < count; ++s) {
        small += (segs[s].m + 31ll) / 32 * tiles_n(segs[s]);
        m_most = std::max(m_most, segs[s].m);
    }
    const bool tall = small >= kF32TallTiles && m_most > 32, low = small <= kF32LowTiles && m_most > 16 && k_in > 64;
    const int rows = tall ? 64 : low ? 16 : 32;
    for (int s = 0; s < 3; ++s) {
        if (s < count) {
            p.seg[s] = segs[s];
            p.tiles_m[s] = (segs[s].m + rows - 1) / rows;
            tiles += p.tiles_m[s] * tiles_n(segs[s]);
        }
        p.tile_end[s] = (int)(tiles < (1ll << 31) ? tiles : (1ll << 31) - 1);
    }
    if (tiles > kF32TilesMax) {
        for (int s = 0; s < count; ++s) {
            for (int n = 0; n < segs[s].n;) {
                F32Seg cols = segs[s];
                cols.n = std::min(kF32FeaturesMax, segs[s].n - n);
                cols.w0 += (size_t)n * k_in;
                if (cols.w1) cols.w1 += (size_t)n * k_in;
                if (cols.bias) cols.bias += n;
                if (cols.residual) cols.residual += n;
                cols.out += n;
                n += cols.n;
                const int step = (int)(kF32TilesMax / tiles_n(cols)) * rows;
                for (int m = 0; m < cols.m;) {
                    F32Seg part = cols;
                    part.m = std::min(step, cols.m - m);
                    part.a += (size_t)m * part.lda;
                    part.out += (size_t)m * part.ldo;
                    if (part.residual) part.residual += (size_t)m * part.ldo;
                    if (part.pos) part.pos += m; else part.pos0 += m;
                    const int rc = launch_f32_linear(&part, 1, k_in, gain, eps, head_dim, theta, st);
                    if (rc) return rc;
                    m += part.m;
                }
            }
        }
        return SLIM_OK;
    }
    p.k = k_in;
    p.gain = gain;
    p.eps = eps;
    p.head_dim = head_dim;
    for (int i = 0; i < head_dim / 2; ++i) p.inv_freq[i] = pow((double)theta, -2.0 * (double)i / (double)head_dim);
    if (tall && k_in <= 32) hipLaunchKernelGGL((f32_linear_kernel<4, 2, 1>), dim3((unsigned)tiles), dim3(128), 0, st, p);
    else if (tall && k_in <= 64) hipLaunchKernelGGL((f32_linear_kernel<4, 4, 1>), dim3((unsigned)tiles), dim3(256), 0, st, p);
    else if (tall) hipLaunchKernelGGL((f32_linear_kernel<4, 4, 2>), dim3((unsigned)tiles), dim3(256), 0, st, p);
    else if (k_in <= 64) hipLaunchKernelGGL((f32_linear_kernel<2, 4, 1>), dim3((unsigned)tiles), dim3(256), 0, st, p);
    else if (low && k_in <= 256) hipLaunchKernelGGL((f32_linear_kernel<1, 8, 2, true>), dim3((unsigned)tiles), dim3(512), 0, st, p);
    else if (low) hipLaunchKernelGGL((f32_linear_kernel<1, 8, 2>), dim3((unsigned)tiles), dim3(512), 0, st, p);
    else hipLaunchKernelGGL((f32_linear_kernel<2, 8, 2>), dim3((unsigned)tiles), dim3(512), 0, st, p);
    return check_launch();
}

// -------------------------------------------------------------------------------------------------
// Causal grouped-query attention.  A workgroup owns 16 queries of one head; its eight waves (four for heads of 128) take the 16-key
// tiles 0, 8, .., 1, 9, .. and so on, each with its own running (maximum, sum, values), merged through LDS at the end: the chain of key
// tiles is what a small launch takes, so it is cut in as many.
//   S^T[key, query] = K . Q^T,   O^T[d, query] = V^T . P^T
// A lane owns one query; the accumulator rows of S (keys 4 q + e) are the rows that the second product reads its P from,
// so nothing moves between lanes but the maximum and the sum.  A wave per query with the keys dealt to its lanes took
// 32.7 us for 256 queries x 4 heads of 64 (six shuffles per output element); this one 8.2.
// The second product of a tile starts from zero and is added to the running values, o = al o + ot, in place of o = al o in front of it: the same
// instructions, and a running value then takes one rounding per tile instead of sixteen.  Relative rms error against float64, 8192 keys, heads of 32 / 64 /
// 128: 6.2 / 6.2 / 8.5e-7 accumulated through, 2.6 / 2.7 / 3.5e-7 so (wave per query: 3.2 / 3.8 / 4.6e-7).
// -------------------------------------------------------------------------------------------------
constexpr int f32_attn_waves(int d) { return d > 64 ? 4 : 8; }     // (64 KB of LDS for the merge)
constexpr int kF32AttnRows = 32768;      // query tiles per plane of the grid
template <int D>
__global__ void __launch_bounds__(64 * f32_attn_waves(D)) f32_attn_kernel(const float* __restrict__ Q, const float* __restrict__ Kg, const float* __restrict__ Vg,
                                                       float* __restrict__ O, int n, int Hq, int Hkv, float scale) {
    constexpr int NW = f32_attn_waves(D);
    constexpr int C = D / 16;                            // 16-wide pieces of a head
    constexpr int LD = D + 4;
    __shared__ __align__(16) float o_part[NW][16][LD];
    __shared__ float m_part[NW][16], l_part[NW][16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, q = lane >> 4;
    const int h = blockIdx.x, g = h / (Hq / Hkv);
    // all heads of the longest query tiles first (2048 queries, 8 heads of 128: 156 us; one head after the other 206)
    const int qt = (n + 15) / 16 - 1 - (int)(blockIdx.z * kF32AttnRows + blockIdx.y);
    if (qt < 0) return;
    const int i = qt * 16 + l16;                         // the lane's query
    const size_t q_stride = (size_t)Hq * D, kv_stride = (size_t)Hkv * D;
    f32x4 qf[C];
    {
        const float* qr = Q + (size_t)min(i, n - 1) * q_stride + (size_t)h * D + q * 4;
#pragma unroll
        for (int c = 0; c < C; ++c) qf[c] = *reinterpret_cast<const f32x4_any*>(qr + c * 16);
    }
    const float* kb = Kg + (size_t)g * D + q * 4;
    const float* vb = Vg + (size_t)g * D + l16;
    f32x4 o[C];
#pragma unroll
    for (int c = 0; c < C; ++c) o[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, l_run = 0.f;
    for (int t = wave; t <= qt; t += NW) {
        // keys past the last one repeat it; they are behind every query that is stored
        f32x4 kf[C];
        const float* kr = kb + (size_t)min(t * 16 + l16, n - 1) * kv_stride;
#pragma unroll
        for (int c = 0; c < C; ++c) kf[c] = *reinterpret_cast<const f32x4_any*>(kr + c * 16);
        float vf[4][C];                                  // value of key 4 q + e, feature c * 16 + l16
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float* vr = vb + (size_t)min(t * 16 + q * 4 + e, n - 1) * kv_stride;
#pragma unroll
            for (int c = 0; c < C; ++c) vf[e][c] = vr[c * 16];
        }
        f32x4 s2[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                s2[c & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][j], qf[c][j], s2[c & 1], 0, 0, 0);
        f32x4 s;
        float mx = -INFINITY;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            s[e] = t * 16 + q * 4 + e <= i ? (s2[0][e] + s2[1][e]) * scale : -INFINITY;
            mx = fmaxf(mx, s[e]);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float mn = fmaxf(m_run, mx), al = expf(m_run - mn);   // every query has a key in every tile up to its own
        f32x4 pr;
#pragma unroll
        for (int e = 0; e < 4; ++e) pr[e] = expf(s[e] - mn);
        l_run = l_run * al + ((pr[0] + pr[1]) + (pr[2] + pr[3]));   // of the lane's keys; the four lanes of a query meet below
        m_run = mn;
        f32x4 ot[C];                                     // of this tile alone
#pragma unroll
        for (int c = 0; c < C; ++c) ot[c] = f32x4{0.f, 0.f, 0.f, 0.f};
        // On the diagonal a key of the tile may lie behind a query: its P is 0, which an infinite or undefined value would
        // turn into an undefined sum.  Such a value is a zero to the queries before it and itself to those from it on.
        bool odd = false;
        if (t == qt) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int c = 0; c < C; ++c) odd |= !(fabsf(vf[e][c]) < INFINITY);
        }
        if (__ballot(odd)) {
#pragma unroll 1
            for (int kk = 0; kk < 16; ++kk) {            // (unrolled it spills, and it is hardly ever run)
                const float pk = __shfl(kk % 4 == 0 ? pr[0] : kk % 4 == 1 ? pr[1] : kk % 4 == 2 ? pr[2] : pr[3], (kk >> 2) * 16 + l16, 64);
                const float* vr = Vg + (size_t)min(t * 16 + kk, n - 1) * kv_stride + (size_t)g * D + q * 4;
#pragma unroll
                for (int c = 0; c < C; ++c)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (t * 16 + kk <= i) ot[c][e] += pk * vr[c * 16 + e];
            }
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int c = 0; c < C; ++c) ot[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[e][c], pr[e], ot[c], 0, 0, 0);
        }
#pragma unroll
        for (int c = 0; c < C; ++c) o[c] = o[c] * al + ot[c];
    }
    l_run += __shfl_xor(l_run, 16, 64);
    l_run += __shfl_xor(l_run, 32, 64);
    // o[c][e]: feature c * 16 + q * 4 + e of the lane's query
#pragma unroll
    for (int c = 0; c < C; ++c) *reinterpret_cast<f32x4*>(&o_part[wave][l16][c * 16 + q * 4]) = o[c];
    if (q == 0) { m_part[wave][l16] = m_run; l_part[wave][l16] = l_run; }
    __syncthreads();
    constexpr int TPR = 4 * NW, DPT = D / TPR;           // threads per query, features per thread
    const int r = threadIdx.x / TPR, d0 = (threadIdx.x % TPR) * DPT, iq = qt * 16 + r;
    if (iq >= n) return;
    const int have = min(qt + 1, NW);                    // the waves behind have no tile and no maximum
    float M = m_part[0][r], l = 0.f, a[DPT] = {};
    for (int x = 1; x < have; ++x) M = fmaxf(M, m_part[x][r]);
    for (int x = 0; x < have; ++x) {
        const float wgt = expf(m_part[x][r] - M);
        l += wgt * l_part[x][r];
#pragma unroll
        for (int d = 0; d < DPT; ++d) a[d] += wgt * o_part[x][r][d0 + d];
    }
    float* dst = O + (size_t)iq * q_stride + (size_t)h * D + d0;
#pragma unroll
    for (int d = 0; d < DPT; ++d) dst[d] = a[d] / l;
}

int launch_f32_attn(const float* q, const float* k, const float* v, int n, int Hq, int Hkv, int d, float scale, float* out, hipStream_t st) {
    const int tiles = (n + 15) / 16;
    const dim3 grid(Hq, std::min(tiles, kF32AttnRows), (tiles + kF32AttnRows - 1) / kF32AttnRows);
#define SLIM_ATTN_F32(D) hipLaunchKernelGGL(f32_attn_kernel<D>, grid, dim3(64 * f32_attn_waves(D)), 0, st, q, k, v, out, n, Hq, Hkv, scale)
    switch (d) {
        case 32: SLIM_ATTN_F32(32); break;
        case 64: SLIM_ATTN_F32(64); break;
        case 128: SLIM_ATTN_F32(128); break;
        default: return SLIM_UNSUPPORTED;
    }
#undef SLIM_ATTN_F32
    return check_launch();
}

}  // namespace slim
