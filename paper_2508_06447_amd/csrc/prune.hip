// Block-wise prompt token pruning (Section 4.2): block scores (Eq. 1-2), block selection,
// hidden-state compaction.  All three are HBM-/latency-bound; none uses matrix cores.
#include "slim_common.h"
#include "routes.h"
#include "window_plan.h"
#include <algorithm>

namespace slim {

// -------------------------------------------------------------------------------------------------
// Scores.  By linearity of Eq. (2),
//   (1/Hq) sum_h q_l^h . k_rep^{g(h)}(j,m) = k_rep(j,m) . qt,   qt[g,:] = (1/Hq) sum_{h in group g} q_l^h,
// so the window query is reduced once to qt[Hkv*d] and each unit needs one dot product of length
// Hkv*d with its mean key.
// -------------------------------------------------------------------------------------------------
// 64 elements of qt per workgroup, 16 slices of the window per element (slice s takes tokens s, s+16, ..);
// the slices are summed in a fixed order through LDS, so the result is deterministic.
template <typename T>
__global__ void __launch_bounds__(1024) window_query_kernel(const T* __restrict__ q_win, int w, int Hq, int Hkv,
                                                            int d, float* __restrict__ qt) {
    __shared__ float part[16][64];
    const int le = threadIdx.x & 63, slice = threadIdx.x >> 6;
    const int e = blockIdx.x * 64 + le;                  // element of [Hkv, d]
    float acc = 0.f;
    if (e < Hkv * d) {
        const int g = e / d, c = e - g * d, G = Hq / Hkv;
        for (int t = slice; t < w; t += 16)
            for (int h = g * G; h < (g + 1) * G; ++h) acc += Elem<T>::ld(q_win + ((size_t)t * Hq + h) * d + c);
    }
    part[slice][le] = acc;
    __syncthreads();
    if (slice == 0 && e < Hkv * d) {
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) s += part[i][le];
        qt[e] = s / ((float)w * (float)Hq);              // mean over the window, then mean over heads
    }
}

// The same with 16-byte loads, for head_dim a multiple of a 16-byte chunk and aligned states: 4 chunks of qt per workgroup,
// 128 slices of the (token, head of the group) pairs per chunk, all loads of a thread independent; the slices are summed in a fixed
// order in two steps.  64 tokens, 32 / 8 heads of 128: 7.8 -> 3.5 us (2-byte loads, sixteen in a row per thread, on half as many CUs).
constexpr int kWqChunks = 4, kWqSlices = 128;
template <typename T>
__global__ void __launch_bounds__(kWqChunks * kWqSlices) window_query_vec_kernel(const T* __restrict__ q_win, int w, int Hq, int Hkv, int d,
                                                                                 float* __restrict__ qt) {
    constexpr int V = Elem<T>::kVec, EL = kWqChunks * V, NG = kWqChunks * kWqSlices / EL, PER = 4;
    __shared__ float part[kWqSlices][EL + 1];
    __shared__ float part2[NG][EL];
    const int tid = threadIdx.x, c = tid % kWqChunks, slice = tid / kWqChunks;
    const int e = (blockIdx.x * kWqChunks + c) * V;      // first of the thread's elements of [Hkv, d]
    const int G = Hq / Hkv, pairs = w * G;
    float acc[V];
#pragma unroll
    for (int i = 0; i < V; ++i) acc[i] = 0.f;
    if (e < Hkv * d) {
        const int g = e / d;
        const T* base = q_win + (size_t)g * G * d + (e - g * d);
        for (int p0 = slice; p0 < pairs; p0 += PER * kWqSlices) {
            uint4 raw[PER];
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const int p = min(p0 + u * kWqSlices, pairs - 1), t = p / G;
                raw[u] = *reinterpret_cast<const uint4*>(base + ((size_t)t * Hq + (p - t * G)) * d);
            }
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                float f[V];
                Elem<T>::unpack(raw[u], f);
                if (p0 + u * kWqSlices < pairs) {
#pragma unroll
                    for (int i = 0; i < V; ++i) acc[i] += f[i];
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < V; ++i) part[slice][c * V + i] = acc[i];
    __syncthreads();
    const int el = tid % EL, grp = tid / EL;
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < kWqSlices / NG; ++i) s += part[grp * (kWqSlices / NG) + i][el];
    part2[grp][el] = s;
    __syncthreads();
    if (grp == 0 && blockIdx.x * EL + el < Hkv * d) {
        float tot[4] = {0.f, 0.f, 0.f, 0.f};             // (one sum of 16 or 32 takes twice their error)
#pragma unroll
        for (int i = 0; i < NG; ++i) tot[i & 3] += part2[i][el];
        qt[blockIdx.x * EL + el] = ((tot[0] + tot[1]) + (tot[2] + tot[3])) / ((float)w * (float)Hq);
    }
}

// A small window is reduced by every workgroup of the scoring launch itself, which saves the launch in front of it: qs[e] as above, C chunks side by
// side and S slices (a power of two) of the (token, head of the group) pairs per chunk, C * S threads; a thread adds four pairs at a time, and everything is
// added pairwise, so that no sum is longer than that of the separate launch.  `part` holds S * E floats.  Ends with a barrier.
template <typename T>
__device__ __forceinline__ void window_query_in_lds(const T* __restrict__ q_win, int w, int Hq, int Hkv, int d, int S, float* qs, float* part) {
    constexpr int V = Elem<T>::kVec;
    const int E = Hkv * d, C = E / V, G = Hq / Hkv, pairs = w * G;
    if ((int)threadIdx.x < C * S) {
        const int slice = threadIdx.x / C, e = (threadIdx.x - slice * C) * V, g = e / d;
        const T* base = q_win + (size_t)g * G * d + (e - g * d);
        float acc[V];
#pragma unroll
        for (int v = 0; v < V; ++v) acc[v] = 0.f;
        for (int p0 = slice; p0 < pairs; p0 += 4 * S) {
            uint4 raw[4];
            float f[4][V];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int p = min(p0 + u * S, pairs - 1), t = p / G;
                raw[u] = *reinterpret_cast<const uint4*>(base + ((size_t)t * Hq + (p - t * G)) * d);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                Elem<T>::unpack(raw[u], f[u]);
                if (p0 + u * S >= pairs) {
#pragma unroll
                    for (int v = 0; v < V; ++v) f[u][v] = 0.f;
                }
            }
#pragma unroll
            for (int v = 0; v < V; ++v) acc[v] += (f[0][v] + f[1][v]) + (f[2][v] + f[3][v]);
        }
#pragma unroll
        for (int v = 0; v < V; ++v) part[(size_t)slice * E + e + v] = acc[v];
    }
    __syncthreads();
    for (; S > 4; S >>= 2) {                             // slices i, i + S/4, i + S/2, i + 3S/4 (an odd power of two: 8 -> 2)
        const int n = (S >> 2) * E;
        for (int i = threadIdx.x; i < n; i += blockDim.x) part[i] = (part[i] + part[i + n]) + (part[i + 2 * n] + part[i + 3 * n]);
        __syncthreads();
    }
    for (int e = threadIdx.x; e < E; e += blockDim.x) {
        float s = part[e];
        if (S > 1) s += part[E + e];
        if (S > 2) s += part[2 * E + e] + part[3 * E + e];
        qs[e] = s / ((float)w * (float)Hq);
    }
    __syncthreads();
}
// Whether the scoring launch reduces the window itself (16-byte chunks of one head, aligned), and with how many slices and threads.
template <typename T> static WindowPlan window_in_score(const void* q_win, int w, int Hq, int Hkv, int d, int nb, int waves, size_t key_bytes) {
    if (d % Elem<T>::kVec != 0 || !aligned16(q_win)) return {0, 64 * waves};
    return window_plan(Hkv * d, Elem<T>::kVec, w, Hq / Hkv, nb, waves, (long long)key_bytes);
}

template <typename T>
static void launch_window_query_t(const void* q_win, int w, int Hq, int Hkv, int d, float* qt, hipStream_t st) {
    const int E = Hkv * d, V = Elem<T>::kVec;
    if (d % V == 0 && aligned16(q_win))
        hipLaunchKernelGGL(window_query_vec_kernel<T>, dim3((E / V + kWqChunks - 1) / kWqChunks), dim3(kWqChunks * kWqSlices), 0, st,
                           (const T*)q_win, w, Hq, Hkv, d, qt);
    else
        hipLaunchKernelGGL(window_query_kernel<T>, dim3((E + 63) / 64), dim3(1024), 0, st, (const T*)q_win, w, Hq, Hkv, d, qt);
}

// One workgroup per block j, one wave per TokenUnit (waves stride over the units).  A wave reads its
// unit's rows in 16-byte chunks, accumulates sum_t k[t,:] . qt, divides by the unit's token count
// (Eq. 1 then the dot of Eq. 2) and the workgroup takes the max over units.  HBM-bound: eight rows of the next piece are
// requested while the last eight are summed, the first before the window query is there.  With a non-temporal hint 67 MB of keys take
// 11.4 instead of 14.3 us, but the compaction that reads them next then misses the memory-side cache: 59 against 57 us for scores,
// selection and compaction of 32768 tokens.
// A unit's rows are summed whole before the products with the window query (LONG: over several pieces of eight), so that a product takes one
// rounding: with the products of every piece added up the error of units of 64 bf16 rows was 2.3e-7 (relative rms), so it is 0.9e-7.
// R: rows of a piece.  Units of one, two and up to four rows have pieces of as many; read as eight they load a row several times (67 MB of
// bf16 keys, blocks of 64, units of 1 / 2 / 4: 29.7 / 19.6 / 16.8 us in pieces of eight, 22.4 / 15.8 / 14.7 so).
// slices > 0: qt is not there yet and the workgroup takes it from the window's w Query rows, in so many.
template <typename T, int R, bool LONG>
__global__ void __launch_bounds__(1024) block_score_kernel(const T* __restrict__ k, const float* __restrict__ qt,
                                                            int N, int E /*Hkv*d*/, int block, int unit,
                                                            float* __restrict__ scores, const T* __restrict__ q_win, int w, int Hq, int d, int slices) {
    constexpr int V = Elem<T>::kVec;
    extern __shared__ float smem[];                      // qt copy [E] + per-wave maxima [16] + slices of the window
    float* qs = smem;
    float* wmax = smem + E;
    const int j = blockIdx.x, lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b0 = j * block, b1 = min(b0 + block, N);
    const int nchunk = E / V;
    // the wave's next piece: rows t .. t + R - 1 of the unit u0 .. u1, chunks c0 + lane
    int u0 = b0 + wave * unit, u1 = min(u0 + unit, b1), t = u0, c0 = 0;
    uint4 raw[R];
    auto load = [&]() {                                  // rows and chunks past the end repeat the last one and are left out below
        const T* p = k + (size_t)min(c0 + lane, nchunk - 1) * V;
#pragma unroll
        for (int r = 0; r < R; ++r) raw[r] = *reinterpret_cast<const uint4*>(p + (size_t)min(t + r, u1 - 1) * E);
    };
    if (u0 < b1) load();
    if (slices > 0) {
        window_query_in_lds<T>(q_win, w, Hq, E / d, d, slices, qs, smem + E + 16);
    } else {
        for (int e = threadIdx.x; e < E; e += blockDim.x) qs[e] = qt[e];
        __syncthreads();
    }
    float best = -INFINITY, acc = 0.f, ksum[V];
#pragma unroll
    for (int i = 0; i < V; ++i) ksum[i] = 0.f;
    while (u0 < b1) {
        uint4 cur[R];
#pragma unroll
        for (int r = 0; r < R; ++r) cur[r] = raw[r];
        const int rows = min(R, u1 - t), c = c0 + lane, count = u1 - u0;
        t += R;
        const bool chunk_done = !LONG || t >= u1;
        if (chunk_done) { t = u0; c0 += 64; }
        const bool unit_done = c0 >= nchunk;
        if (unit_done) { c0 = 0; u0 += nw * unit; u1 = min(u0 + unit, b1); t = u0; }
        if (u0 < b1) load();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float f[V];
            Elem<T>::unpack(cur[r], f);
            if (r < rows) {
#pragma unroll
                for (int i = 0; i < V; ++i) ksum[i] += f[i];
            }
        }
        if (chunk_done) {
            if (c < nchunk) {
#pragma unroll
                for (int i = 0; i < V; ++i) acc += ksum[i] * qs[c * V + i];
            }
#pragma unroll
            for (int i = 0; i < V; ++i) ksum[i] = 0.f;
        }
        if (unit_done) {
            best = fmaxf(best, wave_sum(acc) / (float)count);
            acc = 0.f;
        }
    }
    if (lane == 0) wmax[wave] = best;
    __syncthreads();
    if (threadIdx.x == 0) {
        float m = wmax[0];
        for (int i = 1; i < nw; ++i) m = fmaxf(m, wmax[i]);
        scores[j] = m;
    }
}

// Pooled scoring, the two baselines of the scoring ablation (Table 3): one representative key per block,
// the average or the element-wise maximum of its token keys, then the same dot with qt.  One workgroup
// of 512 threads per block: thread = (token slice s, 16-byte chunk c); slices are combined through LDS in
// a fixed order, then the chunks' partial dots are summed over the workgroup.
template <typename T, bool MAXPOOL>
__global__ void __launch_bounds__(512) block_pool_score_kernel(const T* __restrict__ k, const float* __restrict__ qt,
                                                               int N, int E /*Hkv*d*/, int block,
                                                               float* __restrict__ scores) {
    constexpr int V = Elem<T>::kVec;
    extern __shared__ float smem[];                      // qt copy [E] + slice partials [512*V] + wave sums [8]
    float* qs = smem;
    float* part = smem + E;
    float* wsum = part + 512 * V;
    const int j = blockIdx.x, tid = threadIdx.x;
    for (int e = tid; e < E; e += 512) qs[e] = qt[e];
    const int b0 = j * block, b1 = min(b0 + block, N);
    const int nchunk = E / V;
    int C = 512;
    while (C > nchunk) C >>= 1;                          // chunks handled side by side: power of two <= nchunk
    const int S = 512 / C, c0 = tid % C, sl = tid / C;   // S token slices: slice sl takes tokens sl, sl+S, ..
    float dot = 0.f;
    __syncthreads();
    for (int base = 0; base < nchunk; base += C) {
        const int c = base + c0;
        float p[V];
#pragma unroll
        for (int i = 0; i < V; ++i) p[i] = MAXPOOL ? -INFINITY : 0.f;
        if (c < nchunk) {
            for (int t = b0 + sl; t < b1; t += S) {
                uint4 raw = *reinterpret_cast<const uint4*>(k + (size_t)t * E + (size_t)c * V);
                float f[V];
                Elem<T>::unpack(raw, f);
#pragma unroll
                for (int i = 0; i < V; ++i) p[i] = MAXPOOL ? fmaxf(p[i], f[i]) : p[i] + f[i];
            }
        }
        if (S > 1) {
#pragma unroll
            for (int i = 0; i < V; ++i) part[(sl * C + c0) * V + i] = p[i];
            __syncthreads();
            if (sl == 0) {
                for (int o = 1; o < S; ++o)
#pragma unroll
                    for (int i = 0; i < V; ++i) {
                        const float x = part[(o * C + c0) * V + i];
                        p[i] = MAXPOOL ? fmaxf(p[i], x) : p[i] + x;
                    }
            }
            __syncthreads();
        }
        if (sl == 0 && c < nchunk) {
#pragma unroll
            for (int i = 0; i < V; ++i) dot += p[i] * qs[c * V + i];
        }
    }
    dot = wave_sum(dot);
    if ((tid & 63) == 0) wsum[tid >> 6] = dot;
    __syncthreads();
    if (tid == 0) {
        float m = 0.f;
        for (int i = 0; i < 8; ++i) m += wsum[i];
        scores[j] = MAXPOOL ? m : m / (float)(b1 - b0);
    }
}

// pooling: 0 = TokenUnits (Eq. 1-2), 1 = average pooling, 2 = max pooling
template <typename T>
static void launch_block_score(const T* k, const void* q_win, int w, int Hq, int Hkv, int d, float* qt, int N, int block, int unit,
                               float* scores, hipStream_t st) {
    const int nb = (N + block - 1) / block, waves = std::min(16, (block + unit - 1) / unit), E = Hkv * d;
    const WindowPlan plan = window_in_score<T>(q_win, w, Hq, Hkv, d, nb, waves, (size_t)block * E * sizeof(T));
    const size_t smem = ((size_t)E * (1 + plan.slices) + 16) * sizeof(float);
    if (!plan.slices) launch_window_query_t<T>(q_win, w, Hq, Hkv, d, qt, st);
#define SLIM_SCORE(R, L) hipLaunchKernelGGL((block_score_kernel<T, R, L>), dim3(nb), dim3(plan.threads), smem, st, k, qt, N, E, block, unit, scores, \
                                            (const T*)q_win, w, Hq, d, plan.slices)
    if (unit > 8) SLIM_SCORE(8, true);
    else if (unit > 4) SLIM_SCORE(8, false);
    else if (unit > 2) SLIM_SCORE(4, false);
    else if (unit > 1) SLIM_SCORE(2, false);
    else SLIM_SCORE(1, false);
#undef SLIM_SCORE
}

template <typename T>
static void launch_score_t(const void* q_win, const void* k, int N, int w, int Hq, int Hkv, int d, int block, int unit, int pooling, float* scores,
                           float* qtilde, hipStream_t st) {
    if (pooling == 0) return launch_block_score((const T*)k, q_win, w, Hq, Hkv, d, qtilde, N, block, unit, scores, st);
    const int E = Hkv * d, nb = (N + block - 1) / block;
    const size_t smem = (size_t)(E + 512 * Elem<T>::kVec + 8) * sizeof(float);
    launch_window_query_t<T>(q_win, w, Hq, Hkv, d, qtilde, st);
    if (pooling == 1)
        hipLaunchKernelGGL((block_pool_score_kernel<T, false>), dim3(nb), dim3(512), smem, st, (const T*)k, qtilde, N, E, block, scores);
    else
        hipLaunchKernelGGL((block_pool_score_kernel<T, true>), dim3(nb), dim3(512), smem, st, (const T*)k, qtilde, N, E, block, scores);
}

int launch_score(const void* q_win, const void* k, int N, int w, int Hq, int Hkv, int d, int block, int unit,
                 int pooling, int dtype, float* scores, float* qtilde, hipStream_t st) {
    if (dtype == SLIM_BF16) launch_score_t<bf16_t>(q_win, k, N, w, Hq, Hkv, d, block, unit, pooling, scores, qtilde, st);
    else launch_score_t<float>(q_win, k, N, w, Hq, Hkv, d, block, unit, pooling, scores, qtilde, st);
    return check_launch();
}

// -------------------------------------------------------------------------------------------------
// Decode-time form of the scores (Section 4.2: during decoding the window is the most recent tokens and
// the prompt's Key states may sit in CPU memory).  Eq. (1) is evaluated once, when the keys are produced,
// and kept as k_rep[nb, M, E] in float; Eq. (2) then reads 1/unit of the bytes of the keys.
// -------------------------------------------------------------------------------------------------
// One wave per TokenUnit, 4 units per workgroup.  Units past the end of the prompt are written as zeros.
template <typename T>
__global__ void __launch_bounds__(256) unit_keys_kernel(const T* __restrict__ k, int N, int E, int block, int unit,
                                                         int M, int n_units, float* __restrict__ k_rep) {
    constexpr int V = Elem<T>::kVec;
    const int lane = threadIdx.x & 63;
    const int u = blockIdx.x * 4 + (threadIdx.x >> 6);   // unit index = j*M + m
    if (u >= n_units) return;
    const int j = u / M, m = u - j * M;
    const int b1 = min((j + 1) * block, N);
    const int u0 = j * block + m * unit, u1 = min(u0 + unit, b1);   // u1 <= u0: the unit does not exist
    const float inv = u1 > u0 ? 1.f / (float)(u1 - u0) : 0.f;
    for (int c = lane; c < E / V; c += 64) {
        float ksum[V];
#pragma unroll
        for (int i = 0; i < V; ++i) ksum[i] = 0.f;
#pragma unroll 8
        for (int t = u0; t < u1; ++t) {
            uint4 raw = *reinterpret_cast<const uint4*>(k + (size_t)t * E + (size_t)c * V);
            float f[V];
            Elem<T>::unpack(raw, f);
#pragma unroll
            for (int i = 0; i < V; ++i) ksum[i] += f[i];
        }
        float* dst = k_rep + (size_t)u * E + (size_t)c * V;
#pragma unroll
        for (int q = 0; q < V / 4; ++q)
            *reinterpret_cast<float4*>(dst + 4 * q) = make_float4(ksum[4 * q] * inv, ksum[4 * q + 1] * inv,
                                                                  ksum[4 * q + 2] * inv, ksum[4 * q + 3] * inv);
    }
}

// One workgroup per block, one wave per stored unit key: dot with qt, max over the units the block has.  OWN: the window query as in
// block_score_kernel, with the first kUnitAhead pieces of a wave's first unit key requested before it (only there: the registers cost a workgroup per
// CU, 67 MB of unit keys 15.3 -> 18.7 us).
constexpr int kUnitAhead = 4;
template <typename T, bool OWN>
__global__ void __launch_bounds__(1024) unit_score_kernel(const float* __restrict__ k_rep,
                                                           const float* __restrict__ qt, int N, int E, int block,
                                                           int unit, int M, float* __restrict__ scores, const T* __restrict__ q_win, int w, int Hq,
                                                           int d, int slices) {
    extern __shared__ float smem[];                      // qt copy [E] + per-wave maxima [16] + slices of the window
    float* qs = smem;
    float* wmax = smem + E;
    const int j = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    auto units = [&]() { return (min(block, N - j * block) + unit - 1) / unit; };      // units this block really has
    int m_have;
    float4 ahead[OWN ? kUnitAhead : 1];
    if constexpr (OWN) {
        m_have = units();
        const float* kr = k_rep + ((size_t)j * M + min(wave, m_have - 1)) * E;
#pragma unroll
        for (int u = 0; u < kUnitAhead; ++u) ahead[u] = *reinterpret_cast<const float4*>(kr + 4 * min(lane + 64 * u, E / 4 - 1));
        window_query_in_lds<T>(q_win, w, Hq, E / d, d, slices, qs, smem + E + 16);
    } else {
        for (int e = threadIdx.x; e < E; e += blockDim.x) qs[e] = qt[e];
        m_have = units();                                // (a division: behind the request for qt, not in front of it)
        __syncthreads();
    }
    float best = -INFINITY;
    for (int m = wave; m < m_have; m += nw) {
        const float* kr = k_rep + ((size_t)j * M + m) * E;
        float acc = 0.f;
        auto add = [&](int c, const float4& a) { acc += a.x * qs[4 * c] + a.y * qs[4 * c + 1] + a.z * qs[4 * c + 2] + a.w * qs[4 * c + 3]; };
        int c0 = lane;
        if constexpr (OWN) {
            if (m == wave) {
#pragma unroll
                for (int u = 0; u < kUnitAhead; ++u)
                    if (lane + 64 * u < E / 4) add(lane + 64 * u, ahead[u]);
                c0 += 64 * kUnitAhead;
            }
        }
#pragma unroll 4
        for (int c = c0; c < E / 4; c += 64) add(c, *reinterpret_cast<const float4*>(kr + 4 * c));
        best = fmaxf(best, wave_sum(acc));
    }
    if (lane == 0) wmax[wave] = best;
    __syncthreads();
    if (threadIdx.x == 0) {
        float mx = wmax[0];
        for (int i = 1; i < nw; ++i) mx = fmaxf(mx, wmax[i]);
        scores[j] = mx;
    }
}

// Block scores from per-token partial scores (the K projection's RoPE epilogue leaves, for every token and kv
// head, the dot of the token's key with that head's part of the window query).  Summing the heads gives
// k_t . qt; by linearity the mean of those over a TokenUnit is Eq. (1) dotted as in Eq. (2), and the block takes
// the maximum over its units.  One workgroup per block: a thread sums the heads of a token (16-byte loads where they divide), a thread
// per unit sums its tokens' sums through LDS and divides: fixed order.  With a thread per unit walking its unit's tokens and heads one load after the
// other (8 of 256 threads busy) the launch took 8.4 us for 512 blocks of 64; now 5.0.
constexpr int kTokScores = 2048;                         // tokens of a block at a time (whole units)
__global__ void __launch_bounds__(256) token_score_blocks_kernel(const float* __restrict__ ts, int N, int H, int block,
                                                                 int unit, float* __restrict__ scores) {
    __shared__ float tok[kTokScores];
    __shared__ float wmax[4];
    const int j = blockIdx.x, b0 = j * block, b1 = min(b0 + block, N);
    const bool vec = H % 4 == 0 && (((uintptr_t)ts) & 15) == 0;
    auto heads = [&](int t) {
        const float* p = ts + (size_t)t * H;
        float s = 0.f;
        if (vec) {
#pragma unroll 4
            for (int h = 0; h < H; h += 4) {
                const float4 v = *reinterpret_cast<const float4*>(p + h);
                s += v.x; s += v.y; s += v.z; s += v.w;
            }
        } else {
            for (int h = 0; h < H; ++h) s += p[h];
        }
        return s;
    };
    float best = -INFINITY;
    if (unit <= kTokScores) {
        const int span = kTokScores / unit * unit;
        for (int s0 = b0; s0 < b1; s0 += span) {
            const int s1 = min(s0 + span, b1);
            for (int t = s0 + threadIdx.x; t < s1; t += 256) tok[t - s0] = heads(t);
            __syncthreads();
            for (int u0 = s0 + threadIdx.x * unit; u0 < s1; u0 += 256 * unit) {
                const int u1 = min(u0 + unit, s1);
                float acc = 0.f;
                for (int t = u0; t < u1; ++t) acc += tok[t - s0];
                best = fmaxf(best, acc / (float)(u1 - u0));
            }
            __syncthreads();
        }
    } else {                                             // units longer than the LDS strip
        for (int u0 = b0 + threadIdx.x * unit; u0 < b1; u0 += 256 * unit) {
            const int u1 = min(u0 + unit, b1);
            float acc = 0.f;
            for (int t = u0; t < u1; ++t) acc += heads(t);
            best = fmaxf(best, acc / (float)(u1 - u0));
        }
    }
    best = wave_max(best);
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x == 0) scores[j] = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
}

int launch_token_score_blocks(const float* token_scores, int N, int H, int block, int unit, float* scores, hipStream_t st) {
    const int nb = (N + block - 1) / block;
    hipLaunchKernelGGL(token_score_blocks_kernel, dim3(nb), dim3(256), 0, st, token_scores, N, H, block, unit, scores);
    return check_launch();
}

int launch_window_query(const void* q_win, int w, int Hq, int Hkv, int d, int dtype, float* qtilde, hipStream_t st) {
    if (dtype == SLIM_BF16)
        launch_window_query_t<bf16_t>(q_win, w, Hq, Hkv, d, qtilde, st);
    else
        launch_window_query_t<float>(q_win, w, Hq, Hkv, d, qtilde, st);
    return check_launch();
}

int launch_unit_keys(const void* k, int N, int E, int block, int unit, int dtype, float* k_rep, hipStream_t st) {
    const int nb = (N + block - 1) / block, M = (block + unit - 1) / unit, n_units = nb * M;
    dim3 grid((n_units + 3) / 4);
    if (dtype == SLIM_BF16)
        hipLaunchKernelGGL(unit_keys_kernel<bf16_t>, grid, dim3(256), 0, st, (const bf16_t*)k, N, E, block, unit, M,
                           n_units, k_rep);
    else
        hipLaunchKernelGGL(unit_keys_kernel<float>, grid, dim3(256), 0, st, (const float*)k, N, E, block, unit, M,
                           n_units, k_rep);
    return check_launch();
}

template <typename T>
static void launch_unit_score_t(const void* q_win, const float* k_rep, int N, int w, int Hq, int Hkv, int d, int block, int unit, float* scores,
                                float* qtilde, hipStream_t st) {
    const int E = Hkv * d, nb = (N + block - 1) / block, M = (block + unit - 1) / unit, waves = std::min(16, M);
    const WindowPlan plan = window_in_score<T>(q_win, w, Hq, Hkv, d, nb, waves, 0);
    const size_t smem = ((size_t)E * (1 + plan.slices) + 16) * sizeof(float);
    if (!plan.slices) launch_window_query_t<T>(q_win, w, Hq, Hkv, d, qtilde, st);
    auto kern = plan.slices ? unit_score_kernel<T, true> : unit_score_kernel<T, false>;
    hipLaunchKernelGGL(kern, dim3(nb), dim3(plan.threads), smem, st, k_rep, qtilde, N, E, block, unit, M, scores, (const T*)q_win, w, Hq, d,
                       plan.slices);
}

int launch_score_from_unit_keys(const void* q_win, const float* k_rep, int N, int w, int Hq, int Hkv, int d,
                                int block, int unit, int dtype, float* scores, float* qtilde, hipStream_t st) {
    if (dtype == SLIM_BF16) launch_unit_score_t<bf16_t>(q_win, k_rep, N, w, Hq, Hkv, d, block, unit, scores, qtilde, st);
    else launch_unit_score_t<float>(q_win, k_rep, N, w, Hq, Hkv, d, block, unit, scores, qtilde, st);
    return check_launch();
}

// -------------------------------------------------------------------------------------------------
// Selection: one workgroup.  An 8-bit-digit radix select over order-preserving integer keys finds
// the score of the last block to take; equal scores are taken in ascending index order; the kept
// set is written ascending through a prefix sum of the keep flags.  Integer work only, so the
// result does not depend on the order in which threads run.
// -------------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t score_key(float s) {
    uint32_t b = __builtin_bit_cast(uint32_t, s);
    if ((b << 1) == 0) b = 0;                            // -0.0 == +0.0
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);   // ascending in the float order
}

constexpr int kSelThreads = 1024;

// Exclusive prefix sum of one int per thread across the workgroup; returns the total in `total`.
__device__ int block_exclusive_scan(int v, int* wsum /*[16]*/, int& total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        int t = __shfl_up(inc, o, 64);
        if (lane >= o) inc += t;
    }
    __syncthreads();                                     // wsum free from the previous use
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    int base = 0, tot = 0;
    for (int i = 0; i < kSelThreads / 64; ++i) {
        int s = wsum[i];
        if (i < wave) base += s;
        tot += s;
    }
    total = tot;
    return base + inc - v;
}

__global__ void __launch_bounds__(kSelThreads) select_blocks_kernel(const float* __restrict__ scores, int nb,
                                                                     int n_keep, unsigned flags,
                                                                     int* __restrict__ kept) {
    __shared__ int hist[256];
    __shared__ int wsum[kSelThreads / 64];
    __shared__ uint32_t s_prefix;
    __shared__ int s_remaining;
    const int tid = threadIdx.x;
    const bool f_first = flags & SLIM_FORCE_FIRST, f_last = flags & SLIM_FORCE_LAST;
    auto forced = [&](int j) { return (f_first && j == 0) || (f_last && j == nb - 1); };
    const int n_forced = (f_first ? 1 : 0) + ((f_last && !(f_first && nb == 1)) ? 1 : 0);
    const int take = n_keep - n_forced;                  // > 0 slots for the non-forced blocks, < nb - n_forced

    uint32_t thr = 0;                                    // key of the last block taken
    int n_eq = 0;                                        // how many blocks with that exact key to take
    if (take > 0) {
        if (tid == 0) { s_prefix = 0; s_remaining = take; }
        for (int pass = 0; pass < 4; ++pass) {
            const int shift = 24 - 8 * pass;
            const uint32_t himask = pass == 0 ? 0u : (0xffffffffu << (shift + 8));
            if (tid < 256) hist[tid] = 0;
            __syncthreads();
            const uint32_t prefix = s_prefix;
            for (int j = tid; j < nb; j += kSelThreads) {
                if (forced(j)) continue;
                uint32_t key = score_key(scores[j]);
                if ((key & himask) == prefix) atomicAdd(&hist[(key >> shift) & 255], 1);
            }
            __syncthreads();
            if (tid < 64) {
                // Find the digit that holds the rem-th largest candidate: lane l owns the digits
                // 255-4l .. 252-4l (descending); a wave scan gives the count of larger digits.
                const int rem = s_remaining;
                int c[4], tot = 0;
#pragma unroll
                for (int k = 0; k < 4; ++k) { c[k] = hist[255 - (4 * tid + k)]; tot += c[k]; }
                int inc = tot;
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const int t = __shfl_up(inc, o, 64);
                    if (tid >= o) inc += t;
                }
                int above = inc - tot;                   // candidates with a larger digit than this lane's first
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (above < rem && rem <= above + c[k]) {          // true for exactly one (lane, k)
                        s_prefix = prefix | ((uint32_t)(255 - (4 * tid + k)) << shift);
                        s_remaining = rem - above;
                    }
                    above += c[k];
                }
            }
            __syncthreads();
        }
        thr = s_prefix;
        n_eq = s_remaining;
    }

    int eq_seen = 0, out_base = 0;
    for (int base = 0; base < nb; base += kSelThreads) {
        const int j = base + tid;
        bool in = j < nb, fz = in && forced(j);
        uint32_t key = (in && !fz && take > 0) ? score_key(scores[j]) : 0;
        int is_eq = (in && !fz && take > 0 && key == thr) ? 1 : 0;
        int tot_eq;
        int eq_rank = block_exclusive_scan(is_eq, wsum, tot_eq) + eq_seen;
        int keep = fz || (in && !fz && take > 0 && (key > thr || (is_eq && eq_rank < n_eq)));
        int tot_keep;
        int slot = block_exclusive_scan(keep, wsum, tot_keep) + out_base;
        if (keep) kept[slot] = j;
        eq_seen += tot_eq;
        out_base += tot_keep;
    }
}

constexpr int kSelSmall = 256;
// Inclusive prefix sum over the wave's lanes, in the vector ALU (a shuffle goes through LDS: six of them in a row took longer than the rest of
// a digit).
__device__ __forceinline__ int wave_inclusive_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);            // row_shr:1, 2, 4, 8 inside 16 lanes
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);            // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);            // row_bcast:31 into rows 2 and 3
    return v;
}
// The same selection for up to 256 * KPT blocks: four waves instead of sixteen, the keys read once and kept in registers (thread t
// holds KPT consecutive ones), a histogram per digit so that a pass takes two barriers, no further digits once all candidates with the last one are
// taken, one prefix sum, and a second one over equal scores only when not all of them are taken.  512 blocks 5.7 us at first, 4.7 with that,
// 4.1 with the prefix sums in the vector ALU and the early end (2048 blocks 7.7 -> 5.8): what is left is the launch and the scores' way from the L2.
template <int KPT>
__global__ void __launch_bounds__(kSelSmall) select_few_blocks_kernel(const float* __restrict__ scores, int nb, int n_keep,
                                                                      unsigned flags, int* __restrict__ kept) {
    __shared__ int hist[4][256];
    __shared__ int wsum[2][kSelSmall / 64];
    __shared__ uint32_t s_prefix[4];
    __shared__ int s_remaining[4], s_all[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, j0 = tid * KPT;
    const bool f_first = flags & SLIM_FORCE_FIRST, f_last = flags & SLIM_FORCE_LAST;
    auto forced = [&](int j) { return (f_first && j == 0) || (f_last && j == nb - 1); };
    const int n_forced = (f_first ? 1 : 0) + ((f_last && !(f_first && nb == 1)) ? 1 : 0);
    const int take = n_keep - n_forced;                  // > 0 slots for the non-forced blocks, < nb - n_forced
    uint32_t key[KPT];
    unsigned open = 0, fz = 0;                           // bit i: block j0 + i is a candidate; is forced
#pragma unroll
    for (int i = 0; i < KPT; ++i) {
        key[i] = score_key(scores[min(j0 + i, nb - 1)]);
        if (j0 + i < nb) (forced(j0 + i) ? fz : open) |= 1u << i;
    }
    if (take <= 0) open = 0;
#pragma unroll
    for (int p = 0; p < 4; ++p) hist[p][tid] = 0;
    __syncthreads();
    uint32_t prefix = 0;
    int remaining = take;
    bool all = false;                                    // every candidate from `prefix` up is taken: no further digit matters
    if (take > 0) {
#pragma unroll
        for (int pass = 0; pass < 4; ++pass) {
            const int shift = 24 - 8 * pass;
            const uint32_t himask = pass == 0 ? 0u : (0xffffffffu << ((shift + 8) & 31));
#pragma unroll
            for (int i = 0; i < KPT; ++i)
                if ((open >> i & 1) && (key[i] & himask) == prefix) atomicAdd(&hist[pass][(key[i] >> shift) & 255], 1);
            __syncthreads();
            if (wave == 0) {
                // Find the digit that holds the remaining-th largest candidate: lane l owns the digits
                // 255-4l .. 252-4l (descending); a wave scan gives the count of larger digits.
                int c[4], tot = 0;
#pragma unroll
                for (int k = 0; k < 4; ++k) { c[k] = hist[pass][255 - (4 * lane + k)]; tot += c[k]; }
                const int inc = wave_inclusive_scan(tot);
                int above = inc - tot;                   // candidates with a larger digit than this lane's first
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (above < remaining && remaining <= above + c[k]) {      // true for exactly one (lane, k)
                        s_prefix[pass] = prefix | ((uint32_t)(255 - (4 * lane + k)) << shift);
                        s_remaining[pass] = remaining - above;
                        s_all[pass] = remaining - above == c[k];
                    }
                    above += c[k];
                }
            }
            __syncthreads();
            prefix = s_prefix[pass];
            remaining = s_remaining[pass];
            all = s_all[pass];
            if (all) break;
        }
    }
    // Exclusive prefix sum of one number per thread; `buf` is used once per buffer.
    auto scan = [&](int v, int buf) {
        const int inc = wave_inclusive_scan(v);
        if (lane == 63) wsum[buf][wave] = inc;
        __syncthreads();
        int base = 0;
#pragma unroll
        for (int i = 0; i < kSelSmall / 64; ++i) base += i < wave ? wsum[buf][i] : 0;
        return base + inc - v;
    };
    unsigned keep = fz, eq = 0;
#pragma unroll
    for (int i = 0; i < KPT; ++i) {
        if ((open >> i & 1) && (key[i] > prefix || (all && key[i] == prefix))) keep |= 1u << i;
        if ((open >> i & 1) && key[i] == prefix && !all) eq |= 1u << i;
    }
    if (take > 0 && !all) {                            // equal scores in ascending index order, `remaining` of them
        int rank = scan(__popc(eq), 0);
#pragma unroll
        for (int i = 0; i < KPT; ++i)
            if (eq >> i & 1) {
                if (rank >= remaining) eq &= ~(1u << i);
                ++rank;
            }
    }
    keep |= eq;
    int slot = scan(__popc(keep), 1);
#pragma unroll
    for (int i = 0; i < KPT; ++i)
        if (keep >> i & 1) kept[slot++] = j0 + i;
}

__global__ void iota_kernel(int* out, int n) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = i;
}

__global__ void positions_kernel(const int* __restrict__ pos_in, int* __restrict__ pos_out, int n) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) pos_out[i] = pos_in ? pos_in[i] : i;
}

int launch_positions(const int* pos_in, int* pos_out, int n, hipStream_t st) {
    hipLaunchKernelGGL(positions_kernel, dim3((n + 255) / 256), dim3(256), 0, st, pos_in, pos_out, n);
    return check_launch();
}

// A float32 layer that drops nothing: kept = 0 .. nb - 1 and the positions as they came in, either may be null.  (In bf16 layers the pass over the rows
// writes them.)
__global__ void keep_all_kernel(int* __restrict__ kept, int nb, const int* __restrict__ pos_in, int* __restrict__ pos_out, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (kept && i < nb) kept[i] = i;
    if (pos_out && i < n) pos_out[i] = pos_in ? pos_in[i] : i;
}

int launch_keep_all(int* kept, int nb, const int* pos_in, int* pos_out, int n, hipStream_t st) {
    if (!kept && !pos_out) return SLIM_OK;
    hipLaunchKernelGGL(keep_all_kernel, dim3((std::max(n, nb) + 255) / 256), dim3(256), 0, st, kept, nb, pos_in, pos_out, n);
    return check_launch();
}

int launch_select(const float* scores, int nb, int n_keep, unsigned flags, int* kept, hipStream_t st) {
    if (n_keep >= nb) {
        hipLaunchKernelGGL(iota_kernel, dim3((nb + 255) / 256), dim3(256), 0, st, kept, nb);
    } else {
        if (nb <= kSelSmall * 4)
            hipLaunchKernelGGL(select_few_blocks_kernel<4>, dim3(1), dim3(kSelSmall), 0, st, scores, nb, n_keep, flags, kept);
        else if (nb <= kSelSmall * 16)
            hipLaunchKernelGGL(select_few_blocks_kernel<16>, dim3(1), dim3(kSelSmall), 0, st, scores, nb, n_keep, flags, kept);
        else
            hipLaunchKernelGGL(select_blocks_kernel, dim3(1), dim3(kSelThreads), 0, st, scores, nb, n_keep, flags, kept);
    }
    return check_launch();
}

// -------------------------------------------------------------------------------------------------
// Compaction: a kept block is one contiguous run of block*row bytes in src and in dst, so the gather
// is a segmented copy.  grid = (chunks per block, kept blocks); each thread moves copy_vecs<V>() vectors, past the caches.
// One 16-byte vector each: 81 MB of rows 26.7 us (6.0 TB/s), two 27.5, four 28.6, eight 41.5; without the non-temporal store 28.8 to 43.
// Of the narrow vectors of other rows four each, for more bytes in flight: 22 MB of rows of 1026 (4-byte vectors) or 1025 (2-byte)
// bf16 15.5 and 25.6 us with one, 10.6 and 17.7 with four.
// -------------------------------------------------------------------------------------------------
constexpr int kCopyThreads = 256;
constexpr int kCopyVecs = 1;                             // 16-byte ones
template <typename V> constexpr int copy_vecs() { return sizeof(V) == 16 ? kCopyVecs : 4; }
constexpr size_t kCopyChunks = 1 << 23;                  // workgroups per kept block in one plane of the grid (work items per dimension stay below 2^32)

template <typename V>
__global__ void __launch_bounds__(kCopyThreads) compact_kernel(const V* __restrict__ src, V* __restrict__ dst,
                                                               const int* __restrict__ kept, int block, int N,
                                                               int nb, size_t row_vecs,
                                                               const int* __restrict__ pos_in,
                                                               int* __restrict__ pos_out) {
    constexpr int VECS = copy_vecs<V>();
    const int i = blockIdx.y;
    const int kb = kept[i];
    if ((unsigned)kb >= (unsigned)nb) return;
    const int rows = min(block, N - kb * block);
    const size_t seg = (size_t)rows * row_vecs;
    const V* s = src + (size_t)kb * block * row_vecs;
    V* d = dst + (size_t)i * block * row_vecs;
    const size_t base = (blockIdx.x + blockIdx.z * kCopyChunks) * (kCopyThreads * VECS) + threadIdx.x;
    V tmp[VECS];
#pragma unroll
    for (int u = 0; u < VECS; ++u) {
        size_t o = base + (size_t)u * kCopyThreads;
        if (o < seg) tmp[u] = __builtin_nontemporal_load(s + o);
    }
#pragma unroll
    for (int u = 0; u < VECS; ++u) {
        size_t o = base + (size_t)u * kCopyThreads;
        if (o < seg) __builtin_nontemporal_store(tmp[u], d + o);
    }
    if (blockIdx.x == 0 && blockIdx.z == 0 && pos_out) {
        for (int r = threadIdx.x; r < rows; r += kCopyThreads) {
            int t = kb * block + r;
            pos_out[(size_t)i * block + r] = pos_in ? pos_in[t] : t;
        }
    }
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

int launch_compact(const void* src, const int* pos_in, const int* kept, int n_keep, int block, int N,
                   int row_elems, int dtype, void* dst, int* pos_out, hipStream_t st) {
    const size_t row_bytes = (size_t)row_elems * elem_size(dtype);
    const int nb = (N + block - 1) / block;
    const size_t rows = std::min(block, N);   // (a block may be longer than all there is)
#define SLIM_COMPACT(V) do { \
        const size_t rv = row_bytes / sizeof(V), per = kCopyThreads * copy_vecs<V>(), chunks = (rows * rv + per - 1) / per; \
        const dim3 grid((unsigned)std::min(kCopyChunks, chunks), n_keep, (unsigned)((chunks + kCopyChunks - 1) / kCopyChunks)); \
        hipLaunchKernelGGL(compact_kernel<V>, grid, dim3(kCopyThreads), 0, st, \
                           (const V*)src, (V*)dst, kept, block, N, nb, rv, pos_in, pos_out); } while (0)
    if (row_bytes % 16 == 0 && aligned16(src) && aligned16(dst)) SLIM_COMPACT(u32x4);
    else if (row_bytes % 4 == 0) SLIM_COMPACT(uint32_t);
    else SLIM_COMPACT(uint16_t);
#undef SLIM_COMPACT
    return check_launch();
}

// Several arrays compacted by the same kept set in one launch (hidden rows + positions, keys, row statistics):
// grid = (chunks of all arrays' block runs, kept blocks).  Rows are multiples of 4 bytes; a run is
// moved in 16-byte vectors when it allows, else in words.
struct CompactSegs {
    const unsigned char* src[4];
    unsigned char* dst[4];
    unsigned long long row_bytes[4];
    unsigned chunk_end[4];               // first chunk of the grid behind the array's
};

// Block i of the n_keep that select_few_blocks_kernel keeps of nb <= 64, found by every wave by itself: lane j ranks block j among those that are not forced.
__device__ __forceinline__ int kept_of_wave(const float* __restrict__ scores, int nb, int n_keep, unsigned flags, int i) {
    const int j = threadIdx.x & 63;
    const bool f_first = flags & SLIM_FORCE_FIRST, f_last = flags & SLIM_FORCE_LAST;
    const bool forced = (f_first && j == 0) || (f_last && j == nb - 1), open = j < nb && !forced;
    const int take = n_keep - ((f_first ? 1 : 0) + ((f_last && !(f_first && nb == 1)) ? 1 : 0));
    const uint32_t key = score_key(scores[min(j, nb - 1)]);
    int rank = 0;                                        // candidates in front of block j: larger scores, and equal ones with a smaller index
    for (int b = f_first ? 1 : 0; b < nb - (f_last ? 1 : 0); ++b) {
        const uint32_t other = __builtin_amdgcn_readlane(key, b);
        rank += other > key || (other == key && b < j);
    }
    const bool keep = (j < nb && forced) || (open && rank < take);
    const unsigned long long mask = __ballot(keep);
    const bool mine = keep && __popcll(mask & ((1ull << j) - 1)) == i;
    return __ffsll(__ballot(mine)) - 1;
}

// SELECT: kept is written, from the scores, in place of being read.
template <bool SELECT>
__global__ void __launch_bounds__(kCopyThreads) compact_multi_kernel(CompactSegs segs, int* __restrict__ kept,
                                                                     int block, int N, int nb,
                                                                     const int* __restrict__ pos_in,
                                                                     int* __restrict__ pos_out, const float* __restrict__ scores, unsigned flags) {
    const int i = blockIdx.y;
    const int a = (blockIdx.x >= segs.chunk_end[0]) + (blockIdx.x >= segs.chunk_end[1]) + (blockIdx.x >= segs.chunk_end[2]);
    const unsigned first = a ? segs.chunk_end[a - 1] : 0, chunk = blockIdx.x - first;
    const int kb = SELECT ? kept_of_wave(scores, nb, gridDim.y, flags, i) : kept[i];
    if ((unsigned)kb >= (unsigned)nb) return;
    if (SELECT && blockIdx.x == 0 && threadIdx.x == 0) kept[i] = kb;
    const int rows = min(block, N - kb * block);
    const size_t rb = segs.row_bytes[a];
    const size_t run = (size_t)rows * rb;
    const unsigned char* s = segs.src[a] + (size_t)kb * block * rb;
    unsigned char* d = segs.dst[a] + (size_t)i * block * rb;
    if (((rb * block) % 16 == 0) && (run % 16 == 0) && ((((uintptr_t)segs.src[a]) | ((uintptr_t)segs.dst[a])) & 15) == 0) {
        const u32x4* sv = reinterpret_cast<const u32x4*>(s);
        u32x4* dv = reinterpret_cast<u32x4*>(d);
        const size_t seg = run / 16;
        const size_t base = (size_t)chunk * (kCopyThreads * kCopyVecs) + threadIdx.x;
        u32x4 tmp[kCopyVecs];
#pragma unroll
        for (int u = 0; u < kCopyVecs; ++u) {
            const size_t o = base + (size_t)u * kCopyThreads;
            if (o < seg) tmp[u] = __builtin_nontemporal_load(sv + o);
        }
#pragma unroll
        for (int u = 0; u < kCopyVecs; ++u) {
            const size_t o = base + (size_t)u * kCopyThreads;
            if (o < seg) __builtin_nontemporal_store(tmp[u], dv + o);
        }
    } else {
        const uint32_t* sw = reinterpret_cast<const uint32_t*>(s);
        uint32_t* dw = reinterpret_cast<uint32_t*>(d);
        const size_t seg = run / 4;
        for (size_t o = (size_t)chunk * kCopyThreads + threadIdx.x; o < seg; o += (size_t)(segs.chunk_end[a] - first) * kCopyThreads)
            dw[o] = sw[o];
    }
    if (blockIdx.x == 0 && pos_out) {
        for (int r = threadIdx.x; r < rows; r += kCopyThreads) {
            const int t = kb * block + r;
            pos_out[(size_t)i * block + r] = pos_in ? pos_in[t] : t;
        }
    }
}

static size_t compact_chunks(size_t block, size_t row_bytes) {
    constexpr size_t per = (size_t)kCopyThreads * kCopyVecs * 16;
    return (block * row_bytes + per - 1) / per;
}

bool compact_selects(int n_arrays, const size_t* row_bytes, int block, int n_keep, int nb) {
    size_t chunks = 0;
    for (int a = 0; a < n_arrays; ++a) chunks += compact_chunks(block, row_bytes[a]);
    return compact_selects((long long)chunks, n_keep, nb);
}

// Up to 4 arrays [N, row_bytes[a]] -> [n', row_bytes[a]]; positions ride with array 0.  row_bytes % 4 == 0.  With scores the launch selects the blocks itself
// (launch_select, 64 blocks at most, n_keep < nb).
int launch_compact_multi(int n_arrays, const void* const* src, void* const* dst, const size_t* row_bytes, const int* pos_in,
                         int* pos_out, int* kept, int n_keep, int block, int N, hipStream_t st, const float* scores, unsigned flags) {
    CompactSegs segs;
    size_t chunks = 0;
    for (int a = 0; a < 4; ++a) {
        const bool on = a < n_arrays;
        segs.src[a] = on ? (const unsigned char*)src[a] : nullptr;
        segs.dst[a] = on ? (unsigned char*)dst[a] : nullptr;
        segs.row_bytes[a] = on ? row_bytes[a] : 0;
        if (on) chunks += compact_chunks(block, row_bytes[a]);
        segs.chunk_end[a] = (unsigned)chunks;
    }
    const int nb = (N + block - 1) / block;
    hipLaunchKernelGGL(scores ? compact_multi_kernel<true> : compact_multi_kernel<false>, dim3((unsigned)chunks, n_keep), dim3(kCopyThreads), 0, st, segs, kept,
                       block, N, nb, pos_in, pos_out, scores, flags);
    return check_launch();
}

}  // namespace slim
