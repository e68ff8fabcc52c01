// Decode-step attention over the active blocks (Section 4.1: only active blocks take part in attention and have
// their KV in GPU memory; every response token is retained).  One new token's Query states attend to the prompt
// tokens of the blocks that currently sit in the GPU slot pool -- read through block_of_slot, wherever the KV swap
// (Algorithm 1) has put them -- and to all response tokens.  HBM-bound: every resident key and value is read once.
//
// Split over the keys: the 16-key groups of the slots and of the response are dealt to the waves of up to
// kDecWgs / Hkv workgroups per kv head, each of which leaves a partial (max, sum, weighted values) for the query
// heads of that kv head; a second kernel merges the partials.  Softmax is order-independent, so the slot order does
// not matter.
#include "slim_common.h"
#include <algorithm>
#include <type_traits>

namespace slim {

constexpr int DD = 128;          // head_dim
constexpr int DGK = 16;          // keys per group
constexpr int DGMAX = 8;         // query heads per kv head
constexpr int DPART = DD + 2;    // floats of a partial: values, max (base-2 domain), sum

// Value of lane H of the caller's row of 16 lanes.
template <int H> __device__ __forceinline__ float row_lane(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x150 + H, 0xf, 0xf, true));
}
// Maximum over the four lanes with the same lane % 16.
__device__ __forceinline__ float max_over_rows(float v) {
    const unsigned x = __builtin_bit_cast(unsigned, v);
    const auto a = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    const float m = fmaxf(__builtin_bit_cast(float, a[0]), __builtin_bit_cast(float, a[1]));
    const unsigned y = __builtin_bit_cast(unsigned, m);
    const auto b = __builtin_amdgcn_permlane32_swap(y, y, false, false);
    return fmaxf(__builtin_bit_cast(float, b[0]), __builtin_bit_cast(float, b[1]));
}
template <int G, int H = 0, typename F> __device__ __forceinline__ void for_heads(F f) {
    if constexpr (H < G) {
        f(std::integral_constant<int, H>{});
        for_heads<G, H + 1>(f);
    }
}

// Lane (l16, q) = (lane % 16, lane / 16).
//   S[key, head] = K . Q^T by 16-row matrix instructions: the lane supplies 16-byte pieces of key l16 and of query head l16 (heads
//   past G repeat the last one and are ignored) and holds, for head l16, the logits of keys 4 q .. 4 q + 3: the maximum
//   of a group takes two exchanges, the sum none until the end.
//   O += P V by the vector ALU: the lane loads 16-byte pieces of the value rows of the same keys 4 q + e, 8 features of each, and
//   takes P of head h from lane h of its row of 16.
// The registers of a piece are requested anew as soon as it is used; the slot of the group after that is looked up meanwhile.
template <typename T, int G>
__global__ void __launch_bounds__(256) decode_attn_partial_kernel(
    const T* __restrict__ q, const unsigned char* __restrict__ pool, size_t slot_bytes, size_t layer_offset,
    const int* __restrict__ block_of_slot, int n_slots, int block, int n_prompt, const T* __restrict__ k_resp,
    const T* __restrict__ v_resp, int n_resp, int Hq, int Hkv, float scale_log2e, float* __restrict__ part) {
    constexpr int V = Elem<T>::kVec, NK = DD / (4 * V), NV = 8 / V;   // pieces of a key per lane; of a value row per lane
    __shared__ float red[4][2][G][DD];                   // per wave and half of its lanes: weighted values
    __shared__ float ws_m[4][G], ws_l[4][G];             // per wave: maximum and sum
    const int g = blockIdx.y, tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, qr = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const size_t row_stride = (size_t)Hkv * DD;
    const int nb = (n_prompt + block - 1) / block, per_slot = (block + DGK - 1) / DGK;
    const int n_in_slots = n_slots * per_slot, n_groups = n_in_slots + (n_resp + DGK - 1) / DGK;
    const int step = gridDim.x * 4;

    // The wave's groups are gi, gi + step, ..; those of a free slot and past the end of a short block hold no key and are passed
    // over.  All of this is wave-uniform.
    int gi = (int)blockIdx.x * 4 + wave, rows = 0;
    const T *kp = nullptr, *vp = nullptr;                // first Key and Value row of the group, kv head g
    auto find = [&]() {                                  // from gi on; false: none is left
        for (; gi < n_groups; gi += step) {
            if (gi < n_in_slots) {
                const int slot = gi / per_slot, c0 = (gi - slot * per_slot) * DGK, b = block_of_slot[slot];
                if (b < 0 || b >= nb) continue;
                const int r = min(DGK, min(block, n_prompt - b * block) - c0);
                if (r <= 0) continue;
                rows = r;                                // (only of a group that is taken: the last one may be requested again)
                kp = reinterpret_cast<const T*>(pool + (size_t)slot * slot_bytes + layer_offset) + (size_t)c0 * row_stride + (size_t)g * DD;
                vp = kp + (size_t)block * row_stride;
            } else {
                const int c0 = (gi - n_in_slots) * DGK;
                rows = min(DGK, n_resp - c0);
                kp = k_resp + (size_t)c0 * row_stride + (size_t)g * DD;
                vp = v_resp + (size_t)c0 * row_stride + (size_t)g * DD;
            }
            return true;
        }
        return false;
    };
    uint4 kx[NK], vx[4][NV];
    // Rows past the end repeat the last one: their P is 0.  Addresses are a wave-uniform base and a 32-bit offset of the lane.
    const unsigned stride = (unsigned)(row_stride * sizeof(T));
    auto load_k = [&]() {
        const unsigned off = (unsigned)min(l16, rows - 1) * stride + qr * 16;
#pragma unroll
        for (int c = 0; c < NK; ++c) kx[c] = load_stream16(reinterpret_cast<const unsigned char*>(kp) + off + c * 64);
    };
    auto load_v = [&]() {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const unsigned off = (unsigned)min(qr * 4 + e, rows - 1) * stride + l16 * 16;
#pragma unroll
            for (int c = 0; c < NV; ++c) vx[e][c] = load_stream16(reinterpret_cast<const unsigned char*>(vp) + off + c * 256);
        }
    };
    bool more = find();
    if (more) { load_k(); load_v(); }
    uint4 qx[NK];
    {
        const T* qp = q + (size_t)(g * G + min(l16, G - 1)) * DD + qr * V;
#pragma unroll
        for (int c = 0; c < NK; ++c) qx[c] = *reinterpret_cast<const uint4*>(qp + c * 4 * V);
    }
    float m_run = -INFINITY, l_run = 0.f, o[G][8];       // of head l16 (the sum: of the lane's own keys); of the lane's 8 features
#pragma unroll
    for (int h = 0; h < G; ++h)
#pragma unroll
        for (int i = 0; i < 8; ++i) o[h][i] = 0.f;

    while (more) {
        const int have = rows;
        gi += step;
        more = find();                                   // none left: the last group is requested once more, and not used
        f32x4 s = {0.f, 0.f, 0.f, 0.f}, sp[NK];    // (float32: eight sums of 16 products, half the error of one of 128)
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            if constexpr (sizeof(T) == 2) {
                s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kx[c]), __builtin_bit_cast(bf16x8, qx[c]), s, 0, 0, 0);
            } else {
                const f32x4 a = __builtin_bit_cast(f32x4, kx[c]), b = __builtin_bit_cast(f32x4, qx[c]);
#pragma unroll
                for (int j = 0; j < 4; ++j) sp[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], b[j], j ? sp[c] : s, 0, 0, 0);
            }
        }
        if constexpr (sizeof(T) == 4) s = ((sp[0] + sp[1]) + (sp[2] + sp[3])) + ((sp[4] + sp[5]) + (sp[6] + sp[7]));
        __builtin_amdgcn_sched_barrier(0);
        load_k();                                        // the next group's keys fly under this one's values
        float mx = -INFINITY;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            s[e] = qr * 4 + e < have ? s[e] * scale_log2e : -INFINITY;
            mx = fmaxf(mx, s[e]);
        }
        const float mn = fmaxf(m_run, max_over_rows(mx)), al = __builtin_amdgcn_exp2f(m_run - mn);   // finite: the group has a key
        float p[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) p[e] = __builtin_amdgcn_exp2f(s[e] - mn);
        l_run = l_run * al + ((p[0] + p[1]) + (p[2] + p[3]));
        m_run = mn;
        for_heads<G>([&](auto h) {
            const float a = row_lane<h.value>(al);
#pragma unroll
            for (int i = 0; i < 8; ++i) o[h.value][i] *= a;
        });
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            __builtin_amdgcn_sched_barrier(0);           // (left alone, the four values and all P of a head are unpacked at once: spills)
            float f[8];
#pragma unroll
            for (int c = 0; c < NV; ++c) Elem<T>::unpack(vx[e][c], f + c * V);
            for_heads<G>([&](auto h) {
                const float ph = row_lane<h.value>(p[e]);
#pragma unroll
                for (int i = 0; i < 8; ++i) o[h.value][i] += ph * f[i];
            });
        }
        __builtin_amdgcn_sched_barrier(0);
        load_v();
    }
    // ---- the lanes' and then the four waves' states are merged, and the partial is written
    l_run += __shfl_xor(l_run, 16, 64);
    l_run += __shfl_xor(l_run, 32, 64);
    if (lane < G) { ws_m[wave][lane] = m_run; ws_l[wave][lane] = l_run; }
#pragma unroll
    for (int h = 0; h < G; ++h) {
#pragma unroll
        for (int i = 0; i < 8; ++i) o[h][i] += __shfl_xor(o[h][i], 32, 64);
        if (lane < 32) {
#pragma unroll
            for (int c = 0; c < NV; ++c)
#pragma unroll
                for (int i = 0; i < V; i += 4)
                    *reinterpret_cast<f32x4*>(&red[wave][qr][h][c * 16 * V + l16 * V + i]) =
                        f32x4{o[h][c * V + i], o[h][c * V + i + 1], o[h][c * V + i + 2], o[h][c * V + i + 3]};
        }
    }
    __syncthreads();
    for (int i = tid; i < G * DD; i += 256) {
        const int h = i / DD, dd = i - h * DD;
        const float M = fmaxf(fmaxf(ws_m[0][h], ws_m[1][h]), fmaxf(ws_m[2][h], ws_m[3][h]));
        float acc = 0.f, l = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float sc = ws_l[w][h] > 0.f ? __builtin_amdgcn_exp2f(ws_m[w][h] - M) : 0.f;
            acc += sc * (red[w][0][h][dd] + red[w][1][h][dd]);
            l += sc * ws_l[w][h];
        }
        float* dst = part + ((size_t)blockIdx.x * Hq + g * G + h) * DPART;
        dst[dd] = acc;
        if (dd == 0) { dst[DD] = M; dst[DD + 1] = l; }
    }
}

// One workgroup per query head: out = sum_i 2^(m_i - M) o_i / sum_i 2^(m_i - M) l_i over the at most kDecParts partials.
// 1024 threads = 8 groups of 128 features; group j takes the partials j, j + 8, ..  Everything is requested at once: the
// launch is one trip to memory.  A partial without keys has sum 0 and zero values, and gets weight 0.
constexpr int DMT = 1024;
constexpr int kDecParts = 128;   // partials per query head at most
constexpr int kDecWgs = 512;     // workgroups of the first kernel, over all kv heads
template <typename T>
__global__ void __launch_bounds__(DMT) decode_attn_merge_kernel(const float* __restrict__ part, int n_parts, int Hq,
                                                                T* __restrict__ out) {
    constexpr int NG = DMT / DD, PER = kDecParts / NG;
    __shared__ float wts[kDecParts];
    __shared__ float wred[2][kDecParts / 64];
    __shared__ float accs[NG][DD];
    const int h = blockIdx.x, tid = threadIdx.x, grp = tid >> 7, dd = tid & (DD - 1);
    auto item = [&](int i) { return part + ((size_t)min(i, n_parts - 1) * Hq + h) * DPART; };
    float val[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) val[i] = grp + i * NG < n_parts ? item(grp + i * NG)[dd] : 0.f;
    float m = -INFINITY, l = 0.f;
    if (tid < kDecParts) {
        if (tid < n_parts) { m = item(tid)[DD]; l = item(tid)[DD + 1]; }
        const float wm = wave_max(m);
        if ((tid & 63) == 0) wred[0][tid >> 6] = wm;
    }
    __syncthreads();
    float M = wred[0][0];
#pragma unroll
    for (int i = 1; i < kDecParts / 64; ++i) M = fmaxf(M, wred[0][i]);
    if (tid < kDecParts) {
        const float w = l > 0.f ? __builtin_amdgcn_exp2f(m - M) : 0.f;
        wts[tid] = w;
        const float ws = wave_sum(w * l);
        if ((tid & 63) == 0) wred[1][tid >> 6] = ws;
    }
    __syncthreads();
    float acc = 0.f;
#pragma unroll
    for (int i = 0; i < PER; ++i) acc += wts[grp + i * NG] * val[i];
    accs[grp][dd] = acc;
    __syncthreads();
    if (grp == 0) {
        float a = 0.f, l_all = 0.f;
#pragma unroll
        for (int i = 0; i < NG; ++i) a += accs[i][dd];
#pragma unroll
        for (int i = 0; i < kDecParts / 64; ++i) l_all += wred[1][i];
        Elem<T>::st(out + (size_t)h * DD + dd, a / l_all);
    }
}

// Workgroups per kv head: enough for kDecWgs in all, every wave the same number of groups where that can be, and no more
// partials than the caller's workspace holds (one per slot and per 64 response tokens).
static int decode_parts(int n_slots, int block, int n_resp, int Hkv) {
    const long long groups = (long long)n_slots * ((block + DGK - 1) / DGK) + (n_resp + DGK - 1) / DGK;
    const long long most = std::min<long long>(std::max(16, std::min(kDecParts, kDecWgs / Hkv)), (long long)n_slots + (n_resp + 63) / 64);
    const long long rounds = std::max<long long>(1, (groups + 4 * most - 1) / (4 * most));
    return (int)std::max<long long>(1, std::min(most, (groups + 4 * rounds - 1) / (4 * rounds)));
}

template <typename T, int G>
static void launch_decode_partial(const void* q, const void* pool, size_t slot_bytes, size_t layer_offset,
                                  const int* block_of_slot, int n_slots, int block, int n_prompt, const void* k_resp,
                                  const void* v_resp, int n_resp, int Hq, int Hkv, float sl, float* part, int n_parts,
                                  hipStream_t st) {
    hipLaunchKernelGGL((decode_attn_partial_kernel<T, G>), dim3(n_parts, Hkv), dim3(256), 0, st, (const T*)q,
                       (const unsigned char*)pool, slot_bytes, layer_offset, block_of_slot, n_slots, block, n_prompt,
                       (const T*)k_resp, (const T*)v_resp, n_resp, Hq, Hkv, sl, part);
}

template <typename T>
static int launch_decode_attn_t(const void* q, const void* pool, size_t slot_bytes, size_t layer_offset,
                                const int* block_of_slot, int n_slots, int block, int n_prompt, const void* k_resp,
                                const void* v_resp, int n_resp, int Hq, int Hkv, float sl, void* out, float* part,
                                hipStream_t st) {
    const int n_parts = decode_parts(n_slots, n_slots ? block : 1, n_resp, Hkv);
#define SLIM_DEC(GG) case GG: launch_decode_partial<T, GG>(q, pool, slot_bytes, layer_offset, block_of_slot, n_slots, block, \
                                                            n_prompt, k_resp, v_resp, n_resp, Hq, Hkv, sl, part, n_parts, st); break
    switch (Hq / Hkv) {
        SLIM_DEC(1); SLIM_DEC(2); SLIM_DEC(3); SLIM_DEC(4); SLIM_DEC(5); SLIM_DEC(6); SLIM_DEC(7); SLIM_DEC(8);
        default: return SLIM_UNSUPPORTED;
    }
#undef SLIM_DEC
    hipLaunchKernelGGL(decode_attn_merge_kernel<T>, dim3(Hq), dim3(DMT), 0, st, part, n_parts, Hq, (T*)out);
    return check_launch();
}

int launch_decode_attn(const void* q, const void* pool, size_t slot_bytes, size_t layer_offset, const int* block_of_slot,
                       int n_slots, int block, int n_prompt, const void* k_resp, const void* v_resp, int n_resp, int Hq,
                       int Hkv, float scale, int dtype, void* out, float* part, hipStream_t st) {
    const float sl = scale * 1.4426950408889634f;
    if (dtype == SLIM_BF16)
        return launch_decode_attn_t<bf16_t>(q, pool, slot_bytes, layer_offset, block_of_slot, n_slots, block, n_prompt, k_resp,
                                            v_resp, n_resp, Hq, Hkv, sl, out, part, st);
    return launch_decode_attn_t<float>(q, pool, slot_bytes, layer_offset, block_of_slot, n_slots, block, n_prompt, k_resp,
                                       v_resp, n_resp, Hq, Hkv, sl, out, part, st);
}

}  // namespace slim
