// Dense projections of the layer ("QKV Generation", output projection and FFN of Fig. 2):
//   out[m, n] = sum_k a[m, k] * w[n, k]            (both operands contiguous along k)
// with five epilogues: plain, + bias[n] (Q/K/V projections of models that have one), + residual,
// SwiGLU (two weight matrices, silu(gate) * up), and RoPE (+ bias, + per-token score partials) for the
// Query/Key projections of 128-wide heads.
//
// bf16 path: MFMA with fp32 accumulation, v_mfma_f32_16x16x32_bf16 in the main path (it runs against the power limit, and this
// instruction takes less of it: see the generator) and 32x32x16 in the few-row and ragged kernels.  The weight tile is the MFMA "A" operand
// and the activation tile the "B" operand, so a lane ends up with 4 consecutive output features of
// one token and stores them as one 8-byte vector.
//
// Main path (k_in a multiple of 64, many rows): 4 waves per workgroup, one per SIMD, 256x256 output tile
// (128 features x 2 matrices x 256 tokens for SwiGLU), each wave 128 x 128 of it, so that every MFMA fragment read
// from LDS feeds eight MFMAs.  Measured (us, 32x32x16 -> 16x16x32 loop): SwiGLU 9856 x 14336 from 4096 1705 -> 1540 (1.36 -> 1.50
// PFLOP/s), its down projection 903 -> 839, 8192^3 775 -> 708 (1.56 PFLOP/s), Keys of 32768 rows with rotation and scores 235 -> 216.
// Operand tiles go from global memory straight into LDS (global_load_lds_dwordx4, no VGPR staging), into rings of three weight and two
// activation tiles; MFMA fragments are read one k-step ahead of their use, across k-tiles too.  The
// k-loop is generated assembly (gen_gemm_asm.py -> gemm_bf16_mainloops.inc): with a lone wave per SIMD the order of
// MFMA, LDS and tile-load instructions inside the wave is the schedule.  The residual of the output and down projections comes in
// as MFMA fragments inside that loop.  Few rows, and residuals that the loop does not take (residual_in_four_waves), use C++ tiles with the
// same LDS layout and pipeline; a register-staged kernel with k predicates covers ragged k_in.
#include "slim_common.h"
#include "routes.h"
#include "tile_plan.h"

#include <algorithm>
#include <map>
#include <mutex>
#include <tuple>
#include <type_traits>

namespace slim {

enum { EPI_PLAIN = 0, EPI_RESIDUAL = 1, EPI_SWIGLU = 2, EPI_BIAS = 3, EPI_ROPE = 4, EPI_PARTIAL = 5 };
// EPI_BIAS: R is a bias vector [N].  EPI_ROPE: R is a bias vector or null, the rest comes in a EpiExtra.
// EPI_PARTIAL: the accumulators go to a float buffer as they are (EpiExtra::partial); split_gemm_kernel and split_gemm_large_kernel only.

// Extra operands: of the RoPE epilogue (heads of 128 features, one head per wave tile), of the fused RMSNorm, and
// of a second projection of the same rows carried by the same launch.
struct EpiExtra {
    const float* table = nullptr;        // [M][128]: cos of the 64 rotation angles of the token, then their sin
    const float* qt = nullptr;           // [N] float or null: head-group-summed window query (Eq. 2 by linearity)
    float* token_scores = nullptr;       // [M][N/128]: rotated, rounded key of (token, head) dotted with its part of qt
    const float* row_scale = nullptr;    // [M] float or null: out row m = row_scale[m] * (a[m,:] . w^T) (fused RMSNorm)
    // Second projection (two-size launch only): feature tiles tiles_n1.. belong to it.
    const bf16_t* w_2 = nullptr;         // [n_2][K]
    const bf16_t* r_2 = nullptr;         // its bias (EPI_BIAS)
    bf16_t* c_2 = nullptr;               // [M][ldo_2]
    int n_2 = 0, ldo_2 = 0, tiles_n1 = 0;
    // Key projection in the same launch (gemm_bf16_qkv_kernel only): feature tiles 0 .. tiles_nk - 1, with the RoPE epilogue.
    const bf16_t* w_k = nullptr;         // [n_k][K]
    const bf16_t* r_k = nullptr;         // its bias or null
    bf16_t* c_k = nullptr;               // [M][n_k]
    int n_k = 0, tiles_nk = 0;
    int round_m = 0;                     // > 0 (two-size launch): large tiles in groups of so many token tiles, see rounds_of
    float* partial = nullptr;            // EPI_PARTIAL: [M] rows of ldo floats
};

constexpr int BK = 64;                                   // k-depth of an LDS tile (8 chunks of 16 bytes)

// LDS tile: rows of 64 bf16 = 8 chunks of 16 B; chunk c of row r lives at chunk slot c ^ swz(r),
// so that the 16 lanes served together by a 128-bit LDS read hit distinct banks.
__device__ __forceinline__ int swz(int r) { return (r >> 1) & 7; }
__device__ __forceinline__ int lds_off(int r, int c) { return (r * 8 + (c ^ swz(r))) * 16; }   // bytes

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
#include "gemm_bf16_mainloops.inc"
#pragma clang diagnostic pop
constexpr int kRingW = 3;                                // weight tiles that the generated loops keep in LDS; activation tiles behind them
constexpr size_t kRingBytes = (size_t)(kRingW * 256 + 2 * 256) * BK * 2;   // (two of 256 rows, or three of 128)

// Accumulators of a wave tile of 32 TW features x 32 TA tokens, as MFMA tiles of T x T (T = 16 in the generated k-loops, 32 in the others):
// acc[w][i][j][4 * vg + e] is out[token m][feature n] with
//   m = mw + j*T + (lane % T),   n = nw + i*T + 8*vg + 4*(lane / T) + e      (mw, nw: the wave's origin)
template <int T> struct MfmaTile;
template <> struct MfmaTile<16> { typedef f32x4 Acc; static constexpr int kGroups = 1; };
template <> struct MfmaTile<32> { typedef f32x16 Acc; static constexpr int kGroups = 4; };

template <int T, int TW, int TA, int EPI>
__device__ __forceinline__ void store_tile(typename MfmaTile<T>::Acc (&acc)[EPI == EPI_SWIGLU ? 2 : 1][TW * 32 / T][TA * 32 / T], const bf16_t* R,
                                           bf16_t* C, int ldo, int M, int N, int mw, int nw, int lane, const float (&inv)[TA * 32 / T]) {
    constexpr int NW = EPI == EPI_SWIGLU ? 2 : 1, NI = TW * 32 / T, NJ = TA * 32 / T, VG = MfmaTile<T>::kGroups;
    const bool vec_ok = (N % 4 == 0) && (ldo % 4 == 0);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int m = mw + j * T + (lane & (T - 1));
        if (m >= M) continue;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
#pragma unroll
            for (int vg = 0; vg < VG; ++vg) {
                const int n = nw + i * T + 8 * vg + 4 * (lane / T);
                if (n >= N) continue;
                float o[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (EPI == EPI_SWIGLU) {
                        const float g = acc[0][i][j][vg * 4 + e] * inv[j], u = acc[NW - 1][i][j][vg * 4 + e] * inv[j];
                        o[e] = g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u;   // v_rcp_f32: 1 ulp, the result is rounded to bf16
                    } else {
                        o[e] = acc[0][i][j][vg * 4 + e] * inv[j];
                    }
                }
                bf16_t* dst = C + (size_t)m * ldo + n;
                if (vec_ok) {
                    if (EPI == EPI_RESIDUAL || EPI == EPI_BIAS) {
                        const uint2 r = *reinterpret_cast<const uint2*>(EPI == EPI_BIAS ? R + n : R + (size_t)m * ldo + n);
                        o[0] += lo_bf16(r.x); o[1] += hi_bf16(r.x); o[2] += lo_bf16(r.y); o[3] += hi_bf16(r.y);
                    }
                    *reinterpret_cast<uint2*>(dst) = make_uint2(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]));
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if (n + e < N) {
                            float val = o[e];
                            if (EPI == EPI_RESIDUAL) val += bf16_to_f32(R[(size_t)m * ldo + n + e]);
                            if (EPI == EPI_BIAS) val += bf16_to_f32(R[n + e]);
                            dst[e] = f32_to_bf16(val);
                        }
                    }
                }
            }
        }
    }
}

// Epilogue of the main kernel: the wave's tile goes through a wave-private LDS region so that global
// traffic is 16 bytes per lane and whole rows of the tile are contiguous (a lane of the accumulator
// layout owns only 4 consecutive features of one token).  Steps, all inside one wave (LDS operations
// of a wave complete in program order, so no barrier is needed):
//   residual only: rows of R are loaded coalesced and parked in the region;
//   each lane takes its accumulators, applies SiLU(gate)*up or adds its 4 residual values in fp32,
//   rounds once to bf16 and writes 8 bytes into the region;
//   rows are read back 16 bytes per lane and stored.
// Region layout: row = token (TA*32 rows of TW*64 bytes), 16-byte chunk c of row r at slot
// c ^ (r & (chunks per row - 1)).  Needs N % 8 == 0, ldo % 8 == 0 and 16-byte aligned out / residual.
template <int T, int TW, int TA, int EPI>
__device__ __forceinline__ void store_tile_via_lds(typename MfmaTile<T>::Acc (&acc)[EPI == EPI_SWIGLU ? 2 : 1][TW * 32 / T][TA * 32 / T],
                                                   const bf16_t* R, bf16_t* C, int ldo, int M, int N, int mw, int nw, int lane,
                                                   unsigned char* region, const float (&inv)[TA * 32 / T]) {
    constexpr int NW = EPI == EPI_SWIGLU ? 2 : 1, NI = TW * 32 / T, NJ = TA * 32 / T, VG = MfmaTile<T>::kGroups;
    constexpr int CPR = TW * 4, RB = TW * 64, ROWS = TA * 32, RPI = 64 / CPR;
    const int lt = lane & (T - 1), lq = lane / T;         // token of a tile, and which 4 of 8 (16) features
    const int rrow = lane / CPR, rchunk = lane % CPR;     // coalesced phases: lane -> (row in group, chunk)
    auto slot = [&](int row, int chunk) { return row * RB + ((chunk ^ (row & (CPR - 1))) << 4); };
    if (EPI == EPI_RESIDUAL) {
#pragma unroll
        for (int it = 0; it < ROWS / RPI; ++it) {
            const int row = it * RPI + rrow, m = mw + row, n = nw + rchunk * 8;
            uint4 v = make_uint4(0, 0, 0, 0);
            if (m < M && n < N) v = *reinterpret_cast<const uint4*>(R + (size_t)m * ldo + n);
            *reinterpret_cast<uint4*>(region + slot(row, rchunk)) = v;
        }
    }
    uint2 bias4[EPI == EPI_BIAS ? NI * VG : 1];           // the lane's bias values, requested together
    if (EPI == EPI_BIAS) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int vg = 0; vg < VG; ++vg) {
                const int n = nw + i * T + 8 * vg + 4 * lq;
                bias4[i * VG + vg] = n < N ? *reinterpret_cast<const uint2*>(R + n) : make_uint2(0, 0);
            }
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int vg = 0; vg < VG; ++vg) {
                const int row = j * T + lt;
                uint2* cell = reinterpret_cast<uint2*>(region + slot(row, i * (T / 8) + vg + (lq >> 1)) + (lq & 1) * 8);
                float o[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (EPI == EPI_SWIGLU) {
                        const float g = acc[0][i][j][vg * 4 + e] * inv[j], u = acc[NW - 1][i][j][vg * 4 + e] * inv[j];
                        o[e] = g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u;   // v_rcp_f32: 1 ulp, the result is rounded to bf16
                    } else {
                        o[e] = acc[0][i][j][vg * 4 + e] * inv[j];
                    }
                }
                if (EPI == EPI_RESIDUAL) {
                    const uint2 r = *cell;
                    o[0] += lo_bf16(r.x); o[1] += hi_bf16(r.x); o[2] += lo_bf16(r.y); o[3] += hi_bf16(r.y);
                }
                if (EPI == EPI_BIAS) {                    // 4 consecutive features of the bias vector (N % 8 == 0 here)
                    const uint2 r = bias4[EPI == EPI_BIAS ? i * VG + vg : 0];
                    o[0] += lo_bf16(r.x); o[1] += hi_bf16(r.x); o[2] += lo_bf16(r.y); o[3] += hi_bf16(r.y);
                }
                *cell = make_uint2(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]));
            }
#pragma unroll
    for (int it = 0; it < ROWS / RPI; ++it) {
        const int row = it * RPI + rrow, m = mw + row, n = nw + rchunk * 8;
        const uint4 v = *reinterpret_cast<const uint4*>(region + slot(row, rchunk));
        if (m < M && n < N) *reinterpret_cast<uint4*>(C + (size_t)m * ldo + n) = v;
    }
}

// RoPE epilogue.  The wave tile is 128 features wide and starts at a multiple of 128, so it is one head and the
// rotate-half partner of feature f < 64 is the same accumulator element half of the sub-tiles further on in
// the same lane: the rotation needs no exchange.  out[f] = x[f] cos - x[f+64] sin, out[f+64] = x[f+64] cos +
// x[f] sin with the angle of (token, f) from the table; x includes the bias.  One rounding to bf16.  With a
// window query, the rounded values are dotted with it (2 T of the head's features per lane, the others in the lanes
// T apart) and the per-(token, head) partial goes to token_scores.
template <int T, int TA>
__device__ __forceinline__ void store_tile_rope(typename MfmaTile<T>::Acc (&acc)[1][128 / T][TA * 32 / T], const bf16_t* bias, bf16_t* C, int ldo, int M,
                                                int N, int mw, int nw, int lane, unsigned char* region,
                                                const EpiExtra& re, const float (&inv)[TA * 32 / T]) {
    constexpr int TW = 4, CPR = TW * 4, RB = TW * 64, ROWS = TA * 32, RPI = 64 / CPR;
    constexpr int NJ = TA * 32 / T, VG = MfmaTile<T>::kGroups;
    if (nw >= N) return;                                 // wave-uniform: no head here (N is a multiple of 128)
    const int lt = lane & (T - 1), lq = lane / T;
    const int rrow = lane / CPR, rchunk = lane % CPR;
    auto slot = [&](int row, int chunk) { return row * RB + ((chunk ^ (row & (CPR - 1))) << 4); };
    const bool score = re.qt != nullptr;
    float dot[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) dot[j] = 0.f;
    // Per half of the head's rotation indices (i), every table, bias and window-query value the lane needs is requested
    // first and used afterwards: 8 * TA + 16 (T = 16: half of the second) loads in flight, one wait.  (Left to the compiler, the loads went out two
    // at a time, each pair waited for: forty memory round trips per tile.)
    const float* trow0[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) trow0[j] = re.table + (size_t)min(mw + j * T + lt, M - 1) * 128 + 4 * lq;
    constexpr int NS = 32 / T * VG;                      // pieces of 8 (16) rotation indices in half of the 64
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        float4 c4[NS][NJ], s4[NS][NJ], q1[NS], q2[NS];
        uint2 r1[NS], r2[NS];
#pragma unroll
        for (int p = 0; p < NS; ++p) {
            const int f = h * 32 + p * (32 / NS);        // rotation index of element e = 0 in lane group 0
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                c4[p][j] = *reinterpret_cast<const float4*>(trow0[j] + f);
                s4[p][j] = *reinterpret_cast<const float4*>(trow0[j] + f + 64);
            }
            r1[p] = r2[p] = make_uint2(0, 0);
            if (bias) {
                r1[p] = *reinterpret_cast<const uint2*>(bias + nw + f + 4 * lq);
                r2[p] = *reinterpret_cast<const uint2*>(bias + nw + 64 + f + 4 * lq);
            }
            q1[p] = q2[p] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (score) {
                q1[p] = *reinterpret_cast<const float4*>(re.qt + nw + f + 4 * lq);
                q2[p] = *reinterpret_cast<const float4*>(re.qt + nw + 64 + f + 4 * lq);
            }
        }
#pragma unroll
        for (int p = 0; p < NS; ++p) {
            const float b1[4] = {lo_bf16(r1[p].x), hi_bf16(r1[p].x), lo_bf16(r1[p].y), hi_bf16(r1[p].y)};
            const float b2[4] = {lo_bf16(r2[p].x), hi_bf16(r2[p].x), lo_bf16(r2[p].y), hi_bf16(r2[p].y)};
            const int i = h * (32 / T) + p / VG, vg = p % VG, chunk = i * (T / 8) + vg + (lq >> 1);
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const int row = j * T + lt;
                const float c[4] = {c4[p][j].x, c4[p][j].y, c4[p][j].z, c4[p][j].w};
                const float sn[4] = {s4[p][j].x, s4[p][j].y, s4[p][j].z, s4[p][j].w};
                float o1[4], o2[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float x1 = acc[0][i][j][vg * 4 + e] * inv[j] + b1[e], x2 = acc[0][i + 64 / T][j][vg * 4 + e] * inv[j] + b2[e];
                    o1[e] = x1 * c[e] - x2 * sn[e];
                    o2[e] = x2 * c[e] + x1 * sn[e];
                }
                const uint2 p1 = make_uint2(pack_bf16x2(o1[0], o1[1]), pack_bf16x2(o1[2], o1[3]));
                const uint2 p2 = make_uint2(pack_bf16x2(o2[0], o2[1]), pack_bf16x2(o2[2], o2[3]));
                *reinterpret_cast<uint2*>(region + slot(row, chunk) + (lq & 1) * 8) = p1;
                *reinterpret_cast<uint2*>(region + slot(row, chunk + 8) + (lq & 1) * 8) = p2;
                if (score)
                    dot[j] += lo_bf16(p1.x) * q1[p].x + hi_bf16(p1.x) * q1[p].y + lo_bf16(p1.y) * q1[p].z + hi_bf16(p1.y) * q1[p].w +
                              lo_bf16(p2.x) * q2[p].x + hi_bf16(p2.x) * q2[p].y + lo_bf16(p2.y) * q2[p].z + hi_bf16(p2.y) * q2[p].w;
            }
        }
    }
    if (score) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            float tot = dot[j] + __shfl_xor(dot[j], 32, 64);
            if (T == 16) tot += __shfl_xor(tot, 16, 64);
            const int m = mw + j * T + lt;
            if (lq == 0 && m < M) re.token_scores[(size_t)m * (N >> 7) + (nw >> 7)] = tot;
        }
    }
#pragma unroll
    for (int it = 0; it < ROWS / RPI; ++it) {
        const int row = it * RPI + rrow, m = mw + row, n = nw + rchunk * 8;
        const uint4 v = *reinterpret_cast<const uint4*>(region + slot(row, rchunk));
        if (m < M && n < N) *reinterpret_cast<uint4*>(C + (size_t)m * ldo + n) = v;
    }
}

// Epilogue of the split projections: the wave's float tile, unscaled, to rows of a float buffer.  32 tokens at a time go through the
// wave-private LDS region (rows of TW*128 bytes, 16-byte chunk c of row r at slot c ^ (r & (chunks per row - 1))), so
// that a row of the tile leaves as TW*128 contiguous bytes; a wave's LDS operations complete in order.  Needs N % 4 == 0.
template <int T, int TW, int TA>
__device__ __forceinline__ void store_tile_partial(typename MfmaTile<T>::Acc (&acc)[TW * 32 / T][TA * 32 / T], float* P, int ldp, int M, int N, int mw, int nw,
                                                   int lane, unsigned char* region) {
    constexpr int CPR = TW * 8, RB = TW * 128, RPI = 64 / CPR, VG = MfmaTile<T>::kGroups;
    const int lt = lane & (T - 1), lq = lane / T;
    const int rrow = lane / CPR, rchunk = lane % CPR;
    auto slot = [&](int row, int chunk) { return row * RB + ((chunk ^ (row & (CPR - 1))) << 4); };
#pragma unroll
    for (int j = 0; j < TA; ++j) {
#pragma unroll
        for (int t = 0; t < 32 / T; ++t)
#pragma unroll
            for (int i = 0; i < TW * 32 / T; ++i)
#pragma unroll
                for (int vg = 0; vg < VG; ++vg) {
                    const auto& c = acc[i][j * (32 / T) + t];
                    *reinterpret_cast<f32x4*>(region + slot(t * T + lt, i * (T / 4) + vg * 2 + lq)) =
                        f32x4{c[vg * 4], c[vg * 4 + 1], c[vg * 4 + 2], c[vg * 4 + 3]};
                }
#pragma unroll
        for (int it = 0; it < 32 / RPI; ++it) {
            const int row = it * RPI + rrow, m = mw + j * 32 + row, n = nw + rchunk * 4;
            const f32x4 v = *reinterpret_cast<const f32x4*>(region + slot(row, rchunk));
            if (m < M && n < N) *reinterpret_cast<f32x4*>(P + (size_t)m * ldp + n) = v;
        }
    }
}

// Workgroup -> output tile.  Workgroup ids are dealt round-robin to the 8 XCDs, so each XCD gets a
// contiguous run of logical tiles; inside the run, bands of GM token-tiles are walked feature-tile by
// feature-tile, so the workgroups resident on one XCD share few distinct operand tiles in its L2 (GM = 8: 32
// resident tiles are 8 x 4, the fewest panels; GM = 2 reads each activation panel in one go, see the residual kernel).
// L is the workgroup's index inside a region of tiles_m x tiles_n tiles that starts at a workgroup id
// divisible by 8 when xcd_runs is set.
__device__ __forceinline__ void tile_of_workgroup(int L, bool xcd_runs, int tiles_m, int tiles_n, int& tm, int& tn,
                                                  int GM = 8) {
    const int total = tiles_m * tiles_n;
    if (xcd_runs && total % 8 == 0) L = (L & 7) * (total >> 3) + (L >> 3);
    const int band_sz = GM * tiles_n;
    const int band = L / band_sz;
    const int gm = min(GM, tiles_m - band * GM);
    const int rem = L - band * band_sz;
    tm = band * GM + rem % gm;
    tn = rem / gm;
}

// One output tile of the few-row kernels.  WGN x WGM waves (4 or 8); requires 16-byte aligned rows; K is the row stride
// of the weights and the k-loop runs over the first KT tiles of 64 of the rows that A and W0 / W1 point at.
// The tile starts at token m0, feature n0; M and N bound the loads (clamped) and the stores.
// With re.row_scale the accumulators of token row m are multiplied by row_scale[m] before the epilogue: with
// row_scale = 1/sqrt(mean(a[m,:]^2) + eps) and a = the raw residual stream this is the projection of RMSNorm(a)
// (unit gain; a gain vector is folded into the weights beforehand), and the normalised rows are never stored.
// SPREAD: a k-tile's loads go out in four parts, each behind the LDS reads of a k-step.  In one burst behind the barrier, 4 to 8 of them keep the wave from its LDS reads while the
// address unit works through them; with two stages the burst is still the better one, since a tile's loads have no time to spare.  us, weights from HBM, burst / dealt: 256 x 128 tiles 2360 x
// 2176 from 960 16.4 / 14.6, 3968 x 1915 from 7744 142 / 138; 128 x 128 3993 x 640 from 3392 26.5 / 22.6, 1406 x 2012 from 2304 25.7 / 23.0; SwiGLU 200 x 14336 from 4096
// 67.9 / 65.1; 64 x 64 tiles +-1 %.
template <int TW, int TA, int WGN, int WGM, int EPI, int NS = 2, bool SPREAD = (NS >= 3)>
__device__ __forceinline__ void gemm_tile(const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ W0,
                                          const bf16_t* __restrict__ W1, const bf16_t* R, bf16_t* C, int ldo, int M,
                                          int N, int K, int KT, int m0, int n0, unsigned char* lds, const EpiExtra& re) {
    constexpr int WV = WGN * WGM;                        // waves
    static_assert(WV == 8 || WV == 4, "4 or 8 waves");
    static_assert(NS >= 2 && NS <= 5, "the k-loop is written out for up to 5 stages");
    static_assert(EPI != EPI_ROPE || TW == 4, "the RoPE epilogue needs one 128-wide head per wave");
    constexpr int NW = EPI == EPI_SWIGLU ? 2 : 1;
    constexpr int BN = 32 * TW * WGN, BM = 32 * TA * WGM, WROWS = BN * NW;
    constexpr int STAGE = (WROWS + BM) * BK * 2;
    constexpr int LR = WV * 8;                           // tile rows that one wave-load of every wave covers
    constexpr int WLD = WROWS / LR, ALD = BM / LR;       // wave-loads per k-tile per wave (8 rows each)
    static_assert(WLD * LR == WROWS && ALD * LR == BM && BN % LR == 0, "tile rows must split over the waves x 8 rows");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave % WGN, wm = wave / WGN;
    const int l32 = lane & 31, hh = lane >> 5;

    // Wave-load i covers rows (i*WV + wave)*8 + lane/8 of the tile; lane%8 is the LDS chunk slot, which
    // holds logical chunk slot ^ swz(row).  A load's address is a wave-uniform base (start of the tile's
    // rows + k offset, scalar registers) plus a loop-invariant per-lane byte offset inside the tile, so
    // the k-loop spends no vector instruction on addresses (a tile spans at most 256 rows: 32 bits do).
    unsigned woff[WLD], aoff[ALD];
#pragma unroll
    for (int i = 0; i < WLD; ++i) {
        const int r = (i * WV + wave) * 8 + (lane >> 3);
        const int mat = NW == 2 ? r / BN : 0;
        const int n = min(n0 + r - mat * BN, N - 1) - n0;
        woff[i] = (unsigned)(((size_t)n * K + ((lane & 7) ^ swz(r)) * 8) * 2);
    }
#pragma unroll
    for (int i = 0; i < ALD; ++i) {
        const int r = (i * WV + wave) * 8 + (lane >> 3);
        aoff[i] = (unsigned)(((size_t)(min(m0 + r, M - 1) - m0) * lda + ((lane & 7) ^ swz(r)) * 8) * 2);
    }
    const bf16_t* w0base = W0 + (size_t)n0 * K;
    const bf16_t* w1base = NW == 2 ? W1 + (size_t)n0 * K : W0;
    const bf16_t* abase = A + (size_t)m0 * lda;
    const unsigned lds_wave = (unsigned)(uintptr_t)lds + wave * 1024;
    auto issue_part = [&](int k0, int stage, int from, int to) {   // wave-loads from .. to - 1 of a k-tile
        const unsigned ws = lds_wave + stage * STAGE, as = ws + WROWS * BK * 2;
#pragma unroll
        for (int i = 0; i < WLD; ++i) {
            if (i < from || i >= to) continue;
            const bool second = NW == 2 && (i * LR >= BN);       // rows of wave-load i lie in one matrix (BN % LR == 0)
            load_global_to_lds16((second ? w1base : w0base) + k0, woff[i], ws + i * WV * 1024);
        }
#pragma unroll
        for (int i = 0; i < ALD; ++i)
            if (WLD + i >= from && WLD + i < to) load_global_to_lds16(abase + k0, aoff[i], as + i * WV * 1024);
    };

    f32x16 acc[NW][TW][TA];
#pragma unroll
    for (int w = 0; w < NW; ++w)
#pragma unroll
        for (int i = 0; i < TW; ++i)
#pragma unroll
            for (int j = 0; j < TA; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[w][i][j][v] = 0.f;

    bf16x8 af[2][TA], wf[2][NW][TW];
    // Fragment addresses: one per-lane base per (operand, stage, k-step), computed once; the MFMA tile
    // (i, j) and the matrix (gate/up) are immediate offsets of the LDS reads, so the k-loop spends no
    // vector instruction on them.  The swizzle term (row >> 1) & 7 depends only on lane % 32 because the
    // tile rows of a wave start at multiples of 32.
    const unsigned char* wfrag[NS][BK / 16];
    const unsigned char* afrag[NS][BK / 16];
#pragma unroll
    for (int st = 0; st < NS; ++st)
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            wfrag[st][ks] = lds + st * STAGE + lds_off(wn * TW * 32 + l32, ks * 2 + hh);
            afrag[st][ks] = lds + st * STAGE + WROWS * BK * 2 + lds_off(wm * TA * 32 + l32, ks * 2 + hh);
        }
    auto load_frags = [&](auto stage_c, int ks, int buf) {
        constexpr int stage = decltype(stage_c)::value;
#pragma unroll
        for (int j = 0; j < TA; ++j)
            af[buf][j] = *reinterpret_cast<const bf16x8*>(afrag[stage][ks] + j * 32 * BK * 2);
#pragma unroll
        for (int w = 0; w < NW; ++w)
#pragma unroll
            for (int i = 0; i < TW; ++i)
                wf[buf][w][i] = *reinterpret_cast<const bf16x8*>(wfrag[stage][ks] + (w * BN + i * 32) * BK * 2);
    };
    auto mfmas = [&](int buf) {
#pragma unroll
        for (int w = 0; w < NW; ++w)
#pragma unroll
            for (int i = 0; i < TW; ++i)
#pragma unroll
                for (int j = 0; j < TA; ++j)
                    acc[w][i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[buf][w][i], af[buf][j], acc[w][i][j], 0, 0, 0);
    };
    // NS LDS stages.  Fragments are read one k-step ahead of their MFMAs, also across k-tiles: the
    // workgroup barrier of a k-tile sits before its last k-step, when every wave has pulled that step's
    // fragments into registers.  Past the barrier the stage is free and tile kt+NS is sent into it: all of it at
    // once, or with SPREAD a quarter there and a quarter in each of the first three k-steps of tile kt+1, whose
    // waves still read another stage.  So at the wait before the barrier of tile kt the loads up to tile
    // kt+NS-1 have gone out, and all but the NS-2 youngest tiles of them are waited for: tile kt+1 is visible to
    // all waves past the barrier, and its first fragments are read while the last k-step's MFMAs run.  (The
    // wait in front of the loop is for tile 0 alone: NS-2 tiles and with SPREAD the first quarter of another are
    // behind it, NS-1 tiles without.)  The loop is unrolled by NS so the stage of every read is a compile-time
    // constant.  Loads past the last k-tile re-read it (into a stage that nobody reads), so the number of loads
    // in flight at a wait is a constant.
    constexpr unsigned kStageLoads = WLD + ALD;
    constexpr unsigned kParts = SPREAD ? 4 : 1;
    auto part = [](unsigned p) { return (int)(p * kStageLoads / kParts); };
    constexpr unsigned kFly = (NS - 2) * kStageLoads, kPro = SPREAD ? kFly + kStageLoads / kParts : (NS - 1) * kStageLoads;   // in flight behind a wait
    auto k_tile = [&](int kt, auto stage_c) {
        constexpr int stage = decltype(stage_c)::value;
        using Next = std::integral_constant<int, (stage + 1) % NS>;
#pragma unroll
        for (int ks = 0; ks < BK / 16 - 1; ++ks) {
            load_frags(stage_c, ks + 1, (ks + 1) & 1);
            if (SPREAD) issue_part(min(kt + NS - 1, KT - 1) * BK, (stage + NS - 1) % NS, part(ks + 1), part(ks + 2));
            __builtin_amdgcn_sched_barrier(0);           // keep the next step's LDS reads ahead of these MFMAs
            mfmas(ks & 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_waitcnt((kFly & 15) | 0x0070 | ((kFly >> 4) << 14));   // own reads of this stage and own part of tile kt+1 done
        workgroup_barrier();
        if (!SPREAD) issue_part(min(kt + NS, KT - 1) * BK, stage, 0, kStageLoads);
        load_frags(Next{}, 0, 0);
        if (SPREAD) issue_part(min(kt + NS, KT - 1) * BK, stage, 0, part(1));
        __builtin_amdgcn_sched_barrier(0);
        mfmas((BK / 16 - 1) & 1);
        __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int st = 0; st < NS; ++st) issue_part(min(st, KT - 1) * BK, st, 0, st < NS - 1 ? (int)kStageLoads : part(1));
    // only the first k-tile has to be there; the others stay in flight until the k-tiles' own waits
    __builtin_amdgcn_s_waitcnt((kPro & 15) | 0x0070 | ((kPro >> 4) << 14));
    workgroup_barrier();
    load_frags(std::integral_constant<int, 0>{}, 0, 0);
    for (int kt = 0;;) {
        k_tile(kt, std::integral_constant<int, 0>{});
        if (++kt >= KT) break;
        k_tile(kt, std::integral_constant<int, 1 % NS>{});
        if (++kt >= KT) break;
        if constexpr (NS >= 3) {
            k_tile(kt, std::integral_constant<int, 2 % NS>{});
            if (++kt >= KT) break;
        }
        if constexpr (NS >= 4) {
            k_tile(kt, std::integral_constant<int, 3 % NS>{});
            if (++kt >= KT) break;
        }
        if constexpr (NS >= 5) {
            k_tile(kt, std::integral_constant<int, 4 % NS>{});
            if (++kt >= KT) break;
        }
    }
    float inv[TA];                                       // (all requested before the first is used)
#pragma unroll
    for (int j = 0; j < TA; ++j) inv[j] = re.row_scale ? re.row_scale[min(m0 + (wm * TA + j) * 32 + l32, M - 1)] : 1.f;
    // SwiGLU's two products per output only where there is a scale: they are not hidden here (129 x 4096 from 64 4.72 us, always multiplied 4.89).
    if (EPI == EPI_SWIGLU) {
        if (re.row_scale) {
#pragma unroll
            for (int j = 0; j < TA; ++j)
#pragma unroll
                for (int w = 0; w < NW; ++w)
#pragma unroll
                    for (int i = 0; i < TW; ++i)
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[w][i][j][v] *= inv[j];
        }
#pragma unroll
        for (int j = 0; j < TA; ++j) inv[j] = 1.f;
    }
    // The epilogue reuses the stage buffers: every wave must be past its last fragment reads.
    __builtin_amdgcn_s_waitcnt(0x0070);
    workgroup_barrier();
    const bool wide = (N % 8 == 0) && (ldo % 8 == 0) && (((uintptr_t)C & 15) == 0) &&
                      (EPI != EPI_RESIDUAL || ((uintptr_t)R & 15) == 0) && (EPI != EPI_BIAS || ((uintptr_t)R & 7) == 0);
    if constexpr (EPI == EPI_PARTIAL) {
        store_tile_partial<32, TW, TA>(acc[0], re.partial, ldo, M, N, m0 + wm * TA * 32, n0 + wn * TW * 32, lane,
                                   lds + wave * (32 * TW * 128));
    } else if constexpr (EPI == EPI_ROPE) {              // the launcher has checked what `wide` checks
        store_tile_rope<32, TA>(acc, R, C, ldo, M, N, m0 + wm * TA * 32, n0 + wn * TW * 32, lane,
                            lds + wave * (TA * 32 * TW * 64), re, inv);
    } else {
        if (wide)
            store_tile_via_lds<32, TW, TA, EPI>(acc, R, C, ldo, M, N, m0 + wm * TA * 32, n0 + wn * TW * 32, lane,
                                            lds + wave * (TA * 32 * TW * 64), inv);
        else
            store_tile<32, TW, TA, EPI>(acc, R, C, ldo, M, N, m0 + wm * TA * 32, n0 + wn * TW * 32, lane, inv);
    }
}

// One output tile of the main path: 4 waves arranged 2 (features) x 2 (tokens), each with TW x TA MFMA tiles (of
// each weight matrix); requires K % 64 == 0, 16-byte aligned rows and row strides below 2^23 elements.  The k-loop
// is gemm_mainloop_<TW>_<TA>_<NW>; its operands:
//   wfrag0 / afrag0   LDS byte address of the lane's weight / activation fragment of k-step 0 in stage 0;
//   r0, chunk         the lane's row inside a group of 32 tile rows and its (swizzled) 16-byte chunk of a 128-byte
//                     row: wave-load i of a k-tile covers tile rows 32 i + r0 and lands at ldsw + i * 4096;
//   wlim / alim       last valid row of the tile (loads of rows beyond it are clamped to it; never stored);
//   strides in bytes, kt = K / 64, and the three tile origins.
// The tile starts at token m0, feature n0; M and N bound the loads and the stores.  row_scale as in gemm_tile.  KT: k-tiles to run
// over when that is not all of K (EPI_PARTIAL).  SCALED: there may be a row_scale (without one, a factor of one per output and two for SwiGLU cost
// products of few k-tiles 1 to 3 %, see gemm_bf16_two_size_unscaled_kernel).
template <int TW, int TA, int EPI, bool SCALED = true>
__device__ __forceinline__ void gemm_tile4(const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ W0,
                                           const bf16_t* __restrict__ W1, const bf16_t* R, bf16_t* C, int ldo, int M,
                                           int N, int K, int m0, int n0, unsigned char* lds, const EpiExtra& re, int KT = 0) {
    static_assert(EPI != EPI_ROPE || TW == 4, "the RoPE epilogue needs one 128-wide head per wave");
    constexpr int NW = EPI == EPI_SWIGLU ? 2 : 1;
    constexpr int BN = 64 * TW, WROWS = BN * NW;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave & 1, wm = wave >> 1;
    const int lt = lane & 15, lq = lane >> 4;            // MFMA tiles of 16 x 16, fragments of 16 rows x 32 of k
    const unsigned lds_base = (unsigned)(uintptr_t)lds;
    const unsigned wfrag0 = lds_base + lds_off(wn * TW * 32 + lt, lq);
    const unsigned afrag0 = lds_base + kRingW * WROWS * BK * 2 + lds_off(wm * TA * 32 + lt, lq);
    const unsigned r0 = wave * 8 + (lane >> 3), chunk = ((lane & 7) ^ swz(r0)) * 16;
    const uint64_t w0base = (uint64_t)(uintptr_t)(W0 + (size_t)n0 * K);
    const uint64_t w1base = NW == 2 ? (uint64_t)(uintptr_t)(W1 + (size_t)n0 * K) : w0base;
    const uint64_t abase = (uint64_t)(uintptr_t)(A + (size_t)m0 * lda);
    f32x4 acc[NW][2 * TW][2 * TA];
#define SLIM_LOOP_ARGS wfrag0, afrag0, r0, chunk, N - 1 - n0, M - 1 - m0, (unsigned)K * 2, (unsigned)lda * 2,          \
                       (unsigned)(KT ? KT : K / BK), lds_base + wave * 1024, w0base, w1base, abase, acc
    // With a residual the k-loop itself adds the tile of R to the accumulators (it fetches the tile as MFMA fragments
    // and multiplies it by identity slices), and the tile is then stored as a plain one.  The launcher has checked that
    // the tile has all its features and that the rows of R are 16-byte aligned.
    constexpr int EPI_OUT = EPI == EPI_RESIDUAL ? (int)EPI_PLAIN : EPI;
    if constexpr (EPI == EPI_RESIDUAL) {
        const unsigned rrow0 = wm * TA * 32 + lt;                               // the lane's token row of the tile (j = 0)
        const unsigned rcol0 = (unsigned)(n0 + wn * TW * 32 + 8 * lq) * 2;      // byte column of its 8 features
        const bf16_t* rbase = R + (size_t)m0 * ldo;
        if constexpr (TA == 4) gemm_mainloop_4_4_1_resid(SLIM_LOOP_ARGS, rrow0, rcol0, (unsigned)ldo * 2, rbase);
        else gemm_mainloop_4_2_1_resid(SLIM_LOOP_ARGS, rrow0, rcol0, (unsigned)ldo * 2, rbase);
    } else if constexpr (TW == 4 && TA == 4) gemm_mainloop_4_4_1(SLIM_LOOP_ARGS);
    else if constexpr (TW == 4 && TA == 2) gemm_mainloop_4_2_1(SLIM_LOOP_ARGS);
    else if constexpr (TW == 2 && TA == 4) gemm_mainloop_2_4_2(SLIM_LOOP_ARGS);
    else gemm_mainloop_2_2_2(SLIM_LOOP_ARGS);
#undef SLIM_LOOP_ARGS
    // The epilogue's per-lane values are formed again behind the loop from a lane id that the compiler must take as
    // new: anything it derived from the lane id earlier would otherwise be kept in VGPRs across the loop, which has
    // few to spare, and be spilled to scratch memory.
    int tid_e = tid;
    asm volatile("" : "+v"(tid_e));
    const int lane_e = tid_e & 63;
    static_assert((TW == 4 && NW == 1 && (TA == 4 || TA == 2)) || (TW == 2 && NW == 2 && (TA == 4 || TA == 2)),
                  "no generated k-loop for this wave tile");
    float inv[2 * TA];                                   // (all requested before the first is used)
#pragma unroll
    for (int j = 0; j < 2 * TA; ++j)
        inv[j] = SCALED && re.row_scale ? re.row_scale[min(m0 + wm * TA * 32 + j * 16 + (lane_e & 15), M - 1)] : 1.f;
    // The epilogue reuses the stage buffers: every wave must be past its last fragment reads and tile loads.
    __builtin_amdgcn_s_waitcnt(0x0070);
    workgroup_barrier();
    const bool wide = (N % 8 == 0) && (ldo % 8 == 0) && (((uintptr_t)C & 15) == 0) &&
                      (EPI != EPI_BIAS || ((uintptr_t)R & 7) == 0);
    if constexpr (EPI == EPI_PARTIAL) {
        store_tile_partial<16, TW, TA>(acc[0], re.partial, ldo, M, N, m0 + wm * TA * 32, n0 + wn * TW * 32, lane_e,
                                   lds + wave * (32 * TW * 128));
    } else if constexpr (EPI == EPI_ROPE) {              // the launcher has checked what `wide` checks
        store_tile_rope<16, TA>(acc, R, C, ldo, M, N, m0 + wm * TA * 32, n0 + wn * TW * 32, lane_e,
                            lds + wave * (TA * 32 * TW * 64), re, inv);
    } else {
        if (wide)
            store_tile_via_lds<16, TW, TA, EPI_OUT>(acc, R, C, ldo, M, N, m0 + wm * TA * 32, n0 + wn * TW * 32, lane_e,
                                            lds + wave * (TA * 32 * TW * 64), inv);
        else
            store_tile<16, TW, TA, EPI_OUT>(acc, R, C, ldo, M, N, m0 + wm * TA * 32, n0 + wn * TW * 32, lane_e, inv);
    }
}

// Few-row kernel: every workgroup computes one tile of the same shape, from NS LDS stages.
template <int TW, int TA, int WGN, int WGM, int EPI, int NS, bool SPREAD>
__global__ void __launch_bounds__(64 * WGN * WGM) gemm_bf16_kernel(const bf16_t* __restrict__ A, int lda,
                                                        const bf16_t* __restrict__ W0,
                                                        const bf16_t* __restrict__ W1, const bf16_t* R, bf16_t* C,
                                                        int ldo, int M, int N, int K, int tiles_m, int tiles_n,
                                                        EpiExtra re) {
    extern __shared__ __align__(16) unsigned char lds[];
    int tm, tn;
    tile_of_workgroup(blockIdx.x, true, tiles_m, tiles_n, tm, tn);
    gemm_tile<TW, TA, WGN, WGM, EPI, NS, SPREAD>(A, lda, W0, W1, R, C, ldo, M, N, K, K / BK, tm * 32 * TA * WGM, tn * 32 * TW * WGN, lds, re);
}

// Shapes of the two-size launch: 256-token tiles for the first big_tiles_m token-tiles, 128-token tiles
// (same feature width) for the rest.  Wave tiles: 128 features x 128 tokens (large), 128 x 64 (small); for SwiGLU
// the 128 features are 64 gate + 64 up.  Either way a wave of the plain shapes holds one 128-wide head (RoPE).
template <int EPI> struct TileShapes {
    static constexpr int TW = EPI == EPI_SWIGLU ? 2 : 4;
    static constexpr int TA_BIG = 4, TA_SMALL = 2;
    static constexpr int BN = 64 * TW;
    static constexpr int BM_BIG = 64 * TA_BIG, BM_SMALL = 64 * TA_SMALL;
};

// Two tile sizes in one launch.  Workgroups are started in id order, so the 256-token tiles run first
// and the 128-token tiles fill the last, partly empty round of workgroups: the tail of the launch costs
// about half a tile time instead of a whole one, and a ragged last token-tile wastes no MFMA work.
template <int EPI, bool SCALED>
__device__ __forceinline__ void two_size_tile(const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ W0,
                                              const bf16_t* __restrict__ W1, const bf16_t* R, bf16_t* C, int ldo, int M, int N, int K,
                                              int big_tiles_m, int small_tiles_m, int tiles_n, const EpiExtra& re) {
    using S = TileShapes<EPI>;
    extern __shared__ __align__(16) unsigned char lds[];
    const int n_big = big_tiles_m * tiles_n;
    const bool big = (int)blockIdx.x < n_big;
    int tm, tn;
    if (big) {
        const int rm = re.round_m > 0 ? re.round_m : big_tiles_m, c = blockIdx.x / (rm * tiles_n);
        tile_of_workgroup(blockIdx.x - c * rm * tiles_n, true, min(rm, big_tiles_m - c * rm), tiles_n, tm, tn);
        tm += c * rm;
    } else {
        tile_of_workgroup(blockIdx.x - n_big, n_big % 8 == 0, small_tiles_m, tiles_n, tm, tn);
    }
    if (re.w_2 && tn >= re.tiles_n1) {                   // a feature tile of the second projection
        W0 = re.w_2; R = re.r_2; C = re.c_2; N = re.n_2; ldo = re.ldo_2;
        tn -= re.tiles_n1;
    }
    if (big)
        gemm_tile4<S::TW, S::TA_BIG, EPI, SCALED>(A, lda, W0, W1, R, C, ldo, M, N, K, tm * S::BM_BIG, tn * S::BN, lds, re);
    else
        gemm_tile4<S::TW, S::TA_SMALL, EPI, SCALED>(A, lda, W0, W1, R, C, ldo, M, N, K,
                                                    big_tiles_m * S::BM_BIG + tm * S::BM_SMALL, tn * S::BN, lds, re);
}

template <int EPI>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
gemm_bf16_two_size_kernel(const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ W0,
                          const bf16_t* __restrict__ W1, const bf16_t* R, bf16_t* C, int ldo, int M, int N, int K,
                          int big_tiles_m, int small_tiles_m, int tiles_n, EpiExtra re) {
    two_size_tile<EPI, EPI != EPI_RESIDUAL>(A, lda, W0, W1, R, C, ldo, M, N, K, big_tiles_m, small_tiles_m, tiles_n, re);
}

// Plain and SwiGLU without a row scale.  us, two LDS slots and the scale under a branch / three slots and a factor of one / so: 12345 x 4096 from 128 36.2 / 37.3 / 35.3,
// SwiGLU of 16384 rows 76.2 / 77.7 / 72.9; 12345 x 4096 from 64 31.4 / 31.8 / 29.6, SwiGLU 49.2 / 48.5 / 44.2.
template <int EPI>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
gemm_bf16_two_size_unscaled_kernel(const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ W0,
                                   const bf16_t* __restrict__ W1, const bf16_t* R, bf16_t* C, int ldo, int M, int N, int K,
                                   int big_tiles_m, int small_tiles_m, int tiles_n, EpiExtra re) {
    two_size_tile<EPI, false>(A, lda, W0, W1, R, C, ldo, M, N, K, big_tiles_m, small_tiles_m, tiles_n, re);
}

// Query, Key and Value projections of the same rows in one launch: the feature tiles of the Keys (128-wide heads, rotated in the
// epilogue, which takes longest) come first, then the other two as in the launch of a pair.  As launches of their own the Keys of
// 2048 or 4096 rows are 32 or 64 tiles: a layer of 4096 rows that drops nothing (4096 + 1024 + 1024 features) 1550 -> 1526 us,
// 2048 rows 858 -> 833.
template <int EPI>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
gemm_bf16_qkv_kernel(const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ W0, const bf16_t* R, bf16_t* C, int ldo, int M,
                     int N, int K, int big_tiles_m, int small_tiles_m, int tiles_n, EpiExtra re) {
    using S = TileShapes<EPI>;
    extern __shared__ __align__(16) unsigned char lds[];
    const int n_big = big_tiles_m * tiles_n;
    const bool big = (int)blockIdx.x < n_big;
    int tm, tn;
    if (big) tile_of_workgroup(blockIdx.x, true, big_tiles_m, tiles_n, tm, tn);
    else tile_of_workgroup(blockIdx.x - n_big, n_big % 8 == 0, small_tiles_m, tiles_n, tm, tn);
    const int m0 = big ? tm * S::BM_BIG : big_tiles_m * S::BM_BIG + tm * S::BM_SMALL;
    if (tn < re.tiles_nk) {
        if (big) gemm_tile4<4, S::TA_BIG, EPI_ROPE>(A, lda, re.w_k, nullptr, re.r_k, re.c_k, re.n_k, M, re.n_k, K, m0, tn * S::BN, lds, re);
        else gemm_tile4<4, S::TA_SMALL, EPI_ROPE>(A, lda, re.w_k, nullptr, re.r_k, re.c_k, re.n_k, M, re.n_k, K, m0, tn * S::BN, lds, re);
        return;
    }
    tn -= re.tiles_nk;
    if (tn >= re.tiles_n1) {
        W0 = re.w_2; R = re.r_2; C = re.c_2; N = re.n_2; ldo = re.ldo_2;
        tn -= re.tiles_n1;
    }
    if (big) gemm_tile4<4, S::TA_BIG, EPI>(A, lda, W0, nullptr, R, C, ldo, M, N, K, m0, tn * S::BN, lds, re);
    else gemm_tile4<4, S::TA_SMALL, EPI>(A, lda, W0, nullptr, R, C, ldo, M, N, K, m0, tn * S::BN, lds, re);
}

// Residual projections that the 4-wave loop does not take (residual_in_four_waves).  Their epilogue reads a second tile through LDS; with
// a lone wave per SIMD nothing hides that pass, with two one wave's epilogue steps overlap the other's.  So 8 waves: wave tiles of 64
// tokens x 128 features (large) and 64 x 64 (small), the same workgroup tiles as above.
__global__ void __launch_bounds__(512)
gemm_bf16_two_size_residual_kernel(const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ W0, const bf16_t* R,
                                   bf16_t* C, int ldo, int M, int N, int K, int big_tiles_m, int small_tiles_m,
                                   int tiles_n, int band) {
    using S = TileShapes<EPI_RESIDUAL>;
    extern __shared__ __align__(16) unsigned char lds[];
    const int n_big = big_tiles_m * tiles_n;
    const bool big = (int)blockIdx.x < n_big;
    int tm, tn;
    if (big) tile_of_workgroup(blockIdx.x, true, big_tiles_m, tiles_n, tm, tn, band);
    else tile_of_workgroup(blockIdx.x - n_big, n_big % 8 == 0, small_tiles_m, tiles_n, tm, tn, band);
    const EpiExtra none;
    if (big)
        gemm_tile<4, 2, 2, 4, EPI_RESIDUAL>(A, lda, W0, nullptr, R, C, ldo, M, N, K, K / BK, tm * S::BM_BIG, tn * S::BN, lds, none);
    else
        gemm_tile<2, 2, 4, 2, EPI_RESIDUAL>(A, lda, W0, nullptr, R, C, ldo, M, N, K, K / BK,
                                            big_tiles_m * S::BM_BIG + tm * S::BM_SMALL, tn * S::BN, lds, none);
}

// Split projection: up to three weight matrices that read the same rows, the reduction dimension dealt to `splits`
// workgroups, float partial sums partial[split][m][all features] that split.hip finishes.  What it is for: with few rows
// a launch of one workgroup per output tile leaves most of the chip idle (4096 features x 512 tokens are 64 tiles of
// 256 x 128), and the finishing pass takes the place of the RoPE kernel anyway.  Down projection (k_in 14336, 4096
// features), with the finishing pass: 300 rows 256 -> 67 us, 512 rows 275 -> 79 us, 1024 rows 272 -> 137 us.
struct SplitSegs {
    const bf16_t* w[3];
    int n[3];                            // features (multiples of 4)
    int tile0[3], col0[3];               // first feature tile of the matrix, first column of its sums
    int ldp;                             // floats per row of the partial buffer
};

// Workgroup -> (token tile, feature tile, split), token tiles fastest and splits slowest inside each XCD's contiguous
// run: the tiles that read a weight panel run together on one XCD, which then fetches it from HBM once, and an XCD sees
// few of the splits and so little of the activation matrix.
template <int TW, int TA, int WGN, int WGM, int NS>
__global__ void __launch_bounds__(64 * WGN * WGM, 2)
split_gemm_kernel(const bf16_t* __restrict__ A, int lda, SplitSegs segs, float* __restrict__ partial, int M, int K, int tiles_m,
                  int tiles_n, int splits) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int total = tiles_m * tiles_n * splits;
    int L = blockIdx.x;
    if (total % 8 == 0) L = (L & 7) * (total >> 3) + (L >> 3);
    const int tm = L % tiles_m, rest = L / tiles_m, tn = rest % tiles_n, sp = rest / tiles_n;
    const int seg = (tn >= segs.tile0[1]) + (tn >= segs.tile0[2]);
    const bf16_t* W = seg == 0 ? segs.w[0] : seg == 1 ? segs.w[1] : segs.w[2];
    const int N = seg == 0 ? segs.n[0] : seg == 1 ? segs.n[1] : segs.n[2];
    const int t0 = seg == 0 ? 0 : seg == 1 ? segs.tile0[1] : segs.tile0[2];
    const int c0 = seg == 0 ? 0 : seg == 1 ? segs.col0[1] : segs.col0[2];
    const int KT = K / BK, lo = (int)((long long)KT * sp / splits), hi = (int)((long long)KT * (sp + 1) / splits);
    EpiExtra re;
    re.partial = partial + (size_t)sp * M * segs.ldp + c0;
    gemm_tile<TW, TA, WGN, WGM, EPI_PARTIAL, NS>(A + lo * BK, lda, W + lo * BK, nullptr, nullptr, nullptr, segs.ldp, M, N, K, hi - lo,
                                             tm * 32 * TA * WGM, (tn - t0) * 32 * TW * WGN, lds, re);
}

// The same for one matrix in the 256 x 256 tiles and the k-loop of the main path: long reductions whose tiles alone do not fill the chip.
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
split_gemm_large_kernel(const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ W, float* __restrict__ partial, int M, int N, int K,
                        int tiles_m, int tiles_n, int splits) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int total = tiles_m * tiles_n * splits;
    int L = blockIdx.x;
    if (total % 8 == 0) L = (L & 7) * (total >> 3) + (L >> 3);
    const int sp = L / (tiles_m * tiles_n);
    int tm, tn;
    tile_of_workgroup(L - sp * tiles_m * tiles_n, false, tiles_m, tiles_n, tm, tn);
    const int KT = K / BK, lo = (int)((long long)KT * sp / splits), hi = (int)((long long)KT * (sp + 1) / splits);
    EpiExtra re;
    re.partial = partial + (size_t)sp * M * N;
    gemm_tile4<4, 4, EPI_PARTIAL>(A + lo * BK, lda, W + lo * BK, nullptr, nullptr, nullptr, N, M, N, K, tm * 256, tn * 256, lds, re, hi - lo);
}

// Generic kernel (any k_in that is a multiple of 8): register-staged loads with k predicates.
// TW x TA: number of 32-row MFMA tiles per wave along the weight (n) and activation (m) directions.
// Workgroup = 4 waves arranged WGN x WGM.  SwiGLU uses two weight tiles per n (gate, up).
template <int TW, int TA, int WGN, int WGM, int EPI>
__global__ void __launch_bounds__(256) gemm_bf16_generic_kernel(const bf16_t* __restrict__ A, int lda,
                                                        const bf16_t* __restrict__ W0,
                                                        const bf16_t* __restrict__ W1,
                                                        const bf16_t* R, bf16_t* C, int ldo, int M, int N, int K,
                                                        int tiles_m, int tiles_n) {
    static_assert(WGN * WGM == 4, "4 waves");
    constexpr int NW = EPI == EPI_SWIGLU ? 2 : 1;        // weight matrices
    constexpr int BN = 32 * TW * WGN;                    // output features per workgroup (per matrix)
    constexpr int BM = 32 * TA * WGM;                    // tokens per workgroup
    constexpr int WROWS = BN * NW;                       // weight rows staged per k-tile
    constexpr int STAGE = (WROWS + BM) * BK * 2;         // bytes per LDS stage
    extern __shared__ __align__(16) unsigned char lds[];

    int tm, tn;
    tile_of_workgroup(blockIdx.x, true, tiles_m, tiles_n, tm, tn);
    const int n0 = tn * BN, m0 = tm * BM;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wn = wave % WGN, wm = wave / WGN;
    const int l32 = lane & 31, hh = lane >> 5;

    // global -> register staging: thread owns chunk column (tid & 7) of rows (tid >> 3) + 32*i
    constexpr int WLD = WROWS / 32, ALD = BM / 32;
    uint4 wreg[WLD], areg[ALD];
    const int lc = tid & 7, lr = tid >> 3;
    auto load_tiles = [&](int k0) {
        const int kk = k0 + lc * 8;
        const bool kin = kk < K;
#pragma unroll
        for (int i = 0; i < WLD; ++i) {
            const int r = lr + 32 * i;
            const int mat = NW == 2 ? r / BN : 0;
            const int n = min(n0 + (NW == 2 ? r - mat * BN : r), N - 1);
            const bf16_t* src = (mat ? W1 : W0) + (size_t)n * K + kk;
            wreg[i] = kin ? *reinterpret_cast<const uint4*>(src) : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < ALD; ++i) {
            const int m = min(m0 + lr + 32 * i, M - 1);
            areg[i] = kin ? *reinterpret_cast<const uint4*>(A + (size_t)m * lda + kk) : make_uint4(0, 0, 0, 0);
        }
    };
    auto store_tiles = [&](int stage) {
        unsigned char* ws = lds + stage * STAGE;
        unsigned char* as = ws + WROWS * BK * 2;
#pragma unroll
        for (int i = 0; i < WLD; ++i) *reinterpret_cast<uint4*>(ws + lds_off(lr + 32 * i, lc)) = wreg[i];
#pragma unroll
        for (int i = 0; i < ALD; ++i) *reinterpret_cast<uint4*>(as + lds_off(lr + 32 * i, lc)) = areg[i];
    };

    f32x16 acc[NW][TW][TA];
#pragma unroll
    for (int w = 0; w < NW; ++w)
#pragma unroll
        for (int i = 0; i < TW; ++i)
#pragma unroll
            for (int j = 0; j < TA; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[w][i][j][v] = 0.f;

    const int KT = (K + BK - 1) / BK;
    load_tiles(0);
    store_tiles(0);
    __syncthreads();
    for (int kt = 0; kt < KT; ++kt) {
        if (kt + 1 < KT) load_tiles((kt + 1) * BK);
        const unsigned char* ws = lds + (kt & 1) * STAGE;
        const unsigned char* as = ws + WROWS * BK * 2;
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            bf16x8 af[TA], wf[NW][TW];
#pragma unroll
            for (int j = 0; j < TA; ++j)
                af[j] = *reinterpret_cast<const bf16x8*>(as + lds_off((wm * TA + j) * 32 + l32, ks * 2 + hh));
#pragma unroll
            for (int w = 0; w < NW; ++w)
#pragma unroll
                for (int i = 0; i < TW; ++i)
                    wf[w][i] = *reinterpret_cast<const bf16x8*>(
                        ws + lds_off(w * BN + (wn * TW + i) * 32 + l32, ks * 2 + hh));
#pragma unroll
            for (int w = 0; w < NW; ++w)
#pragma unroll
                for (int i = 0; i < TW; ++i)
#pragma unroll
                    for (int j = 0; j < TA; ++j)
                        acc[w][i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[w][i], af[j], acc[w][i][j], 0, 0, 0);
        }
        if (kt + 1 < KT) store_tiles((kt + 1) & 1);
        __syncthreads();
    }

    float inv[TA];
#pragma unroll
    for (int j = 0; j < TA; ++j) inv[j] = 1.f;
    store_tile<32, TW, TA, EPI>(acc, R, C, ldo, M, N, m0 + wm * TA * 32, n0 + wn * TW * 32, lane, inv);
}

template <int TW, int TA, int WGN, int WGM, int EPI, bool GENERIC, int NS = 2, bool SPREAD = (NS >= 3)>
static int launch_bf16(const bf16_t* A, int lda, const bf16_t* W0, const bf16_t* W1, const bf16_t* R, bf16_t* C,
                       int ldo, int M, int N, int K, hipStream_t st, const EpiExtra& re = EpiExtra()) {
    constexpr int NW = EPI == EPI_SWIGLU ? 2 : 1;
    constexpr int BN = 32 * TW * WGN, BM = 32 * TA * WGM;
    constexpr size_t smem = NS * (size_t)(BN * NW + BM) * BK * 2;
    const void* kern;
    if constexpr (GENERIC) kern = (const void*)gemm_bf16_generic_kernel<TW, TA, WGN, WGM, EPI>;
    else kern = (const void*)gemm_bf16_kernel<TW, TA, WGN, WGM, EPI, NS, SPREAD>;
    static std::once_flag attr_once;                     // raising the LDS limit is per function, once
    static hipError_t attr_err = hipSuccess;
    std::call_once(attr_once, [&] { attr_err = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem); });
    if (attr_err != hipSuccess) return set_hip_error(attr_err);
    const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    if constexpr (GENERIC)
        hipLaunchKernelGGL((gemm_bf16_generic_kernel<TW, TA, WGN, WGM, EPI>), dim3(tiles_m * tiles_n), dim3(64 * WGN * WGM),
                           smem, st, A, lda, W0, W1, R, C, ldo, M, N, K, tiles_m, tiles_n);
    else
        hipLaunchKernelGGL((gemm_bf16_kernel<TW, TA, WGN, WGM, EPI, NS, SPREAD>), dim3(tiles_m * tiles_n), dim3(64 * WGN * WGM), smem,
                           st, A, lda, W0, W1, R, C, ldo, M, N, K, tiles_m, tiles_n, re);
    return check_launch();
}

// plan_tiles, remembered: the result is a pure function of its arguments (guarded, never invalidated).
// makespan_out: of the plan, in times of a 256-token tile.
static int plan_big_tiles(int M, int tiles_n, int n_cu, double small_cost, bool eight_waves, double* makespan_out = nullptr) {
    static std::mutex mu;
    static std::map<std::tuple<int, int, int, bool>, std::pair<int, double>> cache;
    std::lock_guard<std::mutex> lock(mu);
    const auto key = std::make_tuple(M, tiles_n, (int)(small_cost * 1000), eight_waves);
    auto hit = cache.find(key);
    if (hit == cache.end()) hit = cache.emplace(key, plan_tiles(M, tiles_n, n_cu, small_cost, eight_waves)).first;
    if (makespan_out) *makespan_out = hit->second.second;
    return hit->second.first;
}

// Which tile the residual epilogue runs in.  The 4-wave tile takes the residual tile in as MFMA fragments (16-byte loads
// at the lane's own rows and features), which needs every tile to have all of its features and 16-byte aligned rows of
// R.  The 8-wave tile's epilogue parks a coalesced copy of the tile of R in LDS and takes any shape; it issues a k-tile's loads at once.
// One launch of either, all rows (us, 4 waves / 8 waves): 4096 features from 4096, 4096 rows 96 / 116, 9856 232 / 290, 32768 783 / 955; from 14336, 4096 rows
// 307 / 380, 9856 786 / 1005, 32768 2647 / 3176; 6656 from 14336, 6000 rows 837 / 1004, 16384 rows 2187 / 2586.
// The bound on long activation rows was drawn with the 4-wave loops before these, which lost 4-7 % once the rows streamed from HBM; these do not lose, and
// of the shapes that the 4-wave tile could take, widths whose rounds do not fill the chip (6656; residual_round_rows) still go to the 8-wave tile.
constexpr size_t kResidualCacheBytes = (size_t)176 << 20;
static bool residual_in_four_waves(const bf16_t* R, int M, int N, int K, int ldo) {
    const size_t activation_bytes = (size_t)M * K * sizeof(bf16_t);
    return N % 256 == 0 && ldo % 8 == 0 && ((uintptr_t)R & 15) == 0 &&
           (K <= 8192 || activation_bytes <= kResidualCacheBytes);
}

// What a 128-token tile costs next to a 256-token one of the same launch.  Launches of exactly a round (us, 256-token tiles / 128-token tiles, half the rows): 4096
// features from 1024 31.2 / 19.9, from 4096 94 / 52, from 14336 300 / 165, with residual 34.3 / 21.1, 96 / 54, 304 / 167 (8 waves 40 / 24, 117 / 66, 379 / 206); SwiGLU,
// 8192 from 1024 29.7 / 18.1, from 4096 91 / 51.  Rows that come from HBM cost small tiles more: 8192 rows of 14336 605 in large ones, 749 in small.
template <int EPI> constexpr double small_tile_cost(bool eight_waves) {
    return eight_waves ? 0.5 : (EPI == EPI_SWIGLU ? 0.7 : 0.6);
}

int cu_count() {
    static std::once_flag once;                          // immutable once read: a property of the device
    static int n = 256;
    std::call_once(once, [] {
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess && prop.multiProcessorCount > 0)
            n = prop.multiProcessorCount;
    });
    return n;
}

// Token tiles per group of a launch's large tiles: as many as make one round of workgroups, so that all XCDs work on the same few
// activation panels and each on its own weight panels (with one run of tiles per XCD over the whole launch they work on eight distant
// row bands).  0: one group.
// Only where the group fills the chip to 85 %, divides evenly over the XCDs and leaves some CUs: groups of exactly a round lose (us without / with:
// 8192 features from 1024, 27136 rows 364 / 393; with a second matrix of 256 features 380 / 483).
// From 8 rounds of large tiles on: SwiGLU projection, 14336 features (112 tiles, groups of 2 x 112): 9856 rows 1524 -> 1506, 20000 3122 -> 3098, 26240 4036 ->
// 4029 (6000 rows 934 / 937); Query + Value (20 tiles, 12 x 20; 26240 rows are fewer rounds, 786 / 753): 32768 rows 969 -> 928, 40960 1210 -> 1157.
// 18944 features (148 tiles) have no such group, and the nearest, 2 x 148, changes nothing.  Residual and RoPE launches measure the same either way.
static int rounds_of(int big_tiles_m, int tiles_n) {
    const int rm = cu_count() / tiles_n;
    return rm >= 2 && (long long)big_tiles_m * tiles_n >= 8ll * cu_count() && rm * tiles_n * 100 >= cu_count() * 85 && rm * tiles_n < cu_count() && rm * tiles_n % 8 == 0 ? rm : 0;
}

template <int EPI>
static int launch_two_size(const bf16_t* A, int lda, const bf16_t* W0, const bf16_t* W1, const bf16_t* R, bf16_t* C,
                           int ldo, int M, int N, int K, int big_tiles_m, bool eight_waves, hipStream_t st,
                           const EpiExtra& re = EpiExtra()) {
    using S = TileShapes<EPI>;
    constexpr size_t smem8 = 2 * (size_t)(S::BN + S::BM_BIG) * BK * 2;
    static std::once_flag attr_once, attr8_once;
    static hipError_t attr_err = hipSuccess, attr8_err = hipSuccess;
    if ((size_t)K >= (1u << 23) || (size_t)lda >= (1u << 23) || (size_t)ldo >= (1u << 23))
        return SLIM_UNSUPPORTED;                         // 32-bit byte offsets inside a tile
    const int tiles_n = (N + S::BN - 1) / S::BN + (re.w_2 ? (re.n_2 + S::BN - 1) / S::BN : 0);
    const int small_tiles_m = std::max(0, M - big_tiles_m * S::BM_BIG + S::BM_SMALL - 1) / S::BM_SMALL;
    const dim3 grid((big_tiles_m + small_tiles_m) * tiles_n);
    if (EPI == EPI_RESIDUAL && eight_waves) {
        auto kern = gemm_bf16_two_size_residual_kernel;
        std::call_once(attr8_once, [&] {
            attr8_err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem8);
        });
        if (attr8_err != hipSuccess) return set_hip_error(attr8_err);
        // Long activation rows that stream from HBM (the matrix does not fit the memory-side cache): bands of 2
        // token-tiles, so that the tiles resident on an XCD cover every feature tile of a token band and each
        // activation panel is fetched once instead of once per group of 4 feature tiles (down projection of 9856
        // tokens -1.8 %, of 32768 tokens -2.6 %; with rows of 4096 the same walk is 6 % slower, so it is not used there).
        const int band = ((size_t)M * K * sizeof(bf16_t) > ((size_t)160 << 20) && K > 8192) ? 2 : 8;
        hipLaunchKernelGGL(kern, grid, dim3(512), smem8, st, A, lda, W0, R, C, ldo, M, N, K, big_tiles_m, small_tiles_m, tiles_n,
                           band);
    } else {
        auto kern = gemm_bf16_two_size_kernel<EPI>, unscaled = kern;
        if constexpr (EPI == EPI_PLAIN || EPI == EPI_SWIGLU) unscaled = gemm_bf16_two_size_unscaled_kernel<EPI>;
        std::call_once(attr_once, [&] {
            for (auto k : {kern, unscaled})
                if (attr_err == hipSuccess) attr_err = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kRingBytes);
        });
        if (attr_err != hipSuccess) return set_hip_error(attr_err);
        if (EPI == EPI_RESIDUAL && re.row_scale) return SLIM_UNSUPPORTED;      // (no caller has both)
        if (!re.row_scale) kern = unscaled;
        EpiExtra walk = re;
        if (EPI == EPI_SWIGLU || EPI == EPI_PLAIN || EPI == EPI_BIAS) walk.round_m = rounds_of(big_tiles_m, tiles_n);
        hipLaunchKernelGGL(kern, grid, dim3(256), kRingBytes, st, A, lda, W0, W1, R, C, ldo, M, N, K, big_tiles_m, small_tiles_m,
                           tiles_n, walk);
    }
    return check_launch();
}

// Tile shapes of the few-row kernels: (features x tokens), waves, LDS stages.  All of them keep 80-144 KB of operand tiles
// in flight or in use per CU, because with few rows the loop waits for memory (weights come from HBM once, and a k-tile of
// these tiles lasts no longer than a load takes): two stages of the 128 x 128 tile (64 KB) run the k-loop at 0.70 us per
// k-tile, four at 0.45.
//   FEW_A  256 x 128, 8 waves, 3 stages (144 KB, one workgroup per CU): fewest operand bytes per flop
//   FEW_B  128 x 128, 4 waves, 4 stages (128 KB)
//   FEW_C  128 x  64, 4 waves, 3 stages  (72 KB, two per CU)
//   FEW_D   64 x  64, 4 waves, 5 stages  (80 KB, two per CU)
// Taken is the largest that still gives kFewWorkgroups workgroups, else FEW_D; FEW_A also where FEW_B would begin a second round
// (residual, 3584 features, k_in 3584, 1290 rows: A (154) 46, B (308) 65; 2048 from 2048, 2049 rows: A (136) 28, B (272) 40).  Measured with 4096 features and k_in 4096 (us):
// 1024 rows A (128 workgroups) 48, B (256) 37; 1280 rows A (160) 50, B (320) 60; with 1024 features: 512 rows C 23, D 17.6;
// 2048 rows B (128) 38, C (256) 32, D (512) 43.
enum FewShape { FEW_A, FEW_B, FEW_C, FEW_D };
constexpr long long kFewWorkgroups = 160;

static FewShape few_shape(int M, const int* n, int count, int splits) {
    auto workgroups = [&](int bn, int bm) {
        long long t = 0;
        for (int i = 0; i < count; ++i) t += (n[i] + bn - 1) / bn;
        return t * ((M + bm - 1) / bm) * splits;
    };
    if (workgroups(256, 128) >= kFewWorkgroups || workgroups(128, 128) > cu_count()) return FEW_A;
    if (workgroups(128, 128) >= kFewWorkgroups) return FEW_B;
    if (workgroups(128, 64) >= kFewWorkgroups) return FEW_C;
    return FEW_D;
}

bool few_rows(int m, int n) { return few_rows(m, n, cu_count()); }

// The most rows up to m that few_rows takes.
int few_rows_most(int m, int n) {
    return (int)std::min<long long>({m, (1ll << 23) / n, cu_count() / ((n + 255ll) / 256) * 128});
}

template <int TW, int TA, int WGN, int WGM, int NS>
static int launch_split_shape(const bf16_t* A, int lda, const SplitMats& mats, int M, int K, int splits, float* partial, hipStream_t st) {
    constexpr int BN = 32 * TW * WGN, BM = 32 * TA * WGM;
    constexpr size_t stages = NS * (size_t)(BN + BM) * BK * 2, tile = (size_t)WGN * WGM * 32 * TW * 128;
    constexpr size_t smem = stages > tile ? stages : tile;
    auto kern = split_gemm_kernel<TW, TA, WGN, WGM, NS>;
    static std::once_flag attr_once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(attr_once, [&] { attr_err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem); });
    if (attr_err != hipSuccess) return set_hip_error(attr_err);
    SplitSegs s{};
    int tiles_n = 0, cols = 0;
    for (int i = 0; i < 3; ++i) {
        s.tile0[i] = i < mats.count ? tiles_n : 1 << 30;
        s.col0[i] = cols;
        if (i >= mats.count) continue;
        s.w[i] = (const bf16_t*)mats.w[i];
        s.n[i] = mats.n[i];
        tiles_n += (mats.n[i] + BN - 1) / BN;
        cols += mats.n[i];
    }
    s.ldp = cols;
    const int tiles_m = (M + BM - 1) / BM;
    hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n * splits), dim3(64 * WGN * WGM), smem, st, A, lda, s, partial, M, K, tiles_m,
                       tiles_n, splits);
    return check_launch();
}

int launch_split_gemm_large(const void* a, int lda, const void* w, int m, int n, int k_in, int splits, float* partial, hipStream_t st) {
    static std::once_flag attr_once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(attr_once, [&] {
        attr_err = hipFuncSetAttribute((const void*)split_gemm_large_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kRingBytes);
    });
    if (attr_err != hipSuccess) return set_hip_error(attr_err);
    const int tiles_m = (m + 255) / 256, tiles_n = (n + 255) / 256;
    hipLaunchKernelGGL(split_gemm_large_kernel, dim3(tiles_m * tiles_n * splits), dim3(256), kRingBytes, st, (const bf16_t*)a, lda, (const bf16_t*)w,
                       partial, m, n, k_in, tiles_m, tiles_n, splits);
    return check_launch();
}

int launch_split_gemm(const void* a, int lda, const SplitMats& mats, int m, int k_in, int splits, float* partial, hipStream_t st) {
    const bf16_t* A = (const bf16_t*)a;
    switch (few_shape(m, mats.n, mats.count, splits)) {
        case FEW_A: return launch_split_shape<2, 2, 4, 2, 3>(A, lda, mats, m, k_in, splits, partial, st);
        case FEW_B: return launch_split_shape<2, 2, 2, 2, 4>(A, lda, mats, m, k_in, splits, partial, st);
        case FEW_C: return launch_split_shape<2, 1, 2, 2, 3>(A, lda, mats, m, k_in, splits, partial, st);
        default: return launch_split_shape<1, 1, 2, 2, 5>(A, lda, mats, m, k_in, splits, partial, st);
    }
}

// Rows per launch of a residual projection with long rows (down projection): one round of 256 x 256 tiles, if its rows of A stay in the
// memory-side cache and it fills the chip.  As one launch the tiles of all rows drift apart, the rows come from HBM once per
// group of feature tiles, and the last round is as long as a full one.  4-wave tiles, one launch / rounds (us): 4096 features from 14336, 6000 rows 476 / 507, 8192 612 /
// 610, 9856 786 / 797, 16384 1394 / 1229, 32768 2647 / 2455; 3584 from 18944 (rounds of 4608 rows, 167 MB), 6000 rows 618 / 636, 9216 831 / 817, 12288 1188 / 1181.
// With rows of 4096 the same cut is 4 % slower at 9856 rows, so it is not made there.
static int residual_round_rows(const void* R, int N, int K, int ldo) {
    if (K <= 8192 || N % 256 != 0 || ldo % 8 != 0 || ((uintptr_t)R & 15)) return 0;
    const int tiles_n = N / 256, tm = cu_count() / tiles_n;
    return tm * tiles_n * 100 >= 92 * cu_count() && (size_t)tm * 256 * K * sizeof(bf16_t) <= kResidualCacheBytes ? tm * 256 : 0;
}

// How launch_linear's residual projection of m rows is cut when its caller has room for float partial sums: `whole` rows in full rounds,
// the others split over `splits` workgroups per tile (1: not at all, launch_linear takes all rows; !large: split_gemm_kernel's tiles).
// Whole layers (us).  Up to 512 rows the few-row tiles, 1 / 2 / 4 / 8 splits and 8 in large tiles: 4096 features from 14336, 64 rows 164 / 136 / 124 / 124, 137, 128 rows 182 / 157 / 153 / 149,
// 160, 200 rows 190 / 194 / 182 / 186, 192, 300 rows 266 / 225 / 221 / 233, 224, 512 rows 297 / 268 / 259 / 273, 258; 3584 from 18944, 128 rows 224 / 188 / 183 / 177, 190, 300 rows
// 302 / 262 / 257 / 267, 252, 512 rows 372 / 334 / 318 / 330, 311.  Behind them large tiles, not split / 4 splits of few-row tiles / split in large ones: 600 rows, 5 splits 368 / 354 / 320,
// 768, 5 407 / 388 / 356, 1024, 4 459 / 449 / 423, 1280, 3 585 / 577 / 522, 1511, 2 653 / 662 / 627, 1664, 2 671 / 703 / 645; 3584 from 18944, 600 rows, 4 425 / 375 / 359, 1024, 4
// 544 / 523 / 485, 1500, 3 758 / 753 / 698.  One round of workgroups; or 3 splits that make 1.64 rounds and more, of two.  Not split / split: 2 splits 1904 rows 799 / 780,
// 2048 (128 tiles) 830 / 804, 2300 rows of 18944 1000 / 971; 3 splits 2200 rows 920 / 899, 2304 (144 tiles) 921 / 902, of 18944 2560 rows (140 tiles) 1120 / 1088, 2816 1236 / 1196,
// 3072 1321 / 1263.  Not with 176 tiles (2600 rows 1070 / 1121) or with 2 splits of more than a round (2200 rows 950).
static int large_splits(long long tiles_m, int n) {      // for so many 256-row tiles; 1: none
    const long long tiles = tiles_m * ((n + 255) / 256), cu = cu_count();
    long long s = 1;
    if (tiles * 2 <= cu) s = std::min<long long>(8, cu / tiles);
    else if (3 * tiles <= 2 * cu && 3 * tiles * 100 >= 164 * cu) s = 3;
    return 2 * tiles * s < cu ? 1 : (int)s;              // (narrow outputs leave the large tiles' launch half empty)
}

ResidualCut residual_cut(int m, int n, int k_in) {
    ResidualCut c{0, 1, false};
    if (k_in < 8192 || k_in % BK != 0 || k_in >= (1 << 23) || n % 4 != 0) return c;
    if (m <= 1024 && few_rows(m, n)) c.splits = m <= 128 ? 8 : 4;
    if (m <= 512) return c;
    const int round = residual_round_rows(nullptr, n, k_in, n);
    const int whole = round && m > round ? m / round * round : 0, tail = m - whole;
    if (tail <= 128) return c;
    const int s = large_splits((tail + 255) / 256, n);
    if (s < 2) return c;
    c.whole = whole;
    c.splits = s;
    c.large = true;
    return c;
}

// The most floats that residual_cut has its caller keep for any row count up to m.  Splits change only behind 128 rows, behind the last that
// few_rows takes, and from one count of 256-row tiles to the next; behind whole rounds the tails of one come back, from 129 rows on.
size_t residual_cut_partial_floats(int m, int n, int k_in) {
    size_t most = 0;                                     // rows times splits
    for (int rows : {128, 512, 768, few_rows_most(1024, n)}) {
        rows = std::min(rows, m);
        const ResidualCut c = residual_cut(rows, n, k_in);
        if (c.splits > 1 && !c.large) most = std::max(most, (size_t)c.splits * rows);
    }
    if (m <= 512 || residual_cut(128, n, k_in).splits < 2) return most * n;
    const int round = residual_round_rows(nullptr, n, k_in, n), tiles_n = (n + 255) / 256;
    const int last = round ? round / 256 : 2 * cu_count() / (3 * tiles_n);   // (more tiles have no splits)
    for (int t = 1; t <= last && 256 * (t - 1) < m; ++t) {
        const int first = std::min(256 * t, m), later = round ? std::min(256 * t, m - round) : 0;
        const int rows = std::max(first > 512 ? first : 0, later > std::max(128, 256 * (t - 1)) ? later : 0);
        const int s = rows ? large_splits(t, n) : 1;
        if (s > 1) most = std::max(most, (size_t)s * rows);
    }
    return most * n;
}

template <int EPI>
static int dispatch_bf16(const bf16_t* A, int lda, const bf16_t* W0, const bf16_t* W1, const bf16_t* R, bf16_t* C,
                         int ldo, int M, int N, int K, hipStream_t st, const EpiExtra& re = EpiExtra()) {
    if constexpr (EPI != EPI_ROPE) {                     // (row_scale and RoPE callers have checked K % 64 == 0)
        if (K % BK != 0) return launch_bf16<2, 2, 2, 2, EPI, true>(A, lda, W0, W1, R, C, ldo, M, N, K, st);
    }
    if ((size_t)K >= (1u << 23) || (size_t)lda >= (1u << 23)) {   // 32-bit byte offsets inside a tile of 256 rows
        if constexpr (EPI == EPI_ROPE) return SLIM_UNSUPPORTED;
        else if (!re.row_scale && !re.w_2) return launch_bf16<2, 2, 2, 2, EPI, true>(A, lda, W0, W1, R, C, ldo, M, N, K, st);
        else return SLIM_UNSUPPORTED;
    }
    if constexpr (EPI == EPI_RESIDUAL) {
        const int round = residual_round_rows(R, N, K, ldo);
        for (; round && M > round; M -= round, A += (size_t)round * lda, R += (size_t)round * ldo, C += (size_t)round * ldo) {
            const int rc = launch_two_size<EPI>(A, lda, W0, W1, R, C, ldo, round, N, K, round / 256, false, st, re);
            if (rc) return rc;
        }
    }
    if constexpr (EPI == EPI_SWIGLU) {
        // Up to 256 rows the launch streams the weights: 64-feature tiles keep more of it in flight.  A second round of
        // them, one to a CU, costs more than it saves: with two stages two fit a CU, and the two-size launch takes more than 128 rows.  From three rounds on it
        // does not.  us, 64-feature tiles / two-size launch, weights again and again from the memory-side cache: 14336 features, 64 rows 36 / 39, 128 rows 37 / 42,
        // 200 rows 58 / 47, 300 rows 100 / 81; 18944 features, 200 rows 94 / 68; 36864 features (from HBM), 64 rows 136 / 159, 200 rows 180 / 191.
        const int tiles = (N + 63) / 64;
        const bool second_round = tiles > cu_count() && tiles <= 2 * cu_count();
        if (M <= 128 && second_round) return launch_bf16<1, 1, 2, 4, EPI, false, 2>(A, lda, W0, W1, R, C, ldo, M, N, K, st, re);
        if (M <= 128) return launch_bf16<1, 1, 2, 4, EPI, false, 4>(A, lda, W0, W1, R, C, ldo, M, N, K, st, re);
        if (M <= 256 && !second_round) return launch_bf16<1, 2, 2, 4, EPI, false, 3>(A, lda, W0, W1, R, C, ldo, M, N, K, st, re);
    } else if constexpr (EPI == EPI_ROPE) {
        if (M <= 128) return launch_bf16<4, 1, 2, 4, EPI, false>(A, lda, W0, W1, R, C, ldo, M, N, K, st, re);
    } else if (in_few_row_tiles(M, N, K, ldo, EPI == EPI_RESIDUAL, EPI == EPI_RESIDUAL && residual_in_four_waves(R, M, N, K, ldo), cu_count())) {
        switch (few_shape(M, &N, 1, 1)) {
            case FEW_A: return launch_bf16<2, 2, 4, 2, EPI, false, 3>(A, lda, W0, W1, R, C, ldo, M, N, K, st, re);
            case FEW_B: return launch_bf16<2, 2, 2, 2, EPI, false, 4>(A, lda, W0, W1, R, C, ldo, M, N, K, st, re);
            case FEW_C:
                // A workgroup that has its CU for itself takes a k-tile's loads at once, two that share it deal them to the k-steps.  us, at once / dealt: 1500 x 1024 from
                // 4096 (192 workgroups) 20.8 / 21.7, from 14336 86.3 / 87.7, 2048 x 1024 from 4096 (256) 24.3 / 25.1, 257 x 4096 from 14336 (160) 92.1 / 94.0; 2200 x 1024
                // from 4096 (280) 35.6 / 34.5, 1100 x 2048 from 1024 (288) 14.1 / 12.9.
                if ((M + 63ll) / 64 * ((N + 127ll) / 128) <= cu_count()) return launch_bf16<2, 1, 2, 2, EPI, false, 3, false>(A, lda, W0, W1, R, C, ldo, M, N, K, st, re);
                return launch_bf16<2, 1, 2, 2, EPI, false, 3>(A, lda, W0, W1, R, C, ldo, M, N, K, st, re);
            default: return launch_bf16<1, 1, 2, 2, EPI, false, 5>(A, lda, W0, W1, R, C, ldo, M, N, K, st, re);
        }
    }
    const int tiles_n = (N + TileShapes<EPI>::BN - 1) / TileShapes<EPI>::BN;
    const bool eight = EPI == EPI_RESIDUAL && !residual_in_four_waves(R, M, N, K, ldo);
    return launch_two_size<EPI>(A, lda, W0, W1, R, C, ldo, M, N, K,
                                plan_big_tiles(M, tiles_n, cu_count(), small_tile_cost<EPI>(eight), eight), eight, st, re);
}

// Query/Key projection with the RoPE epilogue (bf16, heads of 128, k_in a multiple of 64; checked by the caller).
// row_scale != null: the rows of a are the raw residual stream and row_scale their 1/rms (fused RMSNorm).
int launch_linear_rope(const void* a, int lda, const void* w, const void* bias, const float* table, const float* qt,
                       float* token_scores, const float* row_scale, int m, int n_heads, int k_in, int ldo, void* out,
                       hipStream_t st) {
    EpiExtra re;
    re.table = table;
    re.qt = qt;
    re.token_scores = token_scores;
    re.row_scale = row_scale;
    return dispatch_bf16<EPI_ROPE>((const bf16_t*)a, lda, (const bf16_t*)w, nullptr, (const bf16_t*)bias, (bf16_t*)out, ldo, m,
                                   n_heads * 128, k_in, st, re);
}

// Projection of row-scaled activations: plain, + bias, or SwiGLU (w1).  bf16, k_in a multiple of 64 (checked by
// the caller).
int launch_linear_scaled(const void* a, int lda, const void* w0, const void* w1, const void* bias, const float* row_scale,
                         int m, int n_out, int k_in, int ldo, void* out, hipStream_t st) {
    EpiExtra re;
    re.row_scale = row_scale;
    const bf16_t *A = (const bf16_t*)a, *W0 = (const bf16_t*)w0, *W1 = (const bf16_t*)w1, *B = (const bf16_t*)bias;
    bf16_t* C = (bf16_t*)out;
    if (w1) return dispatch_bf16<EPI_SWIGLU>(A, lda, W0, W1, nullptr, C, ldo, m, n_out, k_in, st, re);
    if (bias) return dispatch_bf16<EPI_BIAS>(A, lda, W0, nullptr, B, C, ldo, m, n_out, k_in, st, re);
    return dispatch_bf16<EPI_PLAIN>(A, lda, W0, nullptr, nullptr, C, ldo, m, n_out, k_in, st, re);
}

// Two projections of the same rows in one launch (the Query and Value projections of the continuing tokens): the
// second one's feature tiles follow the first one's, so the launch fills the chip as one problem of n_1 + n_2
// features.  Both with a bias or both without.  bf16, k_in % 64 == 0, m > 128 (checked by the caller).
int launch_linear_pair(const void* a, int lda, const void* w_1, const void* bias_1, int n_1, int ldo_1, void* out_1,
                       const void* w_2, const void* bias_2, int n_2, int ldo_2, void* out_2, const float* row_scale,
                       int m, int k_in, hipStream_t st) {
    EpiExtra re;
    re.row_scale = row_scale;
    re.w_2 = (const bf16_t*)w_2;
    re.r_2 = (const bf16_t*)bias_2;
    re.c_2 = (bf16_t*)out_2;
    re.n_2 = n_2;
    re.ldo_2 = ldo_2;
    const bf16_t *A = (const bf16_t*)a, *W = (const bf16_t*)w_1, *B = (const bf16_t*)bias_1;
    if (bias_1) {
        using S = TileShapes<EPI_BIAS>;
        re.tiles_n1 = (n_1 + S::BN - 1) / S::BN;
        const int tiles_n = re.tiles_n1 + (n_2 + S::BN - 1) / S::BN;
        return launch_two_size<EPI_BIAS>(A, lda, W, nullptr, B, (bf16_t*)out_1, ldo_1, m, n_1, k_in,
                                         plan_big_tiles(m, tiles_n, cu_count(), small_tile_cost<EPI_BIAS>(false), false),
                                         false, st, re);
    }
    using S = TileShapes<EPI_PLAIN>;
    re.tiles_n1 = (n_1 + S::BN - 1) / S::BN;
    const int tiles_n = re.tiles_n1 + (n_2 + S::BN - 1) / S::BN;
    return launch_two_size<EPI_PLAIN>(A, lda, W, nullptr, nullptr, (bf16_t*)out_1, ldo_1, m, n_1, k_in,
                                      plan_big_tiles(m, tiles_n, cu_count(), small_tile_cost<EPI_PLAIN>(false), false),
                                      false, st, re);
}

// Whether the Keys of m rows go into the launch of the Queries and Values (gemm_bf16_qkv_kernel).  The model says how many tile times
// they add to it; a launch of their own takes about 1.25 rounds of their tiles and a fifth of a tile time.  Measured on a layer with nothing
// dropped (us saved; predicted tile times saved): 16 + 4 + 4 feature tiles: 2048 rows 25; 0.36, 2983 -2; 0.00, 4096 24; 0.27, 5000 80; 0.39, 6000 10; 0.17,
// 8192 45; 0.38, 12000 43; 0.29; 14 + 2 + 2: 2048 -4; -0.15, 3500 18; 0.30, 4096 -24; -0.10, 8192 -23; 0.07.
bool qkv_together(int m, int n_q, int n_k, int n_v) {
    if (m > 16384) return false;                         // many rounds either way
    const int bn = TileShapes<EPI_PLAIN>::BN, tk = (n_k + bn - 1) / bn, tqv = (n_q + bn - 1) / bn + (n_v + bn - 1) / bn;
    double pair = 0.0, all = 0.0;
    plan_big_tiles(m, tqv, cu_count(), small_tile_cost<EPI_PLAIN>(false), false, &pair);
    plan_big_tiles(m, tqv + tk, cu_count(), small_tile_cost<EPI_PLAIN>(false), false, &all);
    return 1.25 * tk * m / 256.0 / cu_count() + 0.2 - (all - pair) > 0.12;
}

template <int EPI>
static int launch_qkv_t(const bf16_t* A, int lda, const bf16_t* W, const bf16_t* B, bf16_t* C, int n_q, int m, int k_in, EpiExtra& re, hipStream_t st) {
    using S = TileShapes<EPI>;
    auto kern = gemm_bf16_qkv_kernel<EPI>;
    static std::once_flag attr_once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(attr_once, [&] { attr_err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kRingBytes); });
    if (attr_err != hipSuccess) return set_hip_error(attr_err);
    re.tiles_nk = (re.n_k + S::BN - 1) / S::BN;
    re.tiles_n1 = (n_q + S::BN - 1) / S::BN;
    const int tiles_n = re.tiles_nk + re.tiles_n1 + (re.n_2 + S::BN - 1) / S::BN;
    const int big = plan_big_tiles(m, tiles_n, cu_count(), small_tile_cost<EPI>(false), false);
    const int small = std::max(0, m - big * S::BM_BIG + S::BM_SMALL - 1) / S::BM_SMALL;
    hipLaunchKernelGGL(kern, dim3((big + small) * tiles_n), dim3(256), kRingBytes, st, A, lda, W, B, C, n_q, m, n_q, k_in, big, small, tiles_n, re);
    return check_launch();
}

// Query (not rotated), Key (rotated with the table) and Value projections of the same rows, each [m, n_*] contiguous.  bias_q and bias_v both or
// neither.  bf16, n_k a multiple of 128, the others of 8, k_in % 64 == 0 and below 2^23, 16-byte aligned (checked by the caller).
int launch_linear_qkv(const void* a, int lda, const void* w_q, const void* bias_q, int n_q, void* out_q, const void* w_k, const void* bias_k,
                      int n_k, const float* table, void* out_k, const void* w_v, const void* bias_v, int n_v, void* out_v,
                      const float* row_scale, int m, int k_in, hipStream_t st) {
    EpiExtra re;
    re.table = table;
    re.row_scale = row_scale;
    re.w_2 = (const bf16_t*)w_v;
    re.r_2 = (const bf16_t*)bias_v;
    re.c_2 = (bf16_t*)out_v;
    re.n_2 = re.ldo_2 = n_v;
    re.w_k = (const bf16_t*)w_k;
    re.r_k = (const bf16_t*)bias_k;
    re.c_k = (bf16_t*)out_k;
    re.n_k = n_k;
    const bf16_t *A = (const bf16_t*)a, *W = (const bf16_t*)w_q, *B = (const bf16_t*)bias_q;
    if (bias_q) return launch_qkv_t<EPI_BIAS>(A, lda, W, B, (bf16_t*)out_q, n_q, m, k_in, re, st);
    return launch_qkv_t<EPI_PLAIN>(A, lda, W, nullptr, (bf16_t*)out_q, n_q, m, k_in, re, st);
}

// At most one of w1 (SwiGLU), residual and bias is set.
int launch_linear(const void* a, int lda, const void* w0, const void* w1, const void* residual, const void* bias,
                  int m, int n_out, int k_in, int ldo, int dtype, void* out, hipStream_t st) {
    if (dtype == SLIM_F32) {
        const F32Seg seg{(const float*)a, lda, m, (const float*)w0, (const float*)w1, (const float*)bias, (const float*)residual,
                         (float*)out, ldo, n_out, w1 ? F32_SWIGLU : F32_PLAIN, nullptr, 0};
        return launch_f32_linear(&seg, 1, k_in, nullptr, 0.f, 0, 0.f, st);
    }
    const bf16_t *A = (const bf16_t*)a, *W0 = (const bf16_t*)w0, *W1 = (const bf16_t*)w1, *R = (const bf16_t*)residual;
    bf16_t* C = (bf16_t*)out;
    if (w1) return dispatch_bf16<EPI_SWIGLU>(A, lda, W0, W1, R, C, ldo, m, n_out, k_in, st);
    if (residual) return dispatch_bf16<EPI_RESIDUAL>(A, lda, W0, W1, R, C, ldo, m, n_out, k_in, st);
    if (bias) return dispatch_bf16<EPI_BIAS>(A, lda, W0, W1, (const bf16_t*)bias, C, ldo, m, n_out, k_in, st);
    return dispatch_bf16<EPI_PLAIN>(A, lda, W0, W1, R, C, ldo, m, n_out, k_in, st);
}

}  // namespace slim
