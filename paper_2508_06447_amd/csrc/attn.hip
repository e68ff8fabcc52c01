// Causal grouped-query prefill attention ("Attention" stage of Fig. 2) over the compacted sequence.
//
// bf16 path (head_dim 128): flash-style single pass with online softmax, v_mfma_f32_32x32x16_bf16.
// A workgroup of 4 waves (one per SIMD) owns 256 queries of one head, each wave 64 of them as two 32-query
// sub-tiles that share every K and V^T fragment read from LDS.  K/V tiles of 128 keys go from global memory
// straight into LDS (global_load_lds_dwordx4), both row-major, two stages (2 x 64 KB); V fragments are read
// with the transposing LDS read (ds_read_b64_tr_b16).
//
// Both products are computed transposed so that no register shuffle is needed between them:
//   S^T[key, query] = K . Q^T      (A operand = K rows from LDS, B operand = Q rows held in registers)
//   O^T[d,   query] = V^T . P^T    (A operand = V^T from LDS, B operand = P^T from the S^T
//                                   accumulators, converted to bf16)
// In the 32x32 accumulator layout a lane owns one query column, so the softmax statistics of a query
// live in two lanes (l and l^32).  The accumulator's row order (rows 8*(v/4) + 4*(lane/32) + v%4) is a
// permutation of the keys; the V^T fragments are read in the same permuted order, which leaves the
// contraction unchanged.
//
// Softmax: Q is pre-multiplied by scale*log2(e) (bf16), logits are kept relative to a per-query reference that
// enters through the S accumulators' initial value, so P = exp2(acc) with no multiply or subtract per element;
// the reference is the row maximum of the first 32 keys and moves only when the P of a later 32-key unit add up to
// more than 2^8 in some lane (a logit may then lie more than 8 above the reference; seen before those P are used:
// the reference moves up to the unit's maximum, O and the row sums are rescaled, the unit's P are formed again),
// so the result does not depend on it.  Row sums add the unrounded P.
//
// The kernel body (main loop, instruction order, register assignment: O accumulators and Q fragments in
// a0-a191, S tiles and everything the vector ALU touches in v0-v231) is the assembly that gen_attn_asm.py writes
// into attn_bf16_body.inc; the C++ below computes its per-lane and per-workgroup operands.
#include "slim_common.h"
#include "routes.h"
#include <mutex>
#include <type_traits>

namespace slim {

constexpr int AD = 128;          // head_dim of the MFMA path
constexpr int ANW = 4;           // waves per workgroup
constexpr int BQ = 64 * ANW;     // queries per workgroup
constexpr int BKV = 128;         // keys per tile
constexpr int NSTAGE = 2;        // K/V tiles resident in LDS
constexpr int TILE_BYTES = BKV * AD * 2;
constexpr int STAGE_BYTES = 2 * TILE_BYTES;             // K tile, then V tile

// Both tiles: row = key, 256 B = 16 chunks of 16 B.  K: chunk c of row r sits at slot c ^ (r & 15), so
// the 128-bit fragment reads (32 rows, one chunk column) are conflict-free.  V: slot c ^ (4 * (r & 3)),
// which spreads the 4 key rows x 4 chunks that one transposing read touches over all banks.
__device__ __forceinline__ int k_off(int r, int c) { return (r * 16 + (c ^ (r & 15))) * 16; }
__device__ __forceinline__ int v_off(int r, int c) { return (r * 16 + (c ^ ((r & 3) << 2))) * 16; }

// GROUPED (4 query heads per kv head): the four waves of a workgroup take the same 64 queries of the four heads
// that share a kv head, so all of them stop at the same diagonal and no wave runs units that are masked for it
// alone.  Otherwise the waves take 4 x 64 consecutive queries of one head.
template <bool GROUPED>
__global__ void __launch_bounds__(64 * ANW) __attribute__((amdgpu_waves_per_eu(1, 1)))
attn_bf16_kernel(const bf16_t* __restrict__ Q, const bf16_t* __restrict__ Kg, const bf16_t* __restrict__ Vg,
                 bf16_t* __restrict__ O, int n, int Hq, int Hkv, float scale_log2e, int n_qt) {
    extern __shared__ __align__(16) unsigned char lds[];
    // Workgroup -> (head, query tile).  Ids are dealt round-robin to the 8 XCDs and each XCD hands its
    // workgroups to its CUs in id order.  Give each XCD a contiguous range of heads, so the query heads
    // sharing a kv head meet in one L2, and walk that range's query tiles from the one with the most keys
    // down, all heads of the range at each size: longest-first order per XCD keeps its CUs evenly loaded.
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hh = lane >> 5;
    const int n_units = GROUPED ? Hkv : Hq;               // (kv heads | heads) that the grid walks per query tile
    int u, qt_idx;
    if (n_units % 8 == 0) {
        const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3, upx = n_units >> 3;
        u = xcd * upx + j % upx;
        qt_idx = n_qt - 1 - j / upx;
    } else {
        u = blockIdx.x % n_units;
        qt_idx = n_qt - 1 - blockIdx.x / n_units;
    }
    const int h = GROUPED ? u * 4 + wave : u;
    const int g = GROUPED ? u : h / (Hq / Hkv);
    constexpr int WGQ = GROUPED ? 64 : BQ;                // query rows per workgroup
    const int q0 = qt_idx * WGQ;
    const int qw0 = GROUPED ? q0 : q0 + wave * 64;        // first query of this wave
    const size_t qstride = (size_t)Hq * AD;
    const unsigned lds_base = (unsigned)(uintptr_t)lds;

    // LDS byte addresses of this lane's fragment reads for k-step 0 / d-tile 0 of stage 0; the others differ
    // by an XOR (k-step st: st << 5, d-tile dt: dt << 6, stage 1: 1 << 16) and an immediate offset per key row.
    // K fragment: row l32 of a 32-key sub-tile, chunk 2*st + hh.  V^T fragment (transposing read): in each group
    // of 16 lanes, lane s supplies the address of 4 consecutive d of key s/4 and receives, for d = D0 + s, the
    // 4 consecutive keys; lane groups 0/1 cover d 0-15 / 16-31, groups 2/3 the keys 4-7.
    const unsigned koff0 = lds_base + k_off(l32, hh);
    const int G4 = lane >> 4, sl = lane & 15;
    const int key_lane = 4 * (G4 >> 1) + (sl >> 2);
    const unsigned voff0 = lds_base + TILE_BYTES + v_off(key_lane, 2 * (G4 & 1) + ((sl & 3) >> 1)) + (sl & 1) * 8;
    // Tile loads: a wave-load moves 4 key rows x 256 B; wave-load i of this wave covers rows 16*i + r0 .., lane l
    // lands at LDS slot l%16 of row l/16 and fetches the global chunk that the swizzle assigns to that slot.
    const unsigned r0 = wave * 4 + (lane >> 4), slot = lane & 15;
    const unsigned kchunk = (slot ^ (r0 & 15)) * 16, vchunk = (slot ^ ((r0 & 3) << 2)) * 16;
    const int qi0 = qw0 + l32, qi1 = qw0 + 32 + l32;      // this lane's two queries
    const bf16_t* qrow0 = Q + (size_t)min(qi0, n - 1) * qstride + (size_t)h * AD + hh * 8;
    const bf16_t* qrow1 = Q + (size_t)min(qi1, n - 1) * qstride + (size_t)h * AD + hh * 8;
    bf16_t* orow0 = O + (size_t)qi0 * qstride + (size_t)h * AD + 4 * hh;     // written only when the query exists
    bf16_t* orow1 = O + (size_t)qi1 * qstride + (size_t)h * AD + 4 * hh;
    // causal / ragged mask: key k0 + ko of a unit is visible to the lane's accumulator row ko iff ko <= limabs - k0
    const int limabs0 = min(qi0, n - 1) - 4 * hh, limabs1 = min(qi1, n - 1) - 4 * hh;
    const unsigned valid0 = qi0 < n, valid1 = qi1 < n;

    const unsigned rowbytes = (unsigned)Hkv * AD * 2, tile_bytes = rowbytes * BKV;
    const unsigned last_tile = (n + BKV - 1) / BKV - 1;   // tiles past it re-read it (into a stage nobody reads)
    const unsigned nl = n - last_tile * BKV, nl1 = nl - 1; // rows of the last tile; its loads clamp their rows to nl1
    const unsigned last_ragged = nl != BKV ? last_tile : 0xffffffffu;
    const int last_q = min(q0 + WGQ, n) - 1;
    const unsigned nkt = last_q / BKV + 1;                // causal: tiles up to the last query's diagonal
    const unsigned nmain = nkt > 3 ? nkt - 3 : 0;         // tiles that need no mask
    const uint64_t kb = (uint64_t)(uintptr_t)(Kg + (size_t)g * AD), vb = (uint64_t)(uintptr_t)(Vg + (size_t)g * AD);
    const unsigned kbase_lo = (unsigned)kb, kbase_hi = (unsigned)(kb >> 32);
    const unsigned vbase_lo = (unsigned)vb, vbase_hi = (unsigned)(vb >> 32);
    const unsigned ldsw = lds_base + wave * 1024;

    asm volatile(
#include "attn_bf16_body.inc"
        :
        : [koff0] "v"(koff0), [voff0] "v"(voff0), [r0] "v"(r0), [kchunk] "v"(kchunk), [vchunk] "v"(vchunk),
          [qrow0] "v"(qrow0), [qrow1] "v"(qrow1), [orow0] "v"(orow0), [orow1] "v"(orow1),
          [limabs0] "v"(limabs0), [limabs1] "v"(limabs1), [valid0] "v"(valid0), [valid1] "v"(valid1),
          [kbase_lo] "s"(kbase_lo), [kbase_hi] "s"(kbase_hi), [vbase_lo] "s"(vbase_lo), [vbase_hi] "s"(vbase_hi),
          [nkt] "s"(nkt), [nmain] "s"(nmain), [last_tile] "s"(last_tile), [last_ragged] "s"(last_ragged),
          [rowbytes] "s"(rowbytes), [tile_bytes] "s"(tile_bytes), [scale] "s"(scale_log2e), [nl1] "s"(nl1),
          [ldsw] "s"(ldsw), [qw0] "s"(qw0)
        :
#include "attn_bf16_clobbers.inc"
    );
}

// Few rows: the kernel above takes 2.5 us for a tile of 128 keys whatever the number of workgroups, and up to 2048 rows of 8 kv heads its launch is as long as its query
// tile with the most keys.  Here a workgroup owns 32 queries of four heads of a kv group and deals the keys to two waves per head (wave = key half * 4 + head, two waves
// per SIMD): tiles of 64 keys in four LDS stages of 32 KB, one barrier each (0.9 us a tile; its MFMAs alone 0.62 at the clock that they run at), and at the end the two
// waves of a head swap halves of O through LDS.  Same products, layouts and kind of reference as above, but Q stays as it is and scale * log2(e) enters in float (error of
// 1000 rows against float64 3.6e-3 -> 2.1e-3).  32 / 8 heads, us, the kernel above / this one: 128 rows 11.6 / 8.6, 512 19.1 / 14.1, 1024 27.9 / 21.6, 1511 37.4 / 30.8.
// S(t + 1) formed under the softmax of tile t, the two key halves in opposite phases, QK and PV MFMAs in turn, the reference tested on sums: within 3 %, none faster.
constexpr int FKV = 64;                                 // keys per tile, 32 per wave
constexpr int FSTAGES = 4;
constexpr int FTILE_BYTES = FKV * AD * 2, FSTAGE_BYTES = 2 * FTILE_BYTES;
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
attn_bf16_few_kernel(const bf16_t* __restrict__ Q, const bf16_t* __restrict__ Kg, const bf16_t* __restrict__ Vg, bf16_t* __restrict__ O, int n, int Hq, int Hkv,
                     float c, int n_qt) {
    extern __shared__ __align__(16) unsigned char lds[];
    typedef __attribute__((address_space(3))) bf16x4* LdsB64;
    typedef __attribute__((address_space(3))) bf16x8* LdsB128;
    typedef __attribute__((address_space(3))) f32x4* LdsF32x4;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), half = wave >> 2;
    // Workgroup -> (four heads of a kv group, query tile): as above, longest first inside each XCD.
    const int G = Hq / Hkv, chunks = (G + 3) / 4, n_units = Hkv * chunks;
    int u, qt;
    if (n_units % 8 == 0) {
        const int j = blockIdx.x >> 3, upx = n_units >> 3;
        u = (blockIdx.x & 7) * upx + j % upx;
        qt = n_qt - 1 - j / upx;
    } else {
        u = blockIdx.x % n_units;
        qt = n_qt - 1 - blockIdx.x / n_units;
    }
    const int g = u / chunks, hg = (u - g * chunks) * 4 + (wave & 3);
    const int h = g * G + min(hg, G - 1);               // (a wave without a head of its own repeats the last one and stores nothing)
    const int q0 = qt * 32, qi = q0 + l32, lim = min(qi, n - 1), q_last = min(q0 + 31, n - 1);
    const int nkt = q_last / FKV + 1;
    const size_t qstride = (size_t)Hq * AD;
    const unsigned lds_base = (unsigned)(uintptr_t)lds, rowbytes = (unsigned)Hkv * AD * 2;

    bf16x8 qf[8];
    const bf16_t* qrow = Q + (size_t)lim * qstride + (size_t)h * AD + hh * 8;
#pragma unroll
    for (int st = 0; st < 8; ++st) qf[st] = *reinterpret_cast<const bf16x8*>(qrow + st * 16);

    // Wave-load i moves rows 4 * (8 i + wave) .. + 3 of a tile, 256 B each, with the swizzles of k_off and v_off.  Rows behind the last key repeat it (masked), tiles behind
    // the last one are it again, in a stage that nobody reads: the number of loads in flight is a constant.
    const unsigned char* kbase = reinterpret_cast<const unsigned char*>(Kg + (size_t)g * AD);
    const unsigned char* vbase = reinterpret_cast<const unsigned char*>(Vg + (size_t)g * AD);
    auto issue = [&](int t) {
        const int k0 = min(t, nkt - 1) * FKV;
        const unsigned dst = lds_base + (t % FSTAGES) * FSTAGE_BYTES + wave * 1024;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = 4 * (8 * i + wave) + (lane >> 4), slot = lane & 15;
            const unsigned row = (unsigned)min(r, n - 1 - k0) * rowbytes;
            load_global_to_lds16(kbase + (size_t)k0 * rowbytes, row + ((slot ^ (r & 15)) << 4), dst + i * 8192);
            load_global_to_lds16(vbase + (size_t)k0 * rowbytes, row + ((slot ^ ((r & 3) << 2)) << 4), dst + FTILE_BYTES + i * 8192);
        }
    };
    for (int t = 0; t < FSTAGES - 1; ++t) issue(t);

    const int G4 = lane >> 4, sl = lane & 15, key_lane = 32 * half + 4 * (G4 >> 1) + (sl >> 2);
    const unsigned koff = lds_base + k_off(32 * half + l32, hh);
    const unsigned voff = lds_base + FTILE_BYTES + v_off(key_lane, 2 * (G4 & 1) + ((sl & 3) >> 1)) + (sl & 1) * 8;
    f32x16 o[4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[dt][v] = 0.f;
    const float step = 8.f / c;                          // how far a logit may lie above the reference: P up to 2^8
    float m = -INFINITY, m_step = -INFINITY, nmc = 0.f, l = 0.f;     // reference, reference + step, -reference * c (0: none yet), the lane's sum of P
    for (int t = 0; t < nkt; ++t) {
        __builtin_amdgcn_s_waitcnt(0x0070 | 4 * (FSTAGES - 2));      // own part of tile t is there, own reads of tile t - 1 are done
        workgroup_barrier();
        issue(t + FSTAGES - 1);                          // into the stage of tile t - 1
        const int k0 = t * FKV + 32 * half;
        if (k0 > q_last) continue;
        const unsigned so = (t % FSTAGES) * FSTAGE_BYTES;
        bf16x8 kf[8], vf[2][4];
#pragma unroll
        for (int st = 0; st < 8; ++st) kf[st] = *(LdsB128)((koff + so) ^ (st << 5));
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int dt = 0; dt < 4; ++dt) {
                const unsigned a = ((voff + so) ^ (dt << 6)) + ks * 16 * AD * 2;
                const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LdsB64)a), hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LdsB64)(a + 8 * AD * 2));
                vf[ks][dt] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            }
        f32x16 s;
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] = 0.f;
#pragma unroll
        for (int st = 0; st < 8; ++st) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[st], qf[st], s, 0, 0, 0);
        if (k0 + 31 > q0)                                // keys above some query (or behind the last one)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (k0 + 8 * (v >> 2) + 4 * hh + (v & 3) > lim) s[v] = -INFINITY;
        float mx = s[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s[v]);
        if (__any(mx > m_step)) {                        // rare behind the first tile: the reference moves up to the maximum of both lanes of a query
            mx = fmaxf(mx, m);
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            const float f = m == mx ? 1.f : __builtin_amdgcn_exp2f((m - mx) * c);
            m = mx;
            m_step = m + step;
            nmc = m == -INFINITY ? 0.f : -m * c;
            l *= f;
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[dt][v] *= f;
        }
        float sum[2] = {0.f, 0.f};
        bf16x8 pb[2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            float p[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                p[e] = __builtin_amdgcn_exp2f(fmaf(s[8 * ks + e], c, nmc));
                sum[e & 1] += p[e];
            }
            pb[ks] = __builtin_bit_cast(bf16x8, Elem<bf16_t>::pack(p));
        }
        l += sum[0] + sum[1];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int dt = 0; dt < 4; ++dt) o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[ks][dt], pb[ks], o[dt], 0, 0, 0);
    }
    l += __shfl_xor(l, 32, 64);
    // The two waves of a head: each sends the half of O that the other finishes, with its reference and sum.  All loads into LDS are through.
    __builtin_amdgcn_s_waitcnt(0x0070);
    workgroup_barrier();
    const unsigned mine = lds_base + wave * 8192 + lane * 16, theirs = lds_base + (wave ^ 4) * 8192 + lane * 16;
    const unsigned stat = lds_base + 65536 + lane * 16;
    auto send = [&](auto first) {
        constexpr int F = decltype(first)::value;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const f32x16& a = o[F + (i >> 2)];
            *(LdsF32x4)(mine + i * 1024) = f32x4{a[4 * (i & 3)], a[4 * (i & 3) + 1], a[4 * (i & 3) + 2], a[4 * (i & 3) + 3]};
        }
    };
    if (half) send(std::integral_constant<int, 0>{});
    else send(std::integral_constant<int, 2>{});
    *(LdsF32x4)(stat + wave * 1024) = f32x4{m, l, 0.f, 0.f};
    __syncthreads();
    const f32x4 other = *(LdsF32x4)(stat + (wave ^ 4) * 1024);
    const float top = fmaxf(m, other[0]);
    const float f0 = m == top ? 1.f : __builtin_amdgcn_exp2f((m - top) * c), f1 = other[0] == top ? 1.f : __builtin_amdgcn_exp2f((other[0] - top) * c);
    const float inv = 1.f / (l * f0 + other[1] * f1), w0 = f0 * inv, w1 = f1 * inv;
    auto finish = [&](auto first) {
        constexpr int F = decltype(first)::value;
        bf16_t* orow = O + (size_t)qi * qstride + (size_t)h * AD + F * 32 + 4 * hh;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const f32x16& a = o[F + (i >> 2)];
            const f32x4 b = *(LdsF32x4)(theirs + i * 1024);
            float r[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) r[e] = a[4 * (i & 3) + e] * w0 + b[e] * w1;
            if (qi < n && hg < G) *reinterpret_cast<uint2*>(orow + (i >> 2) * 32 + (i & 3) * 8) = make_uint2(pack_bf16x2(r[0], r[1]), pack_bf16x2(r[2], r[3]));
        }
    };
    if (half) finish(std::integral_constant<int, 2>{});
    else finish(std::integral_constant<int, 0>{});
}

int launch_attn(const void* q, const void* k, const void* v, int n, int Hq, int Hkv, int d, float scale,
                int dtype, void* out, hipStream_t st) {
    if (scale == 0.f) scale = 1.0f / sqrtf((float)d);
    if (dtype == SLIM_BF16) {
        // rowbytes and the 24-bit multiplies of the tile-load offsets bound the number of kv heads
        if ((long long)Hkv * AD * 2 * BKV >= (1ll << 31) || Hkv > 4096) return SLIM_UNSUPPORTED;
        const int smem = NSTAGE * STAGE_BYTES;
        static std::once_flag attr_once;
        static hipError_t attr_err = hipSuccess;
        std::call_once(attr_once, [&] {
            attr_err = hipFuncSetAttribute((const void*)attn_bf16_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
            if (attr_err == hipSuccess)
                attr_err = hipFuncSetAttribute((const void*)attn_bf16_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
            if (attr_err == hipSuccess)
                attr_err = hipFuncSetAttribute((const void*)attn_bf16_few_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, FSTAGES * FSTAGE_BYTES);
        });
        if (attr_err != hipSuccess) return set_hip_error(attr_err);
        if (few_row_attention(n, Hq, Hkv, scale, cu_count())) {
            const unsigned few_wgs = (unsigned)((n + 31ll) / 32 * Hkv * ((Hq / Hkv + 3) / 4));
            hipLaunchKernelGGL(attn_bf16_few_kernel, dim3(few_wgs), dim3(512), FSTAGES * FSTAGE_BYTES, st, (const bf16_t*)q, (const bf16_t*)k,
                               (const bf16_t*)v, (bf16_t*)out, n, Hq, Hkv, scale * 1.4426950408889634f, (n + 31) / 32);
        } else if (Hq == 4 * Hkv) {
            const int n_qt = (n + 63) / 64;
            hipLaunchKernelGGL(attn_bf16_kernel<true>, dim3(n_qt * Hkv), dim3(64 * ANW), smem, st, (const bf16_t*)q,
                               (const bf16_t*)k, (const bf16_t*)v, (bf16_t*)out, n, Hq, Hkv, scale * 1.4426950408889634f, n_qt);
        } else {
            const int n_qt = (n + BQ - 1) / BQ;
            hipLaunchKernelGGL(attn_bf16_kernel<false>, dim3(n_qt * Hq), dim3(64 * ANW), smem, st, (const bf16_t*)q,
                               (const bf16_t*)k, (const bf16_t*)v, (bf16_t*)out, n, Hq, Hkv, scale * 1.4426950408889634f, n_qt);
        }
        return check_launch();
    }
    return launch_f32_attn((const float*)q, (const float*)k, (const float*)v, n, Hq, Hkv, d, scale, (float*)out, st);
}

}  // namespace slim
