// Which of two kernels a call takes, where sizes decide (host code, no GPU).  cu: compute units of the device.
#pragma once

namespace slim {

// Up to how many outputs the few-row tiles are taken, and only where their 256 x 128 tiles are no more than a round.  us, weights from HBM, few-row / two-size: 4096
// features from 4096, 512 rows 31 / 53, 1024 39 / 54, 1280 to 1664 53 / 53, 2300 (288 tiles) 91 / 69; 5120 features, 1664 rows (260 tiles) 94 / 73; 1024 features, 3000 rows
// 28 / 38, 4096 33 / 38, 6000 47 / 42, 8192 57 / 67; 512 features from 3584, 12000 rows 41 / 59.
inline long long few_row_tiles(int m, int n) { return (m + 127ll) / 128 * ((n + 255ll) / 256); }
inline bool few_rows(int m, int n, int cu) { return (long long)m * n <= (1ll << 23) && few_row_tiles(m, n) <= cu; }

// Of these, the launches that the two-size tiles are faster at all the same: nearly a round of 256 x 128 tiles of a wide output.  us, few-row / two-size, with residual: 4096
// features from 4096, 1664 rows (208 tiles) 57 / 56, 1800 (240) 58 / 52, 2048 (256) 62 / 57, from 14336 2048 rows 199 / 190; 3584 from 3584, 1800 rows (210) 50 / 49, 2048 (224) 53 /
// 51, 2300 (252) 57 / 54; 5120 from 4096, 1511 rows (240) 57 / 54.  Short rows too (2048 x 4096 from 64 8.2 / 7.6, from 256 10.4 / 9.8).  Few rows
// of very wide outputs, without residual, gain less and within 215 tiles up to 3 % either way: 64 x 54016 (211) from 1024 24.2 / 24.9, 300 x 18000 (213) from 4096 69.3 / 70.2, 256 x 27136 (212) from 4096
// 79.2 / 76.0, 256 x 30720 (240) 76.1 / 72.2, 200 x 28672 (224) 69.7 / 66.3.
inline bool nearly_a_round(int m, int n, int cu) { return n >= 2048 && few_row_tiles(m, n) * 16 > cu * 13ll; }

// Whether a projection of m rows runs in the few-row tiles, which take any row stride of the output; the two-size launch takes those below 2^23.  four_waves: the
// residual would be added in that launch's four-wave tile.  Its eight-wave tile is the slower loop: with residual, us, few-row / eight waves: 4104 features from 4096, 1600 rows 59 / 79,
// from 14336 197 / 272; 2880 from 4096, 2300 rows 57 / 76; 2056 from 4096, 3000 rows 56 / 76; 4000 from 4096, 2048 rows 62 / 81; 12104 from
// 768, 640 rows 22.4 / 24.2, from 640 22.3 / 20.3; 4000 from 640, 2048 rows 23.5 / 18.8.
// Short rows with a residual are as fast or faster in the few-row tiles where these divide evenly over the XCDs and leave a sixteenth of the chip: 4096 features, 1665 rows (224 tiles)
// from 256 10.7 / 11.4, from 384 12.4 / 12.9, from 448 13.6 / 13.7, from 512 14.5 / 14.1; 8192, 896 rows (224) 11.2 / 11.7, 12.9 / 13.2, 13.5 / 13.4, 14.6 / 14.3; 9216, 768 rows (216)
// from 256 10.9 / 11.0; 2880, 2300 rows (216, eight waves) from 256 11.1 / 11.6, from 384 13.0 / 13.6.  Elsewhere they depend on where the buffers lie, 2048 x 4096 from 256 (256
// tiles) 11 to 17 / 12, from 512 14 to 20 / 15, and from 192 10 to 16 / 11 to 12; 5120, 1408 rows (220) from 256 14.0 / 12.0; 3840, 1920 rows (225) from 384 14 to 17 / 14.
inline bool in_few_row_tiles(int m, int n, int k, int ldo, bool residual, bool four_waves, int cu) {
    if (!few_rows(m, n, cu)) return false;
    bool leaves = nearly_a_round(m, n, cu) && ldo < 1 << 23;
    if (residual) {
        const bool even = few_row_tiles(m, n) % 8 == 0 && few_row_tiles(m, n) * 16 < cu * 15ll;
        leaves = leaves && k >= (even ? 448 : 256) && (four_waves || (!even && k <= 640));
    }
    return !leaves;
}

// Whether bf16 attention of n rows runs in the few-row kernel: groups whose heads fill three or four of a workgroup's four places, up to two workgroups per CU.  us, the other kernel / this
// one: 32 / 8 heads, 2048 rows 49.2 / 46.3, 2560 63 / 74; 28 / 4 heads 48.5 / 46.3, 62 / 74.  Behind one workgroup per CU only if the rows are long: with many units (four heads of a kv
// group) the second round starts again for a few tiles of keys.  16 units of 416 and 512 workgroups 1.12 and 1.02 times as fast as the other kernel, 24 of 384 1.00 to 1.06, of 480
// 0.92 to 0.97, 28 of 280 1.04 to 1.13, of 336 0.91 to 0.98, 48 of 288 to 384 0.90 to 1.01 (112 / 16 heads, 384 rows 16.7 / 18.7), unless the other kernel, which gives a head's 256 queries (a group of
// four: 64) a workgroup, begins a second round: 28 units of 476 1.43, 36 of 324 to 504 1.38 to 1.64, 96 of 288 1.21 to 1.30, groups of four 30 of 510 1.05, 56 of 504 1.28 (but 20
// to 22 of 500 0.97).  A reference in units of unscaled logits needs a positive scale.
inline bool few_row_attention(int n, int Hq, int Hkv, float scale, int cu) {
    const int group = Hq / Hkv, units = Hkv * ((group + 3) / 4);
    const long long workgroups = (n + 31ll) / 32 * units, others = group == 4 ? (n + 63ll) / 64 * Hkv : (n + 255ll) / 256 * Hq;
    if (group % 4 == 1 || group % 4 == 2 || !(scale > 0.f) || workgroups > 2ll * cu) return false;
    const int eighths = units <= 16 ? 16 : units <= 24 ? 12 : units <= 30 ? 9 : 8;       // of a round
    return 8 * workgroups <= (long long)eighths * cu || (others > cu && (group != 4 || units > 24));
}

// Whether a layer's compaction of n_keep of nb blocks, in `chunks` workgroups each, selects them itself (64 at most): every wave ranks the blocks for its own, one after another, where a launch in
// front takes two microseconds and more of the stream, so only where few waves do it.  Layers, us, selection in front / in the compaction: small float32 (chunks 6), 16 blocks 46.5 / 45.0, 32 51.7 /
// 50.7, 48 59.0 / 58.3, 56 60.5 / 60.5, 64 within 0.5 % either way; bf16 of 4096, blocks of 64 rows (161), 4 of 16 254.3 / 252.1, 8 of 16 (a product of 20608) 316.2 / 314.8, 16 of 32 (82432)
// 501.7 / 500.9, 24 of 48 (185472) 682 / 687; of 2048, blocks of 32, 12 of 24 (11808) 135.0 / 133.2, 16 of 32 (20992) 151.0 / 149.1, 24 of 48 (47232) 187.3 / 187.2, 32 of 64 (83968) 222.2 / 223.4.
inline bool compact_selects(long long chunks, int n_keep, int nb) { return nb <= 64 && chunks * n_keep * nb <= 64 * 256; }

// Splits of a layer's output projection of few rows (1: none), for which a finishing pass of rows of up to 8192 features takes the place of the norm's launch (with a gain, if that is 16-byte
// aligned).  Whole layers, not split / 2 / 4 / 8 splits (us): 4096 features from 4096, 4 rows 123.4 / 117.9 / 115.2 / 117.6, 64 147 / 140 / 137, 65 141.2 / 137.7 / 138.3, 128 156.3 / 151.0 /
// 151.9, 200 177 / 182 / 180, 256 201 / 200 / 199, 257 229 / 217 / 219 / 227, 512 261 / 254 / 254, 640 343 / 335, 768 375 / 369, 896 398 / 392, 1024 411 / 406, 1511 603 / 620; 3584 from 3584,
// 48 rows 153 / 146 / 143 / 148, 128 186 / 180 / 181, 300 256 / 253 / 254, 512 316 / 311 / 311, 768 395 / 389, 819 439 / 442, 896 448 / 448, 1024 485 / 478; 2048, 512 rows 116 / 115, 819
// 156 / 153, 1024 171 / 171; 5120, 384 rows 309 / 299, 768 481 / 471, 819 558 / 553; 8192, 64 rows 380 / 373, 512 830 / 812.
constexpr int kOutSplitRows = 1024, kOutSplitOutputs = 1 << 22;
inline int out_splits(int m, int n, int k_in) {
    if (n < 2048 || n > 8192 || n % 64 != 0 || k_in < 2048 || k_in % 64 != 0 || k_in >= (1 << 23) || (long long)m * n > kOutSplitOutputs) return 1;
    return m <= 64 ? 4 : m <= 128 || (m > 256 && m <= kOutSplitRows) ? 2 : 1;
}

}   // namespace slim
