// What a pass over the rows of the residual stream leaves behind besides their norm: see RowExtras.
#pragma once
#include "slim_common.h"
#include <math.h>

namespace slim {

struct RopeFreq { double inv_freq[128]; };               // head_dim <= 256
RopeFreq rope_freq(int d, float theta);

struct RowExtras {                                       // null: not wanted
    float* rstd = nullptr;               // [n] 1 / sqrt(mean(x[t, :]^2) + eps)
    float* table = nullptr;              // [n][2 half] cos | sin of the rows' angles
    const int* pos = nullptr;            // [n] positions, null: 0 .. n - 1
    int* pos_out = nullptr;              // [n] the positions again, and ..
    int* kept = nullptr;                 // .. [nb] 0 .. nb - 1 (nb <= n), in a layer that drops nothing
    int nb = 0, half = 0;
    RopeFreq fr;
};

}  // namespace slim
