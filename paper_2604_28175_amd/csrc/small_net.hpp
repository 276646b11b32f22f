// A small classifier in one launch (small_net.hip).
#pragma once
#include "kernels.hpp"

namespace strait {

// x [rows][H][W][C] fp16, C <= 4; w0 [16][3][4][8] (rows, columns, channels, the rest zero), w1 [32][3][3][16], w2 [64][3][3][32]; out: as launch_classify_out, with
// the head's w and bias.
struct SmallNet {
    const half_t* x; const half_t* w0; const half_t* w1; const half_t* w2; const float* b0; const float* b1; const float* b2;
    int H, W, C;
    ClassifyOut out;
    int P1, Q1, P2, Q2;                  // filled in by launch_small_net
    Divisor by_xp, by_w, by_q1, by_q2;
};
bool small_net_takes(int H, int W, int C, long long rows, int classes);
int launch_small_net(const SmallNet& p, hipStream_t stream);

}  // namespace strait
