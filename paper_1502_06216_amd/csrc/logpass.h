// Log-domain Gibbs contraction along one axis (see logpass.hip).
#pragma once

#include "jko_internal.h"

namespace jko {

// One axis pass of the log-domain product: the field is [outer][n][inner]
// (the axis has stride inner), Y[o][i][j] = log sum_k exp(X[o][k][j] -
// alpha (i - k)^2) with alpha = 1 / (n^2 gamma), written in the same layout
// or handed (as logs) to the pointwise epilogue.
struct LogPass {
    int64_t outer, inner;
    int n;
    int R0;                // distance the max search starts with
    double alpha;
    const float* X;
    int OI, OF;            // outputs along the axis and fibres of a work item
    int T;                 // contiguous axis: threads staging a fibre
    int chunks;            // items per group of fibres
    int64_t items;
};

LogPass make_log_pass(int64_t outer, int n, int64_t inner, double gamma, const float* X);
int64_t log_pass_blocks(const LogPass& L);
// Every epilogue but the adjoint's; partial sums go to slot blockIdx (at most epi.part.cap blocks).
hipError_t launch_log_pass(const LogPass& L, const EpiArgs& epi, int* nblocks, hipStream_t st);

}  // namespace jko
