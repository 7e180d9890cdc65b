// The reflector of Procedure 2 (Section III of arXiv:1402.4247), shared by the
// blocked columns and the resident reduction.
#pragma once

#include "common.hpp"

namespace kgev {

// Procedure 2's reflector for the sub-column x = (alpha, x_2, ...) with
// sig2 = |x_2|^2 + ...: beta = -sign(Re alpha) ||x||, tau = (beta - alpha) /
// beta and the scale 1 / (alpha - beta) applied to x_2, ...; two reciprocals
// (the latency of a division chain dominates this single-lane step).
template <typename R>
__device__ __attribute__((always_inline)) inline void reflector_core(cx<R> alpha, R sig2, cx<R>& tau, cx<R>& scale, R& beta)
{
    if (sig2 == (R)0 && alpha.y == (R)0) {
        tau = czero<cx<R>>();
        scale = czero<cx<R>>();
        beta = alpha.x;
        return;
    }
    const R nrm = sqrt(alpha.x * alpha.x + alpha.y * alpha.y + sig2);
    beta = (alpha.x >= (R)0) ? -nrm : nrm;
    const R ib = (R)1 / beta;
    tau = mk<R>((beta - alpha.x) * ib, -alpha.y * ib);
    const R dr = alpha.x - beta, di = alpha.y;
    const R iden = (R)1 / (dr * dr + di * di);
    scale = mk<R>(dr * iden, -di * iden);
}

}  // namespace kgev
