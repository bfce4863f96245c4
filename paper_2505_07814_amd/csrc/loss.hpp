// loss.hpp - the batch's loss from its partial sums: one workgroup, launched on
// its own or as one workgroup of the gradient's launch.
#pragma once
#include <hip/hip_runtime.h>

#include "../../include/ptyr.h"

namespace ptyr {

enum : int { ERR_BOUNDS = 1, ERR_NONFINITE = 2, ERR_ZERO_MEAN = 4, ERR_INDEX = 8 };

// The data terms of the loss (Eq. 5 / Eq. 6, or their weighted sum of
// Eq. 9): term t has kind k[t], power p[t] and weight w[t]; n = 1 or 2.
struct LossTerms {
    int n;
    int k[2];
    double p[2], w[2];
};

// loss partial sums per block: E_0, R_0, E_1, R_1 (term means' summands) and
// the count of non-finite inputs
constexpr int NLP = 5;

// pass 2: fixed-order totals, loss and the gradient scales.  Per term t
//   Gaussian: L_t = sqrt(D)/Z, dL/dA = (A-E) / (K sqrt(D) Z)
//   Poisson : L_t = -mean(E log(A+eps) - A)/Z, dL/dA = -(E/(A+eps) - 1)/(K Z)
// and L = sum_t w_t L_t.  scal[5 + t] = w_t c_t (the batch factor of term t,
// which the per-pixel dI of term_val is missing); scal[1] = the factor the
// gradient reductions apply to the weights of k_loss_rows (w_0 c_0, or 1
// when two terms are folded into the weights by k_loss_mix); scal[2] = Z_0.
struct LossFinalArgs {
    const double* part;
    int nblk;
    double K;
    LossTerms lt;
    int check;
    double* scal;
    double* loss_out;
    int* err;
    const double* spart;
    int nsp;
    double spw;
};
constexpr int LOSS_FINAL_LDS = (NLP + 1) * 256;      // doubles
// one workgroup of at least 256 threads; sh: LOSS_FINAL_LDS doubles of LDS
__device__ __forceinline__ void loss_final_block(const LossFinalArgs& a, double* sh) {
    // the sparsity term's partial sums ride along as one more column (one
    // thread adding its B S entries in turn took 27 us at 882 of them)
    double s[NLP + 1] = {0, 0, 0, 0, 0, 0};
    const int tid = threadIdx.x;                          // threads past 256 only meet the barriers
    for (int b = tid; b < a.nblk && tid < 256; b += 256)
        for (int k = 0; k < NLP; ++k) s[k] += a.part[NLP * b + k];
    for (int b = tid; b < a.nsp && tid < 256; b += 256) s[NLP] += a.spart[b];
    if (tid < 256)
        for (int k = 0; k <= NLP; ++k) sh[k * 256 + tid] = s[k];
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o)
            for (int k = 0; k <= NLP; ++k) sh[k * 256 + threadIdx.x] += sh[k * 256 + threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double bad = sh[4 * 256];
        double L = 0.0, c[2] = {0.0, 0.0}, Z0 = 0.0;
        bool zero_mean = false;
        for (int t = 0; t < a.lt.n; ++t) {
            const double sE = sh[(2 * t) * 256], sR = sh[(2 * t + 1) * 256];
            const double Z = sE / a.K;
            if (t == 0) Z0 = Z;
            if (!(Z > 0.0)) { zero_mean = true; continue; }
            if (a.lt.k[t] == PTYR_LOSS_GAUSSIAN) {
                const double D = sR / a.K;
                L += a.lt.w[t] * sqrt(D) / Z;
                c[t] = D > 0.0 ? a.lt.w[t] / (a.K * sqrt(D) * Z) : 0.0;
            } else {
                L += a.lt.w[t] * (-(sR / a.K) / Z);
                c[t] = a.lt.w[t] / (a.K * Z);
            }
        }
        if (zero_mean) {
            atomicOr(a.err, ERR_ZERO_MEAN);
            L = 0.0; c[0] = c[1] = 0.0;
        }
        if (a.nsp > 0) L += a.spw * sh[NLP * 256];         // + sparsity term
        if (a.check && (bad > 0.0 || !isfinite(L))) atomicOr(a.err, ERR_NONFINITE);
        a.scal[0] = L;
        a.scal[1] = a.lt.n > 1 ? 1.0 : c[0];
        a.scal[2] = Z0;
        a.scal[5] = c[0];
        a.scal[6] = c[1];
        if (a.loss_out) *a.loss_out = L;
    }
}

}  // namespace ptyr
