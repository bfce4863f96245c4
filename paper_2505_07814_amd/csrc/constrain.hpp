// constrain.hpp - per-iteration constraints on the object and probe (the
// paper's Sec. "Physical constraints"): the r_z depth filter with phase
// positivity, and probe-mode orthogonalisation.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

namespace ptyr {

constexpr int RZ_MAX_R = 64;        // largest tap radius (rz_sigma <= 16)
constexpr int ORTH_MAX_M = 24;      // most probe modes the orthogonalisation takes
constexpr int RZ_MAX_S = 256;       // deepest stack the depth filter takes
constexpr int GRAM_CHUNK = 1024;    // pixels per partial overlap sum
constexpr int GRAM_MAX_CHUNKS = 64; // N = 256: 65536 / 1024

struct RzTaps {
    float w[2 * RZ_MAX_R + 1];      // normalised taps w[k + R], k = -R..R
    int R;
};

// index i of a stack of S slices extended by mirroring about its outer faces
__device__ __forceinline__ int mirror_slice(int i, int S) {
    if (i >= 0 && i < S) return i;                       // inside, or one reflection (taps within S)
    if (i < 0 && i >= -S) return -1 - i;
    if (i >= S && i < 2 * S) return 2 * S - 1 - i;
    if (S == 1) return 0;
    const int period = 2 * S;
    i %= period;
    if (i < 0) i += period;
    return i < S ? i : period - 1 - i;
}

// r_z filter of one field (S x HW, in place), then optionally max(., 0).
// A thread owns one pixel's column: it reads the S values (consecutive
// threads take consecutive pixels, so each slice is one coalesced row per
// wave) into its own LDS column, which serves as an indexable array, and
// writes the filtered column back.  A thread touches only its own column,
// so no barrier is needed.  Dynamic LDS: S * blockDim.x floats.
__global__ __launch_bounds__(256) void k_rz_filter(float* v, int S, size_t HW, RzTaps taps, int positive) {
    extern __shared__ float col[];
    const int T = blockDim.x;
    const size_t px = (size_t)blockIdx.x * T + threadIdx.x;
    if (px >= HW) return;
    float* c = col + threadIdx.x;
    int s = 0;
    for (; s + 4 <= S; s += 4) {               // four reads in flight per thread
        float x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = v[(size_t)(s + u) * HW + px];
#pragma unroll
        for (int u = 0; u < 4; ++u) c[(s + u) * T] = x[u];
    }
    for (; s < S; ++s) c[s * T] = v[(size_t)s * HW + px];
    const int R = taps.R;
    for (s = 0; s < S; ++s) {
        float acc = 0.f;
        for (int k = -R; k <= R; ++k) acc = fmaf(taps.w[k + R], c[mirror_slice(s + k, S) * T], acc);
        v[(size_t)s * HW + px] = positive ? fmaxf(acc, 0.f) : acc;
    }
}

// The depth filter as an S x S matrix: B[s][s'] = sum of the taps w_k with
// mirror(s + k) = s' (the mirrored boundary folded in).  A whole workgroup.
__device__ __forceinline__ void rz_matrix(const RzTaps& taps, int S, float* Bm) {
    for (int i = threadIdx.x; i < S * S; i += blockDim.x) {
        const int s = i / S, s2 = i % S;
        float b = 0.f;
        for (int k = -taps.R; k <= taps.R; ++k)
            if (mirror_slice(s + k, S) == s2) b += taps.w[k + taps.R];
        Bm[i] = b;
    }
}

// ------------------------------------------------------------ probe modes
struct cd {
    double re, im;
};
__device__ __forceinline__ cd cd_mul(cd a, cd b) { return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }
__device__ __forceinline__ cd cd_conj(cd a) { return {a.re, -a.im}; }
__device__ __forceinline__ cd cd_add(cd a, cd b) { return {a.re + b.re, a.im + b.im}; }
__device__ __forceinline__ cd cd_scale(cd a, double s) { return {a.re * s, a.im * s}; }

struct EigLds {
    cd A[ORTH_MAX_M * ORTH_MAX_M], V[ORTH_MAX_M * ORTH_MAX_M];
    struct Rot {                     // the pairs' rotations of one round
        cd e;
        double c, s;
        int p, q;
    } rot[2][ORTH_MAX_M / 2];
    int done;
    double lam[ORTH_MAX_M];
    int order[ORTH_MAX_M];
};

// LDS accesses of one wave in order: what one lane wrote before is seen after
__device__ __forceinline__ void eig_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 1 / sqrt(x) and 1 / x for normal positive x: the hardware's estimate and two
// Newton steps (each squares the relative error, about 2^-26 to start with).
// The rotations' chain of library square roots and divisions was most of the
// eigen-solve's time.
__device__ __forceinline__ double rsqrt_nr(double x) {
    double y = __builtin_amdgcn_rsq(x);
#pragma unroll
    for (int i = 0; i < 2; ++i) y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
    return y;
}
__device__ __forceinline__ double rcp_nr(double x) {
    double y = __builtin_amdgcn_rcp(x);
#pragma unroll
    for (int i = 0; i < 2; ++i) y = fma(y, fma(-x, y, 1.0), y);
    return y;
}

// place of eigenvalue k in decreasing order, ties in index order, NaN last: a
// permutation whatever the values
__device__ __forceinline__ int eig_rank(const double* lam, int M, int k) {
    const double x = lam[k];
    int rank = 0;
    for (int j = 0; j < M; ++j) {
        const double y = lam[j];
        const bool before = isnan(x) ? !isnan(y) || j < k : y > x || (y == x && j < k);
        rank += before ? 1 : 0;
    }
    return rank;
}

// Eigenvectors of the Hermitian overlap matrix (summed from the chunk
// partials) by complex Jacobi rotations in double, by a workgroup of at least
// two waves, of which wave 0 rotates the matrix and wave 1 the vectors (lane k
// = 0..63 of either), then ordered by decreasing eigenvalue; each eigenvector is scaled by
// a unit phase so that its largest-magnitude entry (first of equals) is real
// and positive.  Writes V (M x M, column k = mode k's mixing coefficients) as
// float pairs and the eigenvalues.  A NaN in a mode is in its overlaps with every
// other, so the rotations make all of V NaN.
// A sweep is m - 1 rounds (m = M rounded up to even) of m / 2 disjoint pairs
// in the round-robin order, whose rotations are formed and applied together:
// the kernel is one serial chain of square roots and divisions, M (M - 1) / 2
// per sweep when the pairs follow one another (six modes: 61 us) and m - 1
// this way.
__device__ void probe_eig(EigLds& L, const cd* part, int nchunk, int M, float2* Vout, double* lam_out) {
    const int k = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int m = M + (M & 1), K = m / 2;
    cd *A = L.A, *V = L.V;
    if (wave == 1)
        for (int i = k; i < M * M; i += 64) V[i] = {(i / M) == (i % M) ? 1.0 : 0.0, 0.0};
    double tol = 0.0, small = 0.0;
    if (wave == 0) {
        // overlap matrix from the chunk sums (fixed order)
        for (int pid = k; pid < M * (M + 1) / 2; pid += 64) {
            int pr = pid, a = 0;
            while (pr >= M - a) { pr -= M - a; ++a; }
            const int b = a + pr;
            double re = 0.0, im = 0.0;
            for (int ch = 0; ch < nchunk; ++ch) {
                re += part[(size_t)pid * nchunk + ch].re;
                im += part[(size_t)pid * nchunk + ch].im;
            }
            A[a * M + b] = {re, a == b ? 0.0 : im};
            A[b * M + a] = {re, a == b ? 0.0 : -im};
        }
        eig_sync();
        double scale = 0.0;
        for (int i = 0; i < M; ++i) scale += A[i * M + i].re;
        tol = 1e-28 * scale * scale;              // off-diagonal norm 1e-14 of the trace
        small = fmax(1e-6 * tol / (M * M), 1e-280);   // entries that cannot matter to it stay (and none is denormal)
    }
    int buf = 0;
    for (int sweep = 0; sweep < 64; ++sweep) {
        if (wave == 0) {
            double off = 0.0;
            for (int i = k; i < M * M; i += 64)
                if (i / M != i % M) off += A[i].re * A[i].re + A[i].im * A[i].im;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) off += __shfl_xor(off, o, 64);
            if (k == 0) L.done = off <= tol;
        }
        __syncthreads();
        if (L.done) break;
        for (int r = 0; r < m - 1; ++r, buf ^= 1) {
            // round r of the round robin: m - 1 stays, the others rotate
            EigLds::Rot* rot = L.rot[buf];
            if (wave == 0 && k < K) {
                int p = k == 0 ? m - 1 : (r + k) % (m - 1), q = k == 0 ? r : (r - k + m - 1) % (m - 1);
                if (p > q) { const int t = p; p = q; q = t; }
                EigLds::Rot w{{1.0, 0.0}, 1.0, 0.0, p, -1};             // q = -1: nothing to rotate
                const cd apq = q < M ? A[p * M + q] : cd{0.0, 0.0};
                const double mag2 = apq.re * apq.re + apq.im * apq.im;
                if (!(mag2 <= small)) {                                 // NaN rotates too, and so spreads
                    // U = D P: D_qq = exp(-i alpha) makes the (p, q) entry real
                    // (alpha = arg a_pq), P the real Jacobi rotation that zeroes it
                    const double inv = rsqrt_nr(mag2);
                    w.e = {apq.re * inv, -apq.im * inv};                // exp(-i alpha)
                    const double zeta = (A[q * M + q].re - A[p * M + p].re) * (0.5 * inv);
                    const double az = fmin(fabs(zeta), 1e100), h = fma(az, az, 1.0);
                    const double t = copysign(rcp_nr(fma(h, rsqrt_nr(h), az)), zeta);
                    w.c = rsqrt_nr(fma(t, t, 1.0));
                    w.s = t * w.c;
                    w.q = q;
                }
                rot[k] = w;
            }
            // wave 1 is at most one round behind: it has passed this barrier
            // before wave 0 writes this half of rot again
            __syncthreads();
            // columns p, q of A U (wave 0) and of V U (wave 1)
            if (wave < 2) {
                cd* X = wave == 0 ? A : V;
                for (int i = k; i < K * M; i += 64) {
                    const int pr = i / M, row = i % M;
                    const EigLds::Rot w = rot[pr];
                    if (w.q < 0) continue;
                    const cd ap = X[row * M + w.p], aq = cd_mul(X[row * M + w.q], w.e);
                    X[row * M + w.p] = {w.c * ap.re - w.s * aq.re, w.c * ap.im - w.s * aq.im};
                    X[row * M + w.q] = {w.s * ap.re + w.c * aq.re, w.s * ap.im + w.c * aq.im};
                }
            }
            if (wave == 0) {
                eig_sync();
                // rows p, q of U^H (A U); the rotated entry is zero, the diagonal real
                for (int i = k; i < K * M; i += 64) {
                    const int pr = i / M, col = i % M;
                    const EigLds::Rot w = rot[pr];
                    if (w.q < 0) continue;
                    const cd bp = A[w.p * M + col], bq = cd_mul(A[w.q * M + col], cd_conj(w.e));
                    cd np = {w.c * bp.re - w.s * bq.re, w.c * bp.im - w.s * bq.im};
                    cd nq = {w.s * bp.re + w.c * bq.re, w.s * bp.im + w.c * bq.im};
                    if (col == w.p) { np.im = 0.0; nq = {0.0, 0.0}; }
                    if (col == w.q) { nq.im = 0.0; np = {0.0, 0.0}; }
                    A[w.p * M + col] = np;
                    A[w.q * M + col] = nq;
                }
                eig_sync();
            }
        }
    }
    __syncthreads();
    if (wave != 0) return;
    if (k < M) L.lam[k] = A[k * M + k].re;
    eig_sync();
    if (k < M) L.order[eig_rank(L.lam, M, k)] = k;
    eig_sync();
    if (k < M) {                                          // lane k: output column k
        const int src = L.order[k];
        int best = 0;
        double bm = -1.0;
        for (int a = 0; a < M; ++a) {
            const cd x = V[a * M + src];
            const double v = x.re * x.re + x.im * x.im;
            if (v > bm) { bm = v; best = a; }
        }
        const cd x = V[best * M + src];
        const double r = sqrt(x.re * x.re + x.im * x.im);
        const cd ph = r > 0 ? cd{x.re / r, -x.im / r} : cd{1.0, 0.0};
        for (int a = 0; a < M; ++a) {
            const cd y = cd_mul(V[a * M + src], ph);
            Vout[a * M + k] = make_float2((float)y.re, (float)y.im);
        }
        lam_out[k] = L.lam[src];
    }
}

// the arguments of probe_eig (M = 0: no orthogonalisation in this call)
struct EigArgs {
    const cd* part;
    int nchunk, M;
    float2* V;
    double* lam;
};
__global__ __launch_bounds__(128) void k_probe_eig(EigArgs a) {
    __shared__ EigLds L;
    probe_eig(L, a.part, a.nchunk, a.M, a.V, a.lam);
}

// ------------------------------------------------------------ r_z filter
// r_z filter for S <= RZ_REG_S: a thread keeps its pixel's column in
// registers and forms out = B x with the matrix read through the scalar
// cache (every thread of the launch reads the same entries).  EIG: workgroup
// (0, 0) runs the probe modes' eigen-solve instead, two waves of serial double
// arithmetic that the filter's stream through memory hides ((0, 1) is idle).
constexpr int RZ_REG_S = 32;
template <bool EIG> __device__ __forceinline__ bool rz_eig_block(const EigArgs& eig) {
    if constexpr (EIG) {
        __shared__ EigLds L;
        if (blockIdx.x == 0) {
            if (blockIdx.y == 0) probe_eig(L, eig.part, eig.nchunk, eig.M, eig.V, eig.lam);
            return true;
        }
    }
    return false;
}
template <bool EIG>
__global__ __launch_bounds__(256) void k_rz_filter_reg(float* v0, float* v1, int S, size_t HW,
                                                       const float* __restrict__ Bm, int positive1, EigArgs eig) {
    if (rz_eig_block<EIG>(eig)) return;
    // blockIdx.y: 0 filters v0 (amplitude), 1 filters v1 (phase; clipped at 0 with positive1)
    float* const v = blockIdx.y ? v1 : v0;
    const int positive = blockIdx.y ? positive1 : 0;
    const size_t px = (size_t)(blockIdx.x - (EIG ? 1 : 0)) * blockDim.x + threadIdx.x;
    if (px >= HW) return;
    float x[RZ_REG_S];
#pragma unroll
    for (int s = 0; s < RZ_REG_S; ++s) x[s] = s < S ? v[(size_t)s * HW + px] : 0.f;
    // a guarded body rather than a break, so that the loop unrolls fully
#pragma unroll
    for (int s = 0; s < RZ_REG_S; ++s) {
        if (s < S) {
            float acc = 0.f;
#pragma unroll
            for (int s2 = 0; s2 < RZ_REG_S; ++s2)
                if (s2 < S) acc = fmaf(Bm[s * S + s2], x[s2], acc);
            v[(size_t)s * HW + px] = positive ? fmaxf(acc, 0.f) : acc;
        }
    }
}

// The same for fields whose slice size is a multiple of 4: a thread owns four
// consecutive pixels (16-byte reads and writes).
// SM: the registers' stack depth, 16 or 32 (S <= SM): at 32 the columns take
// 142 registers, at 16 half, which leaves twice the waves to keep reads in
// flight.
template <bool EIG, int SM>
__global__ __launch_bounds__(256) void k_rz_filter_reg4(float* v0, float* v1, int S, size_t HW,
                                                        const float* __restrict__ Bm, int positive1, EigArgs eig) {
    if (rz_eig_block<EIG>(eig)) return;
    float* const v = blockIdx.y ? v1 : v0;
    const int positive = blockIdx.y ? positive1 : 0;
    const size_t px = ((size_t)(blockIdx.x - (EIG ? 1 : 0)) * blockDim.x + threadIdx.x) * 4;
    if (px >= HW) return;
    float4 x[SM];
#pragma unroll
    for (int s = 0; s < SM; ++s)
        x[s] = s < S ? *reinterpret_cast<const float4*>(v + (size_t)s * HW + px) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int s = 0; s < SM; ++s) {
        if (s < S) {
            float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int s2 = 0; s2 < SM; ++s2)
                if (s2 < S) {
                    const float b = Bm[s * S + s2];
                    acc.x = fmaf(b, x[s2].x, acc.x);
                    acc.y = fmaf(b, x[s2].y, acc.y);
                    acc.z = fmaf(b, x[s2].z, acc.z);
                    acc.w = fmaf(b, x[s2].w, acc.w);
                }
            if (positive)
                acc = make_float4(fmaxf(acc.x, 0.f), fmaxf(acc.y, 0.f), fmaxf(acc.z, 0.f), fmaxf(acc.w, 0.f));
            *reinterpret_cast<float4*>(v + (size_t)s * HW + px) = acc;
        }
    }
}

// threads per workgroup of the depth filter for S slices (LDS <= 64 KiB)
inline int rz_threads(int S) { return S <= 64 ? 256 : (S <= 128 ? 128 : 64); }

// phase positivity alone (elementwise)
__global__ void k_clip_negative(float* v, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        v[i] = fmaxf(v[i], 0.f);
}

// ------------------------------------------------------------ k_z filter
// The 3-D transform of one S x H x W object stack (sides up to 4096 with no prime factor
// other than 2, 3 and 5, e.g. 12 x 640 x 640).  Amplitude and phase travel as
// one complex field a + i phase: the weight W_a is real and even in k, so the
// filtered real and imaginary parts are the two filtered fields.  The
// transform is separable, so its axes may go in any order, and it runs as
// three passes through device memory:
//   1. x and z forward: a workgroup holds the S rows of one y
//   2. y forward, weight, y inverse: a workgroup holds a few columns of one k_z
//   3. z and x inverse
// (five, with x and z apart, where the S rows do not fit one workgroup).  A
// tile's lines are transformed in LDS stage by stage, one butterfly of radix
// 2 to 15 per thread and stage, so 640 = 8 8 10 takes three stages and 12 one;
// the first stage reads its operands straight from device memory and the last
// writes its results there.  At most 64 registers, for two 1024-thread
// workgroups per compute unit: with one (80 registers, five passes, four
// stages of at most radix 8, tiles staged through LDS at both ends) every
// barrier left the unit idle and a 12 x 640 x 640 call took 235 us; now 103 us
// (32 + 45 + 31 us; 82, 120 and 79 MB, of which the middle pass's 40 MB over
// its fields are the weight table, read once per k_z).

constexpr int KZ_MAX_THREADS = 1024;
constexpr int KZ_MAX_SIDE = 4096;
constexpr int KZ_MAX_ST = 6;                   // stages of one axis
constexpr int KZ_LDS_MAX = 80 * 1024;          // bytes per workgroup of a pass with a choice of tile

__device__ __forceinline__ float2 kz_mul_i(float2 a, int sg) {       // a * (sg i)
    return sg > 0 ? make_float2(-a.y, a.x) : make_float2(a.y, -a.x);
}

// cos and sin of 2 pi m / R at compile time (Taylor series on [-pi, pi])
constexpr double kz_series(double x, double term, int k) {
    double s = 0.0;
    for (int i = k; i < k + 40; i += 2) {
        s += term;
        term *= -x * x / ((i + 1) * (i + 2));
    }
    return s;
}
template <int R> struct KzRoots {
    float c[R] = {}, s[R] = {};
    constexpr KzRoots() {
        for (int m = 0; m < R; ++m) {
            const double x = 2.0 * 3.14159265358979323846 * (2 * m > R ? m - R : m) / R;
            c[m] = (float)kz_series(x, 1.0, 0);
            s[m] = (float)kz_series(x, x, 1);
        }
    }
};
template <int R1, int R2, int SG> __device__ __forceinline__ void kz_dft2(float2* x);

// R-point DFT X_b = sum_q x_q exp(SG 2 pi i q b / R) in place
template <int R, int SG> __device__ __forceinline__ void kz_dft(float2* x) {
    if constexpr (R == 2) {
        const float2 a = x[0], b = x[1];
        x[0] = make_float2(a.x + b.x, a.y + b.y);
        x[1] = make_float2(a.x - b.x, a.y - b.y);
    } else if constexpr (R == 4) {
        const float2 y0 = make_float2(x[0].x + x[2].x, x[0].y + x[2].y);
        const float2 y1 = make_float2(x[0].x - x[2].x, x[0].y - x[2].y);
        const float2 y2 = make_float2(x[1].x + x[3].x, x[1].y + x[3].y);
        const float2 y3 = kz_mul_i(make_float2(x[1].x - x[3].x, x[1].y - x[3].y), SG);
        x[0] = make_float2(y0.x + y2.x, y0.y + y2.y);
        x[2] = make_float2(y0.x - y2.x, y0.y - y2.y);
        x[1] = make_float2(y1.x + y3.x, y1.y + y3.y);
        x[3] = make_float2(y1.x - y3.x, y1.y - y3.y);
    } else if constexpr (R == 8) {
        float2 e[4] = {x[0], x[2], x[4], x[6]}, o[4] = {x[1], x[3], x[5], x[7]};
        kz_dft<4, SG>(e);
        kz_dft<4, SG>(o);
        // exp(SG 2 pi i k / 8) for k = 1, 2, 3
        constexpr float r = 0.70710678118654752440f;
        o[1] = make_float2(r * (o[1].x - SG * o[1].y), r * (o[1].y + SG * o[1].x));
        o[2] = kz_mul_i(o[2], SG);
        o[3] = make_float2(r * (-o[3].x - SG * o[3].y), r * (-o[3].y + SG * o[3].x));
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            x[k] = make_float2(e[k].x + o[k].x, e[k].y + o[k].y);
            x[k + 4] = make_float2(e[k].x - o[k].x, e[k].y - o[k].y);
        }
    } else if constexpr (R == 3) {
        constexpr float h = 0.86602540378443864676f;          // sin(2 pi / 3)
        const float2 s = make_float2(x[1].x + x[2].x, x[1].y + x[2].y);
        const float2 t = make_float2(x[0].x - 0.5f * s.x, x[0].y - 0.5f * s.y);
        const float2 u = kz_mul_i(make_float2(h * (x[1].x - x[2].x), h * (x[1].y - x[2].y)), SG);
        x[0] = make_float2(x[0].x + s.x, x[0].y + s.y);
        x[1] = make_float2(t.x + u.x, t.y + u.y);
        x[2] = make_float2(t.x - u.x, t.y - u.y);
    } else if constexpr (R == 6) {
        kz_dft2<2, 3, SG>(x);
    } else if constexpr (R == 9) {
        kz_dft2<3, 3, SG>(x);
    } else if constexpr (R == 10) {
        kz_dft2<2, 5, SG>(x);
    } else if constexpr (R == 12) {
        kz_dft2<3, 4, SG>(x);
    } else if constexpr (R == 15) {
        kz_dft2<3, 5, SG>(x);
    } else {
        static_assert(R == 5, "radix 2, 3, 4, 5, 6, 8, 9, 10, 12 or 15");
        constexpr float c1 = 0.30901699437494742410f, c2 = -0.80901699437494742410f;   // cos(2 pi / 5), cos(4 pi / 5)
        constexpr float s1 = 0.95105651629515357212f, s2 = 0.58778525229247312917f;    // sin(2 pi / 5), sin(4 pi / 5)
        const float2 t1 = make_float2(x[1].x + x[4].x, x[1].y + x[4].y);
        const float2 t2 = make_float2(x[2].x + x[3].x, x[2].y + x[3].y);
        const float2 d1 = make_float2(x[1].x - x[4].x, x[1].y - x[4].y);
        const float2 d2 = make_float2(x[2].x - x[3].x, x[2].y - x[3].y);
        const float2 a1 = make_float2(x[0].x + c1 * t1.x + c2 * t2.x, x[0].y + c1 * t1.y + c2 * t2.y);
        const float2 a2 = make_float2(x[0].x + c2 * t1.x + c1 * t2.x, x[0].y + c2 * t1.y + c1 * t2.y);
        const float2 b1 = kz_mul_i(make_float2(s1 * d1.x + s2 * d2.x, s1 * d1.y + s2 * d2.y), SG);
        const float2 b2 = kz_mul_i(make_float2(s2 * d1.x - s1 * d2.x, s2 * d1.y - s1 * d2.y), SG);
        x[0] = make_float2(x[0].x + t1.x + t2.x, x[0].y + t1.y + t2.y);
        x[1] = make_float2(a1.x + b1.x, a1.y + b1.y);
        x[4] = make_float2(a1.x - b1.x, a1.y - b1.y);
        x[2] = make_float2(a2.x + b2.x, a2.y + b2.y);
        x[3] = make_float2(a2.x - b2.x, a2.y - b2.y);
    }
}

// R = R1 R2: q = R2 q1 + q2, b = b1 + R1 b2
template <int R1, int R2, int SG> __device__ __forceinline__ void kz_dft2(float2* x) {
    constexpr KzRoots<R1 * R2> w;
    float2 y[R1][R2];
#pragma unroll
    for (int q2 = 0; q2 < R2; ++q2) {
        float2 t[R1];
#pragma unroll
        for (int q1 = 0; q1 < R1; ++q1) t[q1] = x[R2 * q1 + q2];
        kz_dft<R1, SG>(t);
#pragma unroll
        for (int b1 = 0; b1 < R1; ++b1) {
            const int m = q2 * b1;             // < R
            const float wc = w.c[m], ws = SG > 0 ? w.s[m] : -w.s[m];
            y[b1][q2] = m == 0 ? t[b1] : make_float2(t[b1].x * wc - t[b1].y * ws, t[b1].x * ws + t[b1].y * wc);
        }
    }
#pragma unroll
    for (int b1 = 0; b1 < R1; ++b1) {
        kz_dft<R2, SG>(y[b1]);
#pragma unroll
        for (int b2 = 0; b2 < R2; ++b2) x[b1 + R1 * b2] = y[b1][b2];
    }
}

// j / d for 0 <= j < 2^13 and 1 <= d < 2^13 from a float reciprocal: the
// product (j + 1/2) (1/d) is within 2^-23 (j + 1/2) / d of the exact quotient,
// less than its distance 1 / (2 d) to the nearest integer
__device__ __forceinline__ int kz_div(int j, float inv_d) { return (int)(((float)j + 0.5f) * inv_d); }

enum : int { KZ_IN_FIELDS = 1, KZ_OUT_FIELDS = 2 };

// A pass over tiles of A x B elements, element (a, b) at base + a * ga + b in
// the field, (a, b) in LDS at a * pitch + b + b / 8 (the padding spreads the
// strided writes of the first stages over the banks).  Tile t starts at
// (t / tpg) * gs + (t % tpg) * gt and holds cnt_a of the A lines (gt lines
// apart, la in all per group) or cnt_b of the B columns.  The stages run in
// order: along b (axis 0) or a (axis 1).
struct KzStage {
    short R, axis;       // radix; 0: along b, 1: along a
    int Ns, n;           // product of the axis's earlier radices, axis length
};
struct KzPass {
    int A, B, pitch, tiles, tpg;
    int rest_a, rest_b;  // lines / columns in the last tile of a group
    size_t gs, gt, ga;
    int nst, nfwd;       // stages; the first nfwd are forward transforms, the others inverse
    KzStage st[2 * KZ_MAX_ST];
    const float2 *twa, *twb;   // exp(-2 pi i k / A), exp(-2 pi i k / B)
    int use_a, use_b;          // entries of them the stages need
    int wgroup, W;             // weight: slice = t / tpg (wgroup), row length of the table
    double sdz;                // S dz
    int S;
};

template <int R, int SG, int F>
__device__ __forceinline__ void kz_stage(const KzPass& p, int i, float2* t, const float2* twl, float2* z, float* amp,
                                         float* phase, const float2* wtab, float kz, size_t base, int tile,
                                         int cnt_a, int cnt_b) {
    const KzStage s = p.st[i];
    const int m = s.n / R, id = threadIdx.x;
    int line, j;
    if (s.axis == 0) {
        line = kz_div(id, 1.0f / (float)m);
        j = id - line * m;
    } else {
        j = kz_div(id, 1.0f / (float)p.B);
        line = id - j * p.B;
    }
    const bool on = s.axis == 0 ? line < cnt_a : (j < m && line < cnt_b);
    const int jd = kz_div(j, 1.0f / (float)s.Ns), k = j - jd * s.Ns;
    const int o0 = jd * s.Ns * R + k;                     // first output
    // LDS slot and field offset of element e of the butterfly's line
    auto slot = [&](int e) {
        return s.axis == 0 ? line * p.pitch + e + (e >> 3) : e * p.pitch + line + (line >> 3);
    };
    auto field = [&](int e) {
        return base + (s.axis == 0 ? (size_t)line * p.ga + (size_t)e : (size_t)e * p.ga + (size_t)line);
    };
    float2 v[R];
    if (on) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int e = j + r * m;
            if (i == 0) {
                const size_t g = field(e);
                if constexpr ((F & KZ_IN_FIELDS) != 0) v[r] = make_float2(amp[g], phase[g]);
                else v[r] = z[g];
            } else {
                v[r] = t[slot(e)];
            }
        }
        if (s.Ns > 1) {
            const float2* tw = twl + (s.axis == 0 ? 0 : p.use_b);
            const int step = k * (s.n / (s.Ns * R));
#pragma unroll
            for (int r = 1; r < R; ++r) {
                const float2 w = tw[r * step];
                const float wy = SG < 0 ? w.y : -w.y;
                v[r] = make_float2(v[r].x * w.x - v[r].y * wy, v[r].x * wy + v[r].y * w.x);
            }
        }
        kz_dft<R, SG>(v);
        if (p.wgroup && i == p.nfwd - 1) {
            // W_a(k) / (S H W) of element (k_z, k_y, k_x): (1 - (2 / pi) atan(A k_z^2)) E
            // (A k_z first: k_z^2 alone may overflow)
            const int x0 = (tile % p.tpg) * (int)p.gt;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float2 ae = wtab[(size_t)(o0 + r * s.Ns) * p.W + x0 + line];
                const float wt = (1.0f - 0.63661977236758134308f * atanf(ae.x * kz * kz)) * ae.y;
                v[r] = make_float2(v[r].x * wt, v[r].y * wt);
            }
        }
    }
    if (i == p.nst - 1) {
        if (on) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const size_t g = field(o0 + r * s.Ns);
                if constexpr ((F & KZ_OUT_FIELDS) != 0) {
                    amp[g] = v[r].x;
                    phase[g] = v[r].y;
                } else {
                    z[g] = v[r];
                }
            }
        }
        return;
    }
    if (i > 0) __syncthreads();                          // every operand of the stage is read
    if (on) {
#pragma unroll
        for (int r = 0; r < R; ++r) t[slot(o0 + r * s.Ns)] = v[r];
    }
    __syncthreads();
}

// exp(-2 pi i k / n) (in double, rounded to float)
__device__ __forceinline__ float2 kz_twiddle(int k, int n) {
    double sn, cs;
    sincospi(2.0 * k / n, &sn, &cs);
    return make_float2((float)cs, (float)-sn);
}

// F: KZ_IN_FIELDS reads amplitude and phase instead of z, KZ_OUT_FIELDS writes
// them.  In the first launch of a call nw workgroups before the others form
// what the later launches read: the weight table, per (k_y, k_x) A = beta^2 /
// (k_r^2 + 1e-3) and E = exp(-alpha k_r^2) / (S H W), k_r^2 in double, k from
// fftfreq with the pixel size, and the twiddle tables of W, H and S.  That
// launch's own workgroups form the twiddles they need themselves.
struct KzWeight {
    int nw, S, H, W;
    double beta, alpha, dx;
    float2* tw;
};
template <int F>
__global__ __launch_bounds__(KZ_MAX_THREADS, 8) void k_kz_pass(KzPass p, KzWeight w, float2* z, float* amp,
                                                               float* phase, float2* wtab) {
    extern __shared__ float2 kz_lds[];
    if ((int)blockIdx.x < w.nw) {
        const int id = blockIdx.x * blockDim.x + threadIdx.x;
        for (int i = id; i < w.W + w.H + w.S; i += w.nw * blockDim.x)
            w.tw[i] = i < w.W ? kz_twiddle(i, w.W)
                              : (i < w.W + w.H ? kz_twiddle(i - w.W, w.H) : kz_twiddle(i - w.W - w.H, w.S));
        for (int i = id; i < w.H * w.W; i += w.nw * blockDim.x) {
            const int y = i / w.W, x = i - y * w.W;
            const double kx = (x < (w.W + 1) / 2 ? x : x - w.W) / (w.W * w.dx);
            const double ky = (y < (w.H + 1) / 2 ? y : y - w.H) / (w.H * w.dx);
            const double kr2 = kx * kx + ky * ky;
            wtab[i] = make_float2((float)(w.beta * w.beta / (kr2 + 1e-3)),
                                  (float)(exp(-w.alpha * kr2) / ((double)w.S * w.H * w.W)));
        }
        return;
    }
    // workgroups are dealt to the 8 XCDs in turn; tile t runs as workgroup
    // (t mod G8) * 8 + t / G8, so neighbouring tiles (which share cache lines
    // along a row in the column passes) run side by side on one XCD's L2
    const int bid = (int)blockIdx.x - w.nw, g8 = ((int)gridDim.x - w.nw) >> 3;
    const int tile = (bid & 7) * g8 + (bid >> 3);
    if (tile >= p.tiles) return;
    const int u = tile % p.tpg;
    const bool last = u == p.tpg - 1;
    const int cnt_a = last ? p.rest_a : p.A, cnt_b = last ? p.rest_b : p.B;
    const size_t base = (size_t)(tile / p.tpg) * p.gs + (size_t)u * p.gt;
    float2* tw = kz_lds + p.A * p.pitch;                  // twiddles along b, then along a
    if (w.nw > 0)
        for (int k = threadIdx.x; k < p.use_b + p.use_a; k += blockDim.x)
            tw[k] = k < p.use_b ? kz_twiddle(k, p.B) : kz_twiddle(k - p.use_b, p.A);
    else
        for (int k = threadIdx.x; k < p.use_b + p.use_a; k += blockDim.x)
            tw[k] = k < p.use_b ? p.twb[k] : p.twa[k - p.use_b];
    const int sl = tile / p.tpg;                          // k_z in double, rounded once
    const float kz = p.wgroup ? (float)((sl < (p.S + 1) / 2 ? sl : sl - p.S) / p.sdz) : 0.f;
    // the first stage needs no twiddles; its closing barrier publishes them
    for (int i = 0; i < p.nst; ++i) {
        auto run = [&](auto sg) {
            constexpr int SG = decltype(sg)::value;
            switch (p.st[i].R) {
                case 2: kz_stage<2, SG, F>(p, i, kz_lds, tw, z, amp, phase, wtab, kz, base, tile, cnt_a, cnt_b); break;
                case 3: kz_stage<3, SG, F>(p, i, kz_lds, tw, z, amp, phase, wtab, kz, base, tile, cnt_a, cnt_b); break;
                case 4: kz_stage<4, SG, F>(p, i, kz_lds, tw, z, amp, phase, wtab, kz, base, tile, cnt_a, cnt_b); break;
                case 5: kz_stage<5, SG, F>(p, i, kz_lds, tw, z, amp, phase, wtab, kz, base, tile, cnt_a, cnt_b); break;
                case 6: kz_stage<6, SG, F>(p, i, kz_lds, tw, z, amp, phase, wtab, kz, base, tile, cnt_a, cnt_b); break;
                case 8: kz_stage<8, SG, F>(p, i, kz_lds, tw, z, amp, phase, wtab, kz, base, tile, cnt_a, cnt_b); break;
                case 9: kz_stage<9, SG, F>(p, i, kz_lds, tw, z, amp, phase, wtab, kz, base, tile, cnt_a, cnt_b); break;
                case 10: kz_stage<10, SG, F>(p, i, kz_lds, tw, z, amp, phase, wtab, kz, base, tile, cnt_a, cnt_b); break;
                case 15: kz_stage<15, SG, F>(p, i, kz_lds, tw, z, amp, phase, wtab, kz, base, tile, cnt_a, cnt_b); break;
                default: kz_stage<12, SG, F>(p, i, kz_lds, tw, z, amp, phase, wtab, kz, base, tile, cnt_a, cnt_b); break;
            }
        };
        if (i < p.nfwd) run(std::integral_constant<int, -1>());
        else run(std::integral_constant<int, +1>());
    }
}

// Radices of a length-n line: the fewest stages, then the largest smallest
// radix (a stage has n / R butterflies per line).  Returns the number of
// stages, 0 for n = 1, or -1 if n has a prime factor other than 2, 3 and 5 or
// needs more than KZ_MAX_ST stages.
inline int fft_radices(int n, int* rs) {
    constexpr int RAD[] = {15, 12, 10, 9, 8, 6, 5, 4, 3, 2};
    if (n == 1) return 0;
    const int from = n == 3375 ? 0 : 1;       // 15 only where a stage would need more than KZ_MAX_THREADS butterflies
    int cur[KZ_MAX_ST], best_min = 0;
    for (int want = 1; want <= KZ_MAX_ST; ++want) {
        // radices in non-increasing order
        auto search = [&](auto&& self, int left, int depth, int first) -> void {
            if (depth == want) {
                if (left == 1 && cur[depth - 1] > best_min) {
                    best_min = cur[depth - 1];
                    for (int i = 0; i < depth; ++i) rs[i] = cur[i];
                }
                return;
            }
            for (int i = first; i < 10; ++i)
                if (left % RAD[i] == 0) {
                    cur[depth] = RAD[i];
                    self(self, left / RAD[i], depth + 1, i);
                }
        };
        search(search, n, 0, from);
        if (best_min) return want;
    }
    return -1;
}

// appends the stages of one axis (lengths n, radices rs); returns the
// butterflies of its largest stage per line
inline int kz_add_axis(KzPass& p, int axis, int n, const int* rs, int nr) {
    int Ns = 1, most = 0;
    for (int i = 0; i < nr; ++i) {
        p.st[p.nst++] = KzStage{(short)rs[i], (short)axis, Ns, n};
        most = most > n / rs[i] ? most : n / rs[i];
        Ns *= rs[i];
    }
    return most;
}
inline int kz_pitch(int B) { return (B + (B >> 3)) | 1; }
inline size_t kz_lds_bytes(const KzPass& p) {
    return ((size_t)p.A * p.pitch + p.use_a + p.use_b) * sizeof(float2);
}
inline int kz_most(int n, const int* rs, int nr) {      // butterflies of the largest stage of a line
    int most = 0;
    for (int i = 0; i < nr; ++i) most = most > n / rs[i] ? most : n / rs[i];
    return most;
}

// The passes of a call: plans[0 .. n).  in / out: whether the pass reads or
// writes the two fields.  rx, ry, rz: radices of W, H and S.
struct KzPlan {
    KzPass p;
    int threads, in, out;
};
inline int kz_plan(int S, int H, int W, const int* rx, int nx, const int* ry, int ny, const int* rz, int nz,
                   const float2* twx, const float2* twy, const float2* twz, double sdz, KzPlan* plans) {
    const size_t HW = (size_t)H * W;
    int np = 0;
    auto finish = [&](KzPass& p, int threads, int in, int out) {
        plans[np].p = p;
        plans[np].threads = (threads + 63) / 64 * 64;
        plans[np].in = in;
        plans[np++].out = out;
    };
    // lines side by side in a tile: a power of two, as many as `threads`
    // butterflies and KZ_LDS_MAX allow (at least one), no more than there are
    auto lines = [&](int n, int most, int threads, int cap, size_t total) {
        int nl = 1;
        while (2 * nl <= cap && (size_t)nl < total && 2 * nl * most <= threads &&
               ((size_t)n * kz_pitch(2 * nl) + n) * sizeof(float2) <= KZ_LDS_MAX)
            nl *= 2;
        return nl;
    };
    const int mx = kz_most(W, rx, nx), my = kz_most(H, ry, ny), mz = kz_most(S, rz, nz);
    // x and z together: S rows of one y
    KzPass xz{};
    xz.A = S;
    xz.B = W;
    xz.pitch = kz_pitch(W);
    xz.tiles = xz.tpg = H;
    xz.rest_a = S;
    xz.rest_b = W;
    xz.gt = W;
    xz.ga = HW;
    xz.twa = twz;
    xz.twb = twx;
    xz.use_a = S;
    xz.use_b = W;
    const int xzt = mx * S > mz * W ? mx * S : mz * W;
    const bool fused = S > 1 && xzt <= KZ_MAX_THREADS && kz_lds_bytes(xz) <= KZ_LDS_MAX;
    // x alone: rows of the whole stack, one after the other
    KzPass x{};
    {
        int nl = 1;
        const size_t rows = (size_t)S * H;
        while (2 * nl <= 16 && 2 * nl * mx <= 512 && ((size_t)2 * nl * kz_pitch(W) + W) * sizeof(float2) <= KZ_LDS_MAX)
            nl *= 2;
        x.A = nl;
        x.B = W;
        x.pitch = kz_pitch(W);
        x.tiles = x.tpg = (int)((rows + nl - 1) / nl);
        x.rest_a = (int)(rows - (size_t)(x.tiles - 1) * nl);
        x.rest_b = W;
        x.gt = (size_t)nl * W;
        x.ga = W;
        x.twb = twx;
        x.use_b = W;
    }
    // z alone: columns of S over consecutive pixels
    KzPass zc{};
    {
        const int nl = lines(S, mz, 512, 256, HW);
        zc.A = S;
        zc.B = nl;
        zc.pitch = kz_pitch(nl);
        zc.tiles = zc.tpg = (int)((HW + nl - 1) / nl);
        zc.rest_a = S;
        zc.rest_b = (int)(HW - (size_t)(zc.tiles - 1) * nl);
        zc.gt = nl;
        zc.ga = HW;
        zc.twa = twz;
        zc.use_a = S;
    }
    // y forward, weight, y inverse: columns of one slice
    KzPass y{};
    const int ynl = lines(H, my, KZ_MAX_THREADS, 16, W);
    y.A = H;
    y.B = ynl;
    y.pitch = kz_pitch(ynl);
    y.tpg = (W + ynl - 1) / ynl;
    y.tiles = S * y.tpg;
    y.rest_a = H;
    y.rest_b = W - (y.tpg - 1) * ynl;
    y.gs = HW;
    y.gt = ynl;
    y.ga = W;
    y.twa = twy;
    y.use_a = H;
    y.wgroup = 1;
    y.W = W;
    y.S = S;
    y.sdz = sdz;
    kz_add_axis(y, 1, H, ry, ny);
    y.nfwd = y.nst;
    kz_add_axis(y, 1, H, ry, ny);

    auto add = [&](KzPass p, bool ax, bool az, bool fwd, int threads, int in, int out) {
        if (ax && fwd) kz_add_axis(p, 0, W, rx, nx);
        if (az) kz_add_axis(p, 1, S, rz, nz);
        if (ax && !fwd) kz_add_axis(p, 0, W, rx, nx);
        p.nfwd = fwd ? p.nst : 0;
        finish(p, threads, in, out);
    };
    const bool z_apart = !fused && S > 1;
    if (fused) add(xz, true, true, true, xzt, 1, 0);
    else add(x, true, false, true, x.A * mx, 1, 0);
    if (z_apart) add(zc, false, true, true, zc.B * mz, 0, 0);
    finish(y, ynl * my, 0, 0);
    if (z_apart) add(zc, false, true, false, zc.B * mz, 0, 0);
    if (fused) add(xz, true, true, false, xzt, 0, 1);
    else add(x, true, false, false, x.A * mx, 0, 1);
    return np;
}

// Partial overlaps conj(P_m(r)) P_n(r) summed over one chunk of GRAM_CHUNK
// pixels, in double: workgroup (pair m <= n) * nchunk + chunk, written to
// part[pair * nchunk + chunk]; the eigen kernel adds the chunks in order.  A
// last workgroup (with Bm) forms the depth filter's matrix.
__global__ __launch_bounds__(256) void k_constrain_head(const float2* P, int M, int NN, cd* part, int nchunk,
                                                        RzTaps taps, int S, float* Bm) {
    if (Bm && blockIdx.x == gridDim.x - 1) {
        rz_matrix(taps, S, Bm);
        return;
    }
    const int chunk = blockIdx.x % nchunk;
    int pair = blockIdx.x / nchunk, m = 0;
    const int pair_id = pair;
    while (pair >= M - m) { pair -= M - m; ++m; }
    const int n = m + pair;
    const float2* a = P + (size_t)m * NN;
    const float2* b = P + (size_t)n * NN;
    double re = 0.0, im = 0.0;
    const int r1 = min(NN, (chunk + 1) * GRAM_CHUNK);
    for (int r = chunk * GRAM_CHUNK + threadIdx.x; r < r1; r += blockDim.x) {
        const float2 x = a[r], y = b[r];
        re += (double)x.x * y.x + (double)x.y * y.y;       // conj(x) y
        im += (double)x.x * y.y - (double)x.y * y.x;
    }
    __shared__ double sr[256], si[256];
    sr[threadIdx.x] = re;
    si[threadIdx.x] = im;
    __syncthreads();
    for (int o = blockDim.x / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            sr[threadIdx.x] += sr[threadIdx.x + o];
            si[threadIdx.x] += si[threadIdx.x + o];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) part[(size_t)pair_id * nchunk + chunk] = {sr[0], si[0]};
}

// Q_k(r) = sum_m V[m][k] P_m(r), in place: a workgroup stages the M values of
// its 256 pixels in LDS before writing.  Dynamic LDS: M * 256 float2 + M^2 float2.
__global__ __launch_bounds__(256) void k_probe_mix(float2* P, int M, int NN, const float2* V) {
    extern __shared__ float2 sm[];
    float2* vals = sm;                        // vals[m * 256 + t]
    float2* Vs = sm + (size_t)M * 256;
    const int t = threadIdx.x;
    const int r = blockIdx.x * 256 + t;
    for (int i = t; i < M * M; i += 256) Vs[i] = V[i];
    for (int m = 0; m < M; ++m) vals[m * 256 + t] = r < NN ? P[(size_t)m * NN + r] : make_float2(0.f, 0.f);
    __syncthreads();
    if (r >= NN) return;
    for (int kk = 0; kk < M; ++kk) {
        float re = 0.f, im = 0.f;
        for (int m = 0; m < M; ++m) {
            const float2 v = Vs[m * M + kk], p = vals[m * 256 + t];
            re = fmaf(v.x, p.x, fmaf(-v.y, p.y, re));
            im = fmaf(v.x, p.y, fmaf(v.y, p.x, im));
        }
        P[(size_t)kk * NN + r] = make_float2(re, im);
    }
}

}  // namespace ptyr
