// cnn.hpp - kernels of the learned initial guess: a 5-layer 3x3 convolutional
// net that maps the log diffraction patterns of a 3 x 3 scan neighbourhood
// (9 x 64 x 64) to the projected phase of the 32 x 32 patch centred on the
// middle position.
//
//   layer  in          out         stride   reduction K = 9 taps x Cin (padded)
//   0      9(16) x 64  32 x 64     1        144 -> 160
//   1      32 x 64     32 x 32     2        288
//   2      32 x 32     32 x 32     1        288
//   3      32 x 32     32 x 32     1        288
//   4      32 x 32     1(16) x 32  1        288        (no ReLU after it)
//
// Every convolution and both of its gradients is an implicit GEMM on the
// gfx950 matrix cores (v_mfma_f32_16x16x32_bf16: BF16 operands, FP32
// accumulation).  Activations and back-propagated gradients are stored NHWC in
// BF16 with channels padded to 16 / 32, so the 8 consecutive reduction elements
// a lane feeds to the MFMA are 8 consecutive channels of one pixel: one
// 16-byte load.  Lane i of a wave holds A[i%16][8(i/16)..+7],
// B[8(i/16)..+7][i%16] and receives D[4(i/16)..+3][i%16].
//
// Parameters are one FP32 vector: per layer W[Cout_p][K_p] with reduction
// index k = (3 u + v) * Cin_p + c for tap (u, v) and input channel c (padding
// entries are zero and stay zero under training, their gradient being exactly
// zero), followed by bias[Cout_p].
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ptyr {
namespace cnn {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) float floatx4;
typedef __attribute__((ext_vector_type(4))) short shortx4;

constexpr int NLAYER = 5;
constexpr int NB = 9;             // patterns per neighbourhood
constexpr int IN = 64;            // pattern side
constexpr int OUT = 32;           // phase patch side
constexpr int CIN[NLAYER] = {9, 32, 32, 32, 32};
constexpr int CINP[NLAYER] = {16, 32, 32, 32, 32};
constexpr int COUT[NLAYER] = {32, 32, 32, 32, 1};
constexpr int COUTP[NLAYER] = {32, 32, 32, 32, 16};
constexpr int STRIDE[NLAYER] = {1, 2, 1, 1, 1};
constexpr int HIN[NLAYER] = {64, 64, 32, 32, 32};
constexpr int HOUT[NLAYER] = {64, 32, 32, 32, 32};

constexpr int pad32(int x) { return (x + 31) / 32 * 32; }
constexpr int kp(int l) { return pad32(9 * CINP[l]); }          // forward / weight-gradient reduction
constexpr int kd(int l) { return pad32(9 * COUTP[l]); }         // input-gradient reduction
constexpr int w_size(int l) { return COUTP[l] * kp(l); }
constexpr int w_off(int l) { return l == 0 ? 0 : w_off(l - 1) + w_size(l - 1) + COUTP[l - 1]; }
constexpr int b_off(int l) { return w_off(l) + w_size(l); }
constexpr int NPARAM = b_off(NLAYER - 1) + COUTP[NLAYER - 1];
constexpr int wt_size(int l) { return CINP[l] * kd(l); }
constexpr int wt_off(int l) { return l == 0 ? 0 : wt_off(l - 1) + wt_size(l - 1); }
constexpr int WT_TOTAL = wt_off(NLAYER - 1) + wt_size(NLAYER - 1);
constexpr int WPARTS = 256;                    // weight-gradient partial sums per layer while batches are small
constexpr int WPIXELS = 2048;                  // pixels that one float32 accumulator of them adds, at most
constexpr int ERR_INDEX = 1;

// per-sample element counts of the stored BF16 tensors
constexpr int act_elems(int l) { return HIN[l] * HIN[l] * CINP[l]; }      // input of layer l
constexpr int grad_elems(int l) { return HOUT[l] * HOUT[l] * COUTP[l]; }  // dL/dz_l

__device__ __forceinline__ floatx4 mfma(bf16x8 a, bf16x8 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ bf16x8 zero8() {
    bf16x8 z;
#pragma unroll
    for (int e = 0; e < 8; ++e) z[e] = (__bf16)0.0f;
    return z;
}
__device__ __forceinline__ bf16x8 ld8(const __bf16* p) { return *reinterpret_cast<const bf16x8*>(p); }

// FP32 parameters -> BF16 W (same offsets) and, per layer, the transposed
// BF16 weights WT_l[c][(3u+v) * Cout_p + o] = W_l[o][(3u+v) * Cin_p + c] used by
// the input gradient (zero for reduction indices >= 9 Cout_p).
template <int L>
__device__ __forceinline__ void prep_wt(const float* p, __bf16* wt, int r) {
    constexpr int cinp = CINP[L], coutp = COUTP[L], K = kp(L), KD = kd(L);
    const int c = r / KD, kk = r % KD;
    float w = 0.f;
    if (kk < 9 * coutp) w = p[w_off(L) + (kk % coutp) * K + (kk / coutp) * cinp + c];
    wt[wt_off(L) + r] = (__bf16)w;
}
__device__ __forceinline__ void prep_weights(const float* p, __bf16* wbf, __bf16* wt, int i) {
    if (i < NPARAM) wbf[i] = (__bf16)p[i];
    if (i >= WT_TOTAL) return;
    if (i < wt_off(1)) prep_wt<0>(p, wt, i);
    else if (i < wt_off(2)) prep_wt<1>(p, wt, i - wt_off(1));
    else if (i < wt_off(3)) prep_wt<2>(p, wt, i - wt_off(2));
    else if (i < wt_off(4)) prep_wt<3>(p, wt, i - wt_off(3));
    else prep_wt<4>(p, wt, i - wt_off(4));
}

// Gather the 9 patterns of each neighbourhood (nbr: B x 9 indices into the
// n_pat patterns of 64 x 64) and store log(1 + max(I, 0)) as BF16 NHWC with 16
// channels (9 used).  An index outside [0, n_pat) raises ERR_INDEX and reads
// as an all-zero pattern.  A thread takes two pixels half a pattern apart, 18
// reads in flight.  The nprep first workgroups convert the parameters
// (prep_weights), which needs nothing of the input.
__global__ __launch_bounds__(256) void k_input(const float* pat, int n_pat, const int* nbr, int B, __bf16* X0,
                                               int* err, const float* params, __bf16* wbf, __bf16* wt, int nprep) {
    if ((int)blockIdx.x < nprep) {
        prep_weights(params, wbf, wt, blockIdx.x * blockDim.x + threadIdx.x);
        return;
    }
    constexpr int HALF = IN * IN / 2;
    const int n = B * HALF;
    for (int q = (blockIdx.x - nprep) * blockDim.x + threadIdx.x; q < n; q += (gridDim.x - nprep) * blockDim.x) {
        const int b = q / HALF, yx = q % HALF;                 // HALF is a multiple of the block: b is uniform
        float v[2][NB];
#pragma unroll
        for (int c = 0; c < NB; ++c) {
            const int j = nbr[b * NB + c];
            const bool ok = j >= 0 && j < n_pat;
            if (!ok && yx == 0) atomicOr(err, ERR_INDEX);
#pragma unroll
            for (int h = 0; h < 2; ++h) v[h][c] = ok ? pat[(size_t)j * IN * IN + yx + h * HALF] : 0.f;
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            bf16x8 lo, hi = zero8();
#pragma unroll
            for (int c = 0; c < 8; ++c) lo[c] = (__bf16)log1pf(fmaxf(v[h][c], 0.f));
            hi[0] = (__bf16)log1pf(fmaxf(v[h][8], 0.f));
            bf16x8* dst = reinterpret_cast<bf16x8*>(X0 + ((size_t)b * IN * IN + yx + h * HALF) * 16);
            dst[0] = lo;
            dst[1] = hi;
        }
    }
}

// Forward convolution of layer L over B samples:
//   z[p][o] = bias[o] + sum_k W[o][k] Xcol[k][p],   Y = bf16(max(z, 0))  (L < 4)
//   out[p] = z[p][0]                                                   (L = 4)
// A wave takes 16 output pixels and all output channels at a time and walks
// consecutive groups of 16 with its weights in registers (72 of them at 288 x
// 32), so a group costs its K / 32 input reads, all in flight together, and
// the MFMAs; with one group per wave the weights were read from cache with
// every group, two thirds of the bytes, in three dependent batches.
template <int L>
__global__ __launch_bounds__(256) void k_fwd(const __bf16* X, const __bf16* W, const float* bias, __bf16* Y,
                                             float* out, int B, int per) {
    constexpr int cinp = CINP[L], coutp = COUTP[L], s = STRIDE[L], hin = HIN[L], hout = HOUT[L], K = kp(L);
    constexpr int MT = coutp / 16, KS = K / 32;
    const int lane = threadIdx.x % 64, g = lane / 16, n = lane % 16;
    const int g0 = (blockIdx.x * 4 + threadIdx.x / 64) * per, g1 = min(g0 + per, B * hout * hout / 16);
    bf16x8 w[KS][MT];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) w[ks][mt] = ld8(W + (mt * 16 + n) * K + 32 * ks + 8 * g);
    for (int grp = g0; grp < g1; ++grp) {
        const int p = grp * 16 + n;
        const int b = p / (hout * hout), yo = (p / hout) % hout, xo = p % hout;
        const __bf16* Xb = X + (size_t)b * hin * hin * cinp;
        bf16x8 x[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int k = 32 * ks + 8 * g, tap = k / cinp, c0 = k % cinp;
            const int yi = yo * s + tap / 3 - 1, xi = xo * s + tap % 3 - 1;
            x[ks] = zero8();
            if (k < 9 * cinp && yi >= 0 && yi < hin && xi >= 0 && xi < hin) x[ks] = ld8(Xb + (yi * hin + xi) * cinp + c0);
        }
        floatx4 acc[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[mt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[mt] = mfma(w[ks][mt], x[ks], acc[mt]);
        if constexpr (L < NLAYER - 1) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                bf16x4 y4;
#pragma unroll
                for (int r = 0; r < 4; ++r) y4[r] = (__bf16)fmaxf(acc[mt][r] + bias[mt * 16 + 4 * g + r], 0.f);
                *reinterpret_cast<bf16x4*>(Y + (size_t)p * coutp + mt * 16 + 4 * g) = y4;
            }
        } else {
            if (g == 0) out[p] = acc[0][0] + bias[0];
        }
    }
}

// Mean squared error over n outputs, in FP64: per-block partial sums (added up
// by k_wreduce), and dL/dz_4 = bf16(2 (out - target) / n) in channel 0 of 16.
__global__ __launch_bounds__(256) void k_mse(const float* out, const float* target, int n, double* part, __bf16* G4) {
    __shared__ double sh[256];
    double s = 0.0;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const float o = out[i], t = target[i];
        const double d = (double)o - (double)t;
        s += d * d;
        bf16x8 lo = zero8();
        lo[0] = (__bf16)(2.0f * (o - t) / (float)n);
        bf16x8* dst = reinterpret_cast<bf16x8*>(G4 + (size_t)i * 16);
        dst[0] = lo;
        dst[1] = zero8();
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

// Weight and bias gradient of layer L, summed over a range of tiles:
//   part[w][o * K + k] = sum_p G[p][o] Xcol[k][p],  part[w][Cout_p * K + o] = sum_p G[p][o]
// A tile is TR output rows of one sample.  Its gradients G and the input rows
// under it (one zero column either side, rows outside the input zero) are
// staged in LDS as they lie in memory, pixel by pixel, 16 bytes per thread
// and load, the next tile's loads in flight while the current one is summed.
// The pixel sum is the MFMA reduction, so an operand is 8 consecutive pixels
// of one channel: two transposing LDS reads (ds_read_b64_tr_b16: 16 lanes
// read 4 pixels x 16 channels and get 4 pixels of one channel each), at the
// tap's pixel offset, so no im2col copy is formed.  (Staged transposed, by 8
// dword writes per two pixels, and per third of the reduction range, the five
// layers took 283 us at 256 samples.)
// Eight waves: wave w takes channel tile w % NC, the taps of group w / NC, and
// every other group of 32 pixels (w / 4); the two halves are added at the end.
template <int L> struct WGrad {
    static constexpr int cinp = CINP[L], coutp = COUTP[L], s = STRIDE[L], hin = HIN[L], hout = HOUT[L], K = kp(L);
    static constexpr int TR = L == 1 ? 4 : 8;                  // output rows per tile
    static constexpr int PX = TR * hout, XR = (TR - 1) * s + 3, XC = hin + 2;
    static constexpr int MT = coutp / 16, NC = cinp / 16, TG = 4 / NC, TPW = (9 + TG - 1) / TG;
    static constexpr int GB = PX * coutp * 2, XB = XR * XC * cinp * 2;         // bytes
    static constexpr int ACC = 4 * 64 * (TPW * MT * 4 + MT) * 4;              // the second half's sums
    static constexpr int LDS = GB + XB > ACC ? GB + XB : ACC;
    static constexpr int TPS = hout / TR;                       // tiles per sample
    static constexpr int TMAX = 2 * WPIXELS / PX;               // tiles per workgroup at most (its halves share them)
    static constexpr int NGI = PX * coutp / 8, NXI = XR * hin * cinp / 8;      // 16-byte pieces
    static constexpr int NG = (NGI + 511) / 512, NX = (NXI + 511) / 512;
};
constexpr int wgrad_lds() {
    int m = WGrad<0>::LDS;
    m = WGrad<1>::LDS > m ? WGrad<1>::LDS : m;
    m = WGrad<2>::LDS > m ? WGrad<2>::LDS : m;
    return WGrad<4>::LDS > m ? WGrad<4>::LDS : m;
}
// 4 pixels of one channel of a pixel-major tile, by the wave's 16-lane groups
__device__ __forceinline__ shortx4 ld_tr(const char* p) {
    typedef __attribute__((address_space(3))) shortx4* lds4;
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(__attribute__((address_space(3))) char*)p);
}
__device__ __forceinline__ bf16x8 join(shortx4 a, shortx4 b) {
    typedef __attribute__((ext_vector_type(8))) short shortx8;
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

template <int L>
__device__ void wgrad(char* lds, const __bf16* G, const __bf16* X, float* part, int B, int w0, int nw) {
    using Q = WGrad<L>;
    constexpr int K = Q::K, MT = Q::MT, NC = Q::NC, TG = Q::TG, TPW = Q::TPW;
    const int tid = threadIdx.x, lane = tid % 64, g = lane / 16, i = lane % 16, wave = tid / 64;
    const int ct = wave % NC, tg = (wave % 4) / NC, hv = wave / 4;
    const int tap0 = tg * 9 / TG, tap1 = (tg + 1) * 9 / TG;
    const int tiles = B * Q::TPS, t0 = (int)((long)tiles * w0 / nw), t1 = (int)((long)tiles * (w0 + 1) / nw);
    char *gs = lds, *xs = lds + Q::GB;
    bf16x8 gv[Q::NG], xv[Q::NX];
    auto fetch = [&](int t) {
        const int b = t / Q::TPS, y0 = (t % Q::TPS) * Q::TR;
        const __bf16* Gt = G + ((size_t)b * Q::hout + y0) * Q::hout * Q::coutp;
        const __bf16* Xb = X + (size_t)b * Q::hin * Q::hin * Q::cinp;
#pragma unroll
        for (int j = 0; j < Q::NG; ++j) {
            const int it = tid + 512 * j;
            gv[j] = it < Q::NGI ? ld8(Gt + (size_t)it * 8) : zero8();
        }
#pragma unroll
        for (int j = 0; j < Q::NX; ++j) {
            const int it = tid + 512 * j, row = it / (Q::hin * Q::cinp / 8), in = it % (Q::hin * Q::cinp / 8);
            const int y = y0 * Q::s - 1 + row;
            xv[j] = it < Q::NXI && y >= 0 && y < Q::hin ? ld8(Xb + (size_t)y * Q::hin * Q::cinp + in * 8) : zero8();
        }
    };
    floatx4 acc[TPW][MT];
    float bs[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        bs[mt] = 0.f;
#pragma unroll
        for (int t = 0; t < TPW; ++t) acc[t][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    // the zero columns
    for (int e = tid; e < Q::XR * 2 * Q::cinp / 8; e += 512) {
        const int c8 = e % (Q::cinp / 8), r = e / (Q::cinp / 8), col = (r & 1) ? Q::XC - 1 : 0;
        *reinterpret_cast<bf16x8*>(xs + ((r >> 1) * Q::XC + col) * Q::cinp * 2 + c8 * 16) = zero8();
    }
    if (t0 < t1) fetch(t0);
    for (int t = t0; t < t1; ++t) {
#pragma unroll
        for (int j = 0; j < Q::NG; ++j) {
            const int it = tid + 512 * j;
            if (it < Q::NGI) *reinterpret_cast<bf16x8*>(gs + it * 16) = gv[j];
        }
#pragma unroll
        for (int j = 0; j < Q::NX; ++j) {
            const int it = tid + 512 * j, row = it / (Q::hin * Q::cinp / 8), in = it % (Q::hin * Q::cinp / 8);
            if (it < Q::NXI) *reinterpret_cast<bf16x8*>(xs + (row * Q::XC + 1) * Q::cinp * 2 + in * 16) = xv[j];
        }
        __syncthreads();
        if (t + 1 < t1) fetch(t + 1);
        // lane i of group g addresses pixel 8 g + i / 4 (and 4 further), channels 4 (i % 4) ..
        for (int ks = hv; ks < Q::PX / 32; ks += 2) {
            const int px = 32 * ks + 8 * g + i / 4, yo = px / Q::hout, xo = px % Q::hout;
            const char* ga = gs + px * Q::coutp * 2 + (i % 4) * 8;
            bf16x8 av[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                av[mt] = join(ld_tr(ga + mt * 32), ld_tr(ga + mt * 32 + 4 * Q::coutp * 2));
                if (ct == 0 && tg == 0) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) bs[mt] += (float)av[mt][e];
                }
            }
            const char* xa = xs + (yo * Q::s * Q::XC + xo * Q::s) * Q::cinp * 2 + ct * 32 + (i % 4) * 8;
#pragma unroll
            for (int t2 = 0; t2 < TPW; ++t2) {
                const int tap = tap0 + t2;
                if (tap < tap1) {
                    const char* xt = xa + ((tap / 3) * Q::XC + tap % 3) * Q::cinp * 2;
                    const bf16x8 bv = join(ld_tr(xt), ld_tr(xt + 4 * Q::s * Q::cinp * 2));
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) acc[t2][mt] = mfma(av[mt], bv, acc[t2][mt]);
                }
            }
        }
        __syncthreads();
    }
    // second half's sums to the first half
    float* sum = reinterpret_cast<float*>(lds) + (size_t)(wave % 4) * 64 * (TPW * MT * 4 + MT) + lane;
    if (hv == 1) {
#pragma unroll
        for (int t2 = 0; t2 < TPW; ++t2)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) sum[((t2 * MT + mt) * 4 + r) * 64] = acc[t2][mt][r];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) sum[(TPW * MT * 4 + mt) * 64] = bs[mt];
    }
    __syncthreads();
    float* dst = part + (size_t)w0 * (w_size(L) + Q::coutp);
    if (hv == 0) {
#pragma unroll
        for (int t2 = 0; t2 < TPW; ++t2)
            if (tap0 + t2 < tap1) {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        dst[(mt * 16 + 4 * g + r) * K + (tap0 + t2) * Q::cinp + ct * 16 + i] =
                            acc[t2][mt][r] + sum[((t2 * MT + mt) * 4 + r) * 64];
            }
        if (ct == 0 && tg == 0) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                float b = bs[mt] + sum[(TPW * MT * 4 + mt) * 64];
                b += __shfl_xor(b, 16, 64);
                b += __shfl_xor(b, 32, 64);
                if (g == 0) dst[w_size(L) + mt * 16 + i] = b;
            }
        }
    }
    // reduction rows past 9 Cin_p are padding with zero gradient
    if constexpr (K > 9 * Q::cinp) {
        constexpr int pad = K - 9 * Q::cinp;
        for (int e = tid; e < Q::coutp * pad; e += 512) dst[(e / pad) * K + 9 * Q::cinp + e % pad] = 0.f;
    }
}

// Partial sums of every layer in one launch: workgroup w of layer blockIdx.y
// (nw[l] of them) sums its share of the layer's tiles.
struct WGradArgs {
    const __bf16 *G[NLAYER], *X[NLAYER];
    float* part[NLAYER];
    int nw[NLAYER], B;
};
__global__ __launch_bounds__(512) void k_wgrad(WGradArgs a) {
    __shared__ __align__(16) char lds[wgrad_lds()];
    const int l = NLAYER - 1 - blockIdx.y, w = blockIdx.x;
    if (w >= a.nw[l]) return;
    switch (l) {
        case 0: wgrad<0>(lds, a.G[0], a.X[0], a.part[0], a.B, w, a.nw[0]); break;
        case 1: wgrad<1>(lds, a.G[1], a.X[1], a.part[1], a.B, w, a.nw[1]); break;
        case 2: wgrad<2>(lds, a.G[2], a.X[2], a.part[2], a.B, w, a.nw[2]); break;
        case 3: wgrad<3>(lds, a.G[3], a.X[3], a.part[3], a.B, w, a.nw[3]); break;
        default: wgrad<4>(lds, a.G[4], a.X[4], a.part[4], a.B, w, a.nw[4]); break;
    }
}

// grad[i] += sum over the layer's partial sums, in order, of part[w][i], every
// layer in one launch.  A block covers 32 entries with 8 threads each; thread
// t sums the parts t, t + 8, ... and the 8 partial sums are added in thread
// order.  The last block adds up the loss (loss_part, nblk of them).
struct WReduceArgs {
    const float* part[NLAYER];
    int nw[NLAYER];
    const double* loss_part;
    int nblk, n;
    double* loss;
};
constexpr int wreduce_blocks(int l) { return (w_size(l) + COUTP[l] + 31) / 32; }
__global__ __launch_bounds__(256) void k_wreduce(WReduceArgs a, float* grad) {
    int blk = blockIdx.x;
    if (blk == (int)gridDim.x - 1) {
        __shared__ double sd[256];
        double s = 0.0;
        for (int b = threadIdx.x; b < a.nblk; b += 256) s += a.loss_part[b];
        sd[threadIdx.x] = s;
        __syncthreads();
        for (int o = 128; o > 0; o >>= 1) {
            if ((int)threadIdx.x < o) sd[threadIdx.x] += sd[threadIdx.x + o];
            __syncthreads();
        }
        if (threadIdx.x == 0) *a.loss = sd[0] / a.n;
        return;
    }
    int l = 0, n = 0, off = 0;
#pragma unroll
    for (int q = 0; q < NLAYER; ++q) {
        constexpr int PW[NLAYER] = {w_size(0) + COUTP[0], w_size(1) + COUTP[1], w_size(2) + COUTP[2],
                                    w_size(3) + COUTP[3], w_size(4) + COUTP[4]};
        constexpr int OFF[NLAYER] = {w_off(0), w_off(1), w_off(2), w_off(3), w_off(4)};
        constexpr int NBLK[NLAYER] = {wreduce_blocks(0), wreduce_blocks(1), wreduce_blocks(2), wreduce_blocks(3),
                                      wreduce_blocks(4)};
        if (n == 0) {
            if (blk < NBLK[q]) { l = q; n = PW[q]; off = OFF[q]; }
            else blk -= NBLK[q];
        }
    }
    __shared__ float sh[8][33];
    const int e = threadIdx.x % 32, t = threadIdx.x / 32;
    const int i = blk * 32 + e;
    const float* part = a.part[l];
    const int nw = a.nw[l];
    float s = 0.f;
    if (i < n) {
        int w = t;
        for (; w + 24 < nw; w += 32) {                 // four reads in flight, added in order
            float v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = part[(size_t)(w + 8 * q) * n + i];
#pragma unroll
            for (int q = 0; q < 4; ++q) s += v[q];
        }
        for (; w < nw; w += 8) s += part[(size_t)w * n + i];
    }
    sh[t][e] = s;
    __syncthreads();
    if (t == 0 && i < n) {
        float r = sh[0][e];
#pragma unroll
        for (int q = 1; q < 8; ++q) r += sh[q][e];
        grad[off + i] += r;
    }
}

// Input gradient of layer L (L >= 1) through the ReLU of layer L-1:
//   Gprev[q][c] = bf16([X[q][c] > 0] sum_{tap, o} WT[c][tap * Cout_p + o] G[p_out(q, tap)][o])
// where output pixel p_out = ((y + 1 - u) / s, (x + 1 - v) / s) when that is an
// integer inside the output.  A wave takes 16 input pixels and all channels at
// a time and walks consecutive groups with its weights in registers, as k_fwd
// (stride 2: groups of one parity class, see below).
template <int L>
__global__ __launch_bounds__(256) void k_dgrad(const __bf16* G, const __bf16* WT, const __bf16* X, __bf16* Gprev,
                                               int B, int per) {
    constexpr int cinp = CINP[L], coutp = COUTP[L], s = STRIDE[L], hin = HIN[L], hout = HOUT[L], KD = kd(L);
    constexpr int MT = cinp / 16;
    const int lane = threadIdx.x % 64, g = lane / 16, n = lane % 16;
    const int wv = blockIdx.x * 4 + threadIdx.x / 64;
    // dL/dz of the wave's 16 pixels q (one per lane n) from the accumulators
    auto put = [&](size_t q, const floatx4 (&acc)[MT]) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const size_t o = q * cinp + mt * 16 + 4 * g;
            const bf16x4 x4 = *reinterpret_cast<const bf16x4*>(X + o);
            bf16x4 g4;
#pragma unroll
            for (int r = 0; r < 4; ++r) g4[r] = (float)x4[r] > 0.f ? (__bf16)acc[mt][r] : (__bf16)0.0f;
            *reinterpret_cast<bf16x4*>(Gprev + o) = g4;
        }
    };
    if constexpr (s == 2) {
        // A wave stays in one class of row and column parity: only the taps
        // (u, v) with y + 1 - u and x + 1 - v even meet an output pixel, the
        // same for all pixels of the class (u = 1 for even rows, u = 0, 2 for
        // odd ones; v likewise), so the reduction runs over those 1, 2 or 4
        // taps in increasing order (the other taps' products are zero) and
        // the wave keeps only their weights.  A group is every other pixel of
        // half a row.
        static_assert(coutp == 32, "one 32-wide reduction step per tap");
        const int py = wv & 1, px = (wv >> 1) & 1;
        const int nu = py ? 2 : 1, nv = px ? 2 : 1;
        bf16x8 w[2][2][MT];
#pragma unroll
        for (int iu = 0; iu < 2; ++iu)
#pragma unroll
            for (int iv = 0; iv < 2; ++iv) {
                const int tap = 3 * (py ? 2 * iu : 1) + (px ? 2 * iv : 1);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    w[iu][iv][mt] = iu < nu && iv < nv ? ld8(WT + (mt * 16 + n) * KD + tap * coutp + 8 * g) : zero8();
            }
        const int g0 = (wv >> 2) * per, g1 = min(g0 + per, B * hin);       // B x hin / 2 rows x 2 halves
        for (int grp = g0; grp < g1; ++grp) {
            const int b = grp / hin, yi = 2 * ((grp % hin) / 2) + py, xi = 2 * (16 * (grp & 1) + n) + px;
            bf16x8 bv[2][2];
#pragma unroll
            for (int iu = 0; iu < 2; ++iu)
#pragma unroll
                for (int iv = 0; iv < 2; ++iv) {
                    const int ty = yi + 1 - (py ? 2 * iu : 1), tx = xi + 1 - (px ? 2 * iv : 1);
                    bv[iu][iv] = zero8();
                    if (iu < nu && iv < nv && ty >= 0 && tx >= 0 && ty / 2 < hout && tx / 2 < hout)
                        bv[iu][iv] = ld8(G + (((size_t)b * hout + ty / 2) * hout + tx / 2) * coutp + 8 * g);
                }
            floatx4 acc[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[mt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int iu = 0; iu < 2; ++iu)
#pragma unroll
                for (int iv = 0; iv < 2; ++iv)
                    if (iu < nu && iv < nv) {
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt) acc[mt] = mfma(w[iu][iv][mt], bv[iu][iv], acc[mt]);
                    }
            put(((size_t)b * hin + yi) * hin + xi, acc);
        }
    } else {
        constexpr int KS = KD / 32;
        bf16x8 w[KS][MT];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) w[ks][mt] = ld8(WT + (mt * 16 + n) * KD + 32 * ks + 8 * g);
        const int g0 = wv * per, g1 = min(g0 + per, B * hin * hin / 16);
        for (int grp = g0; grp < g1; ++grp) {
            const int q = grp * 16 + n, b = q / (hin * hin), yi = (q / hin) % hin, xi = q % hin;
            const __bf16* Gb = G + (size_t)b * hout * hout * coutp;
            bf16x8 bv[KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const int kk = 32 * ks + 8 * g, tap = kk / coutp, o0 = kk % coutp;
                const int ty = yi + 1 - tap / 3, tx = xi + 1 - tap % 3;
                bv[ks] = zero8();
                if (kk < 9 * coutp && ty >= 0 && tx >= 0 && ty < hout && tx < hout)
                    bv[ks] = ld8(Gb + (ty * hout + tx) * coutp + o0);
            }
            floatx4 acc[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[mt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) acc[mt] = mfma(w[ks][mt], bv[ks], acc[mt]);
            put((size_t)q, acc);
        }
    }
}

// Adam on the FP32 parameter vector (PyTorch's form: bias-corrected moments,
// eps added to the corrected square root).
__global__ void k_adam(float* p, const float* gr, float* m, float* v, int n, float lr, float b1, float b2, float eps,
                       float bc1, float bc2s) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const float gi = gr[i];
        const float mi = b1 * m[i] + (1.f - b1) * gi;
        const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        p[i] -= (lr / bc1) * mi / (sqrtf(vi) / bc2s + eps);
    }
}

// Average the 32 x 32 patches (P of them, centred at round_half_even(centre),
// rows [cy - 16, cy + 16)) that cover each image pixel; uncovered pixels keep
// their value.  A workgroup takes a 16 x 16 tile, one thread per pixel; lane k
// of each wave tests one patch against the tile, 64 at a time, and the wave
// walks the ballot, so the patches are visited in order and only those near
// the tile by each pixel (with every pixel reading every centre, 64 patches on
// a 144 x 144 image took 18 us; 6 us this way).
__global__ __launch_bounds__(256) void k_stitch(const float* patches, const float* centres, int P, int H, int W,
                                                float* img) {
    const int ntx = (W + 15) / 16, ty = ((int)blockIdx.x / ntx) * 16, tx = ((int)blockIdx.x % ntx) * 16;
    const int y = ty + (int)threadIdx.x / 16, x = tx + (int)threadIdx.x % 16, lane = threadIdx.x % 64;
    float s = 0.f;
    int cnt = 0;
    for (int p0 = 0; p0 < P; p0 += 64) {
        const int q = p0 + lane;
        int y0 = 0, x0 = 0;
        bool near = false;
        if (q < P) {
            y0 = (int)rintf(centres[2 * q]) - OUT / 2;
            x0 = (int)rintf(centres[2 * q + 1]) - OUT / 2;
            near = ty + 16 > y0 && ty < y0 + OUT && tx + 16 > x0 && tx < x0 + OUT;
        }
        // eight patches' reads in flight, added in order
        for (unsigned long long m = __ballot(near); m;) {
            float v[8];
            bool in[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const bool live = m != 0;
                const int k = live ? __builtin_ctzll(m) : 0;
                const int py = y - __builtin_amdgcn_readlane(y0, k), px = x - __builtin_amdgcn_readlane(x0, k);
                in[u] = live && py >= 0 && py < OUT && px >= 0 && px < OUT;
                v[u] = in[u] ? patches[(size_t)(p0 + k) * OUT * OUT + py * OUT + px] : 0.f;
                m &= m - 1;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (in[u]) {
                    s += v[u];
                    ++cnt;
                }
        }
    }
    if (cnt && y < H && x < W) img[(size_t)y * W + x] = s / (float)cnt;
}

}  // namespace cnn
}  // namespace ptyr
