// cnn.hip - C ABI of the learned initial guess (include/ptyr_cnn.h): launches
// of the BF16 matrix-core convolution kernels of cnn.hpp for inference,
// training gradients, Adam and patch stitching.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <new>

#include "cnn.hpp"
#include "ptyr_cnn.h"

using namespace ptyr::cnn;

struct ptyr_cnn {
    int B_max;
    char* ws;
    hipStream_t stream;
    size_t X[NLAYER], G[NLAYER], out, wbf, wt, wpart[NLAYER], lpart, loss, err, total;
    int n_cu;
};

namespace {

constexpr int LOSS_BLOCKS = 256;

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// workgroups (partial sums) of layer l's weight gradient for B samples: one
// per tile up to WPARTS, then as many as keep every float32 sum within
// WPIXELS pixels at any batch (from 257 samples on in layer 0, 1025 in others)
template <int L> int wgrad_parts(int B) {
    const long tiles = (long)B * WGrad<L>::TPS, most = WGrad<L>::TMAX;
    return (int)std::max(std::min(tiles, (long)WPARTS), (tiles + most - 1) / most);
}

// workspace offsets for batches of up to B neighbourhoods
void layout(ptyr_cnn* c, int B) {
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off += align256(bytes);
        return o;
    };
    for (int l = 0; l < NLAYER; ++l) c->X[l] = take((size_t)B * act_elems(l) * 2);
    for (int l = 0; l < NLAYER; ++l) c->G[l] = take((size_t)B * grad_elems(l) * 2);
    c->out = take((size_t)B * OUT * OUT * 4);
    c->wbf = take((size_t)NPARAM * 2);
    c->wt = take((size_t)WT_TOTAL * 2);
    const int nw[NLAYER] = {wgrad_parts<0>(B), wgrad_parts<1>(B), wgrad_parts<2>(B), wgrad_parts<3>(B),
                            wgrad_parts<4>(B)};
    for (int l = 0; l < NLAYER; ++l) c->wpart[l] = take((size_t)nw[l] * (w_size(l) + COUTP[l]) * 4);
    c->lpart = take(LOSS_BLOCKS * 8);
    c->loss = take(8);
    c->err = take(4);
    c->total = off;
}

template <class T>
T* at(ptyr_cnn* c, size_t off) {
    return reinterpret_cast<T*>(c->ws + off);
}

int blocks_for(size_t n, int per = 256) {
    size_t b = (n + per - 1) / per;
    return (int)(b > 4096 ? 4096 : (b < 1 ? 1 : b));
}

ptyr_status launched() { return hipGetLastError() == hipSuccess ? PTYR_OK : PTYR_E_DEVICE; }

// Groups of 16 pixels per wave, and the workgroups for them: about twelve waves
// per compute unit (what the weights' registers leave room for), each walking
// its share; at least one group.
struct GroupPlan {
    int per, blocks;
};
GroupPlan group_plan(const ptyr_cnn* c, long groups) {
    const long waves = 12L * c->n_cu;
    const int per = (int)std::max(1L, (groups + waves - 1) / waves);
    return {per, (int)((groups + 4L * per - 1) / (4L * per))};
}

template <int L>
void fwd_layer(ptyr_cnn* c, const float* params, int B, float* out) {
    const GroupPlan q = group_plan(c, (long)B * HOUT[L] * HOUT[L] / 16);
    __bf16* Y = L < NLAYER - 1 ? at<__bf16>(c, c->X[L + 1]) : nullptr;
    hipLaunchKernelGGL(k_fwd<L>, dim3(q.blocks), dim3(256), 0, c->stream, at<__bf16>(c, c->X[L]),
                       at<__bf16>(c, c->wbf) + w_off(L), params + b_off(L), Y, out, B, q.per);
}

// dL/dz of layer L - 1 from that of layer L.  Stride 2: the four waves of a
// workgroup take the four parity classes of the same rows.
template <int L>
void input_grad(ptyr_cnn* c, int B) {
    const long groups = STRIDE[L] == 2 ? (long)B * HIN[L] : (long)B * HIN[L] * HIN[L] / 16;
    GroupPlan q = group_plan(c, STRIDE[L] == 2 ? 4 * groups : groups);
    if (STRIDE[L] == 2) q.blocks = (int)((groups + q.per - 1) / q.per);
    hipLaunchKernelGGL(k_dgrad<L>, dim3(q.blocks), dim3(256), 0, c->stream, at<__bf16>(c, c->G[L]),
                       at<__bf16>(c, c->wt) + wt_off(L), at<__bf16>(c, c->X[L]), at<__bf16>(c, c->G[L - 1]), B, q.per);
}

// weights to BF16, gathered log input, the five layers; output to `out`
void run_forward(ptyr_cnn* c, const float* params, const float* pat, int n_pat, const int* nbr, int B, float* out) {
    const int nprep = NPARAM > WT_TOTAL ? NPARAM : WT_TOTAL;
    const int np = (nprep + 255) / 256;
    hipLaunchKernelGGL(k_input, dim3(np + blocks_for((size_t)B * IN * IN / 2)), dim3(256), 0, c->stream, pat, n_pat, nbr,
                       B, at<__bf16>(c, c->X[0]), at<int>(c, c->err), params, at<__bf16>(c, c->wbf),
                       at<__bf16>(c, c->wt), np);
    fwd_layer<0>(c, params, B, nullptr);
    fwd_layer<1>(c, params, B, nullptr);
    fwd_layer<2>(c, params, B, nullptr);
    fwd_layer<3>(c, params, B, nullptr);
    fwd_layer<4>(c, params, B, out);
}

ptyr_status check_batch(ptyr_cnn* c, const float* params, const float* pat, int n_pat, const int* nbr, int B) {
    if (!c || !params || !pat || !nbr) return PTYR_E_ARG;
    if (B < 1 || B > c->B_max || n_pat < 1) return PTYR_E_ARG;
    return PTYR_OK;
}

}  // namespace

extern "C" {

size_t ptyr_cnn_param_count(void) { return (size_t)NPARAM; }

size_t ptyr_cnn_workspace_bytes(int B_max) {
    if (B_max < 1) return 0;
    ptyr_cnn c;
    layout(&c, B_max);
    return c.total;
}

ptyr_status ptyr_cnn_create(int B_max, void* workspace, size_t ws_bytes, void* stream, ptyr_cnn** out) {
    if (!out) return PTYR_E_ARG;
    *out = nullptr;
    if (B_max < 1 || !workspace) return PTYR_E_ARG;
    ptyr_cnn* c = new (std::nothrow) ptyr_cnn;
    if (!c) return PTYR_E_NOMEM;
    c->B_max = B_max;
    c->ws = static_cast<char*>(workspace);
    c->stream = static_cast<hipStream_t>(stream);
    layout(c, B_max);
    if (ws_bytes < c->total) {
        delete c;
        return PTYR_E_NOMEM;
    }
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&c->n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || c->n_cu < 1) {
        delete c;
        return PTYR_E_DEVICE;
    }
    if (hipMemsetAsync(at<int>(c, c->err), 0, sizeof(int), c->stream) != hipSuccess) {
        delete c;
        return PTYR_E_DEVICE;
    }
    *out = c;
    return PTYR_OK;
}

void ptyr_cnn_destroy(ptyr_cnn* ctx) { delete ctx; }

ptyr_status ptyr_cnn_sync(ptyr_cnn* c) {
    if (!c) return PTYR_E_ARG;
    if (hipStreamSynchronize(c->stream) != hipSuccess) return PTYR_E_DEVICE;
    int e = 0;
    if (hipMemcpy(&e, at<int>(c, c->err), sizeof(int), hipMemcpyDeviceToHost) != hipSuccess) return PTYR_E_DEVICE;
    if (e) {
        const int z = 0;
        if (hipMemcpy(at<int>(c, c->err), &z, sizeof(int), hipMemcpyHostToDevice) != hipSuccess) return PTYR_E_DEVICE;
        return PTYR_E_ARG;
    }
    return PTYR_OK;
}

ptyr_status ptyr_cnn_forward(ptyr_cnn* c, const float* params, const float* patterns, int n_pat, const int* nbr,
                             int B, float* out) {
    ptyr_status st = check_batch(c, params, patterns, n_pat, nbr, B);
    if (st != PTYR_OK) return st;
    if (!out) return PTYR_E_ARG;
    run_forward(c, params, patterns, n_pat, nbr, B, out);
    return launched();
}

ptyr_status ptyr_cnn_gradient(ptyr_cnn* c, const float* params, const float* patterns, int n_pat, const int* nbr,
                              const float* target, int B, float* grad, double* loss_dev) {
    ptyr_status st = check_batch(c, params, patterns, n_pat, nbr, B);
    if (st != PTYR_OK) return st;
    if (!target || !grad) return PTYR_E_ARG;
    float* out = at<float>(c, c->out);
    run_forward(c, params, patterns, n_pat, nbr, B, out);
    const int n = B * OUT * OUT;
    const int nblk = blocks_for(n) < LOSS_BLOCKS ? blocks_for(n) : LOSS_BLOCKS;
    hipLaunchKernelGGL(k_mse, dim3(nblk), dim3(256), 0, c->stream, out, target, n, at<double>(c, c->lpart),
                       at<__bf16>(c, c->G[NLAYER - 1]));
    input_grad<4>(c, B);
    input_grad<3>(c, B);
    input_grad<2>(c, B);
    input_grad<1>(c, B);
    // every layer's weight gradient at once, then every layer's sum
    WGradArgs wg{};
    WReduceArgs wr{};
    const int nw[NLAYER] = {wgrad_parts<0>(B), wgrad_parts<1>(B), wgrad_parts<2>(B), wgrad_parts<3>(B),
                            wgrad_parts<4>(B)};
    int most = 0, blocks = 1;
    for (int l = 0; l < NLAYER; ++l) {
        wg.G[l] = at<__bf16>(c, c->G[l]);
        wg.X[l] = at<__bf16>(c, c->X[l]);
        wg.part[l] = at<float>(c, c->wpart[l]);
        wr.part[l] = wg.part[l];
        wg.nw[l] = wr.nw[l] = nw[l];
        most = std::max(most, nw[l]);
        blocks += wreduce_blocks(l);
    }
    wg.B = B;
    wr.loss_part = at<double>(c, c->lpart);
    wr.nblk = nblk;
    wr.n = n;
    wr.loss = loss_dev ? loss_dev : at<double>(c, c->loss);
    hipLaunchKernelGGL(k_wgrad, dim3(most, NLAYER), dim3(512), 0, c->stream, wg);
    hipLaunchKernelGGL(k_wreduce, dim3(blocks), dim3(256), 0, c->stream, wr, grad);
    return launched();
}

ptyr_status ptyr_cnn_adam(ptyr_cnn* c, float* params, const float* grad, float* m, float* v, int64_t step, float lr,
                          float beta1, float beta2, float eps) {
    if (!c || !params || !grad || !m || !v || step < 1) return PTYR_E_ARG;
    const double bc1 = 1.0 - std::pow((double)beta1, (double)step);
    const double bc2 = 1.0 - std::pow((double)beta2, (double)step);
    hipLaunchKernelGGL(k_adam, dim3(blocks_for(NPARAM)), dim3(256), 0, c->stream, params, grad, m, v, NPARAM, lr, beta1,
                       beta2, eps, (float)bc1, (float)std::sqrt(bc2));
    return launched();
}

ptyr_status ptyr_cnn_stitch(ptyr_cnn* c, const float* patches, const float* centres, int P, int H, int W, float* img) {
    if (!c || !img || H < 1 || W < 1 || P < 0) return PTYR_E_ARG;
    if (P > 0 && (!patches || !centres)) return PTYR_E_ARG;
    hipLaunchKernelGGL(k_stitch, dim3((unsigned)(((H + 15) / 16) * ((W + 15) / 16))), dim3(256), 0, c->stream, patches,
                       centres, P, H, W, img);
    return launched();
}

}  // extern "C"
