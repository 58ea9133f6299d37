// Generic direct forward convolution: one thread per output element, any filter size, padding,
// stride, dilation and group count, all three data types, fp32 accumulation, fused epilogue.
// This is the correctness net behind the specialised kernels (the "direct" family of Sec. IV-A of
// the MIOpen paper in its plainest form), plus the separate bias / activation operators that the
// unfused path of Sec. V uses.
#include "cvx_device.h"

namespace cvx {

// CS = 1: one thread per output.  CS = 8: eight neighbouring lanes share an output, each taking every
// eighth channel, and add their partial sums with three lane exchanges: small problems are a chain of
// dependent loads per thread, and this cuts the chain by eight.
template <int DT, int CS>
__global__ void __launch_bounds__(256) direct_conv_kernel(ConvArgs a)
{
    warm_kernel_arguments<sizeof(ConvArgs)>();
    const long long total = (long long)a.N * a.K * a.Ho * a.Wo;
    const int cg = a.C / a.groups;
    const int kg = a.K / a.groups;
    const bool has_bn = a.bn_scale != nullptr;
    const long long tid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const int part = (int)(tid % CS);
    for (long long o = tid / CS; o < total; o += (long long)gridDim.x * blockDim.x / CS) {
        const int q = (int)(o % a.Wo);
        long long t = o / a.Wo;
        const int p = (int)(t % a.Ho);
        t /= a.Ho;
        const int k = (int)(t % a.K);
        const int n = (int)(t / a.K);
        const int c0 = (k / kg) * cg;
        const int h0 = p * a.stride_h - a.pad_h;
        const int w0 = q * a.stride_w - a.pad_w;
        float acc = 0.0f;
        for (int c = part; c < cg; c += CS) {
            const size_t xbase = ((size_t)n * a.C + (c0 + c)) * a.H * a.W;
            const size_t wbase = ((size_t)k * cg + c) * a.R * a.S;
            for (int r = 0; r < a.R; ++r) {
                const int h = h0 + r * a.dil_h;
                if (h < 0 || h >= a.H) continue;
                for (int s = 0; s < a.S; ++s) {
                    const int wv = w0 + s * a.dil_w;
                    if (wv < 0 || wv >= a.W) continue;
                    acc = fmaf(Elem<DT>::load(a.x, xbase + (size_t)h * a.W + wv),
                               Elem<DT>::load(a.w, wbase + (size_t)r * a.S + s), acc);
                }
            }
        }
        if constexpr (CS > 1) {
            // the CS lanes of an output are neighbours in one wave and reach this point together
#pragma unroll
            for (int d = 1; d < CS; d <<= 1) acc += __shfl_xor(acc, d);
            if (part != 0) continue;
        }
        const ChannelAffine ca = channel_affine<DT>(a, k);
        Elem<DT>::store(a.y, (size_t)o, finish(acc, ca, has_bn, a.act, a.alpha));
    }
}

bool direct_plan(const ConvArgs& a, const PlanEnv&, LaunchPlan* out)
{
    const long long total = (long long)a.N * a.K * a.Ho * a.Wo;
    const bool split = total <= kDirectSplitOutputs && a.C / a.groups >= 8;      // latency-bound sizes
    long long blocks = (total * (split ? 8 : 1) + 255) / 256;
    if (blocks > (1 << 20)) blocks = 1 << 20;           // grid-stride loop covers the rest
    out->id = KID_DIRECT;
    out->name = a.dtype == DT_F32 ? "direct_f32" : a.dtype == DT_F16 ? "direct_f16" : "direct_bf16";
    out->variant = split ? 8 : 1;
    out->grid_x = (unsigned)blocks;
    out->grid_y = 1;
    out->block = 256;
    out->lds = 0;
    return true;
}

hipError_t direct_launch(const ConvArgs& a, const LaunchPlan& p, hipStream_t s)
{
    const dim3 grid(p.grid_x), block(p.block);
    const bool split = p.variant == 8;
#define CVX_LAUNCH_DIRECT(DT)                                                                   \
    do {                                                                                        \
        if (split) hipLaunchKernelGGL((direct_conv_kernel<DT, 8>), grid, block, 0, s, a);       \
        else hipLaunchKernelGGL((direct_conv_kernel<DT, 1>), grid, block, 0, s, a);             \
    } while (0)
    switch (a.dtype) {
    case DT_F32:  CVX_LAUNCH_DIRECT(DT_F32); break;
    case DT_F16:  CVX_LAUNCH_DIRECT(DT_F16); break;
    case DT_BF16: CVX_LAUNCH_DIRECT(DT_BF16); break;
    default: return hipErrorInvalidValue;
    }
#undef CVX_LAUNCH_DIRECT
    return hipGetLastError();
}

// ---- unfused element-wise operators --------------------------------------------------------------
// One read and one write of y each, bound by memory.  Each thread handles kEwUnroll pieces of 16 bytes (8 fp16/bf16
// or 4 fp32 elements), all loaded before the first is used, when y is 16-byte aligned (`vec` = elements per
// piece, else 1); the elements past the last whole piece are done one by one.  In the bias kernel a piece may
// straddle two channels (planes that are not a multiple of it), never three: planes smaller than a piece go one by
// one.  The channel of a piece comes from two multiply-high divisions; with 64-bit divisions, one piece a thread and
// straddling planes element by element, the bias took 13.0 us on 32x512x28x28 bf16 and ReLU 8.2; these take 9.4 and 6.8.
constexpr int kEwUnroll = 4;

template <int DT, typename F>      // f(value, element of the piece)
__device__ __forceinline__ u32x4 ew_piece(u32x4 q, F&& f)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if constexpr (DT == DT_F32) q[e] = __float_as_uint(f(__uint_as_float(q[e]), e));
        else q[e] = pack2<DT>(f(bits16_to_f32<DT>((uint16_t)(q[e] & 0xffffu)), 2 * e), f(bits16_to_f32<DT>((uint16_t)(q[e] >> 16)), 2 * e + 1));
    }
    return q;
}

// piece_fn(first element, piece) and one_fn(element index, value) give the new values.
template <int DT, typename P, typename O>
__device__ __forceinline__ void ew_apply(void* y, int total, int vec, P&& piece_fn, O&& one_fn)
{
    const int nvec = vec > 1 ? total / vec : 0;
    const int first = blockIdx.x * (256 * kEwUnroll) + threadIdx.x;
    u32x4* yv = (u32x4*)y;
    if (first < nvec) {
        u32x4 q[kEwUnroll];
#pragma unroll
        for (int u = 0; u < kEwUnroll; ++u) q[u] = yv[min(first + u * 256, nvec - 1)];
#pragma unroll
        for (int u = 0; u < kEwUnroll; ++u)
            if (first + u * 256 < nvec) yv[first + u * 256] = piece_fn((first + u * 256) * vec, q[u]);
    }
    const long long nthreads = (long long)gridDim.x * 256;
    for (long long i = (long long)nvec * vec + blockIdx.x * 256 + threadIdx.x; i < total; i += nthreads)
        Elem<DT>::store(y, (size_t)i, one_fn((int)i, Elem<DT>::load(y, (size_t)i)));
}

template <int DT>
__global__ void __launch_bounds__(256) bias_add_kernel(void* y, const void* bias, int bias_f32, int K, int HW,
                                                        Div31 by_k, Div31 by_hw, int total, int vec)
{
    const auto bias_of = [&](int k) { return bias_f32 ? ((const float*)bias)[k] : Elem<DT>::load(bias, k); };
    ew_apply<DT>(
        y, total, vec,
        [&](int e0, u32x4 q) {
            const int plane = by_hw.div(e0), k = plane - by_k.div(plane) * K;
            const int left = HW - (e0 - plane * HW);                  // elements of the piece (or more) in this plane
            const float b0 = bias_of(k), b1 = left < vec ? bias_of(k + 1 == K ? 0 : k + 1) : b0;
            return ew_piece<DT>(q, [&](float t, int e) { return t + (e < left ? b0 : b1); });
        },
        [&](int i, float t) {
            const int plane = by_hw.div(i);
            return t + bias_of(plane - by_k.div(plane) * K);
        });
}

template <int DT>
__global__ void __launch_bounds__(256) activation_kernel(void* y, int act, float alpha, int total, int vec)
{
    const auto one = [&](int, float t) { return activate(t, act, alpha); };
    if (act == ACT_RELU)
        ew_apply<DT>(y, total, vec, [](int, u32x4 q) { return ew_piece<DT>(q, [](float t, int) { return fmaxf(t, 0.0f); }); }, one);
    else
        ew_apply<DT>(y, total, vec, [&](int, u32x4 q) { return ew_piece<DT>(q, [&](float t, int) { return activate(t, act, alpha); }); }, one);
}

static int ew_vector(const void* y, int dtype)
{
    return ((uintptr_t)y & 15) ? 1 : (dtype == DT_F32 ? 4 : 8);
}

// With pieces the grid covers them exactly; the (few) single elements past them, or all of them, are strided over it.
static unsigned ew_blocks(int total, int vec)
{
    const long long per = 256LL * (vec > 1 ? kEwUnroll * vec : 1);
    const long long b = (total + per - 1) / per;
    return (unsigned)(vec > 1 || b < 8192 ? b : 8192);
}

hipError_t launch_bias_add(void* y, const void* bias, int dtype, int bias_f32, int N, int K, int HW, hipStream_t s)
{
    const int total = (int)((long long)N * K * HW);              // tensors have fewer than 2^31 elements
    int vec = ew_vector(y, dtype);
    if (HW < vec) vec = 1;
    const Div31 by_k = div31(K), by_hw = div31(HW);
    const dim3 grid(ew_blocks(total, vec)), block(256);
    switch (dtype) {
    case DT_F32:  hipLaunchKernelGGL(bias_add_kernel<DT_F32>, grid, block, 0, s, y, bias, bias_f32, K, HW, by_k, by_hw, total, vec); break;
    case DT_F16:  hipLaunchKernelGGL(bias_add_kernel<DT_F16>, grid, block, 0, s, y, bias, bias_f32, K, HW, by_k, by_hw, total, vec); break;
    case DT_BF16: hipLaunchKernelGGL(bias_add_kernel<DT_BF16>, grid, block, 0, s, y, bias, bias_f32, K, HW, by_k, by_hw, total, vec); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_activation(void* y, int dtype, int act, float alpha, long long count, hipStream_t s)
{
    const int total = (int)count;
    const int vec = ew_vector(y, dtype);
    const dim3 grid(ew_blocks(total, vec)), block(256);
    switch (dtype) {
    case DT_F32:  hipLaunchKernelGGL(activation_kernel<DT_F32>, grid, block, 0, s, y, act, alpha, total, vec); break;
    case DT_F16:  hipLaunchKernelGGL(activation_kernel<DT_F16>, grid, block, 0, s, y, act, alpha, total, vec); break;
    case DT_BF16: hipLaunchKernelGGL(activation_kernel<DT_BF16>, grid, block, 0, s, y, act, alpha, total, vec); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace cvx
