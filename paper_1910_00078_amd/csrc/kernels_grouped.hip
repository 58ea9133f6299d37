// Forward convolution with few input channels per group -- depthwise and grouped layers (Sec. IV-A of the
// MIOpen paper): up to 7 in the 16-bit types, 8 in fp32, square 3x3 and 5x5 filters at stride 1 or 2.
//
// With so short a reduction there is nothing for the 16-bit matrix pipe: the operands would be mostly padding.  What
// bounds these layers is device memory (depthwise 3x3: 4.5 FLOP per byte) and, in fp32 with several channels, the
// vector pipe.  So a thread owns a register tile -- KF filters of one group x TR output rows x PX
// output columns (PX elements = 16 bytes of y) -- and reads the input rows it needs straight from memory, PX +
// halo columns at a time; an input element is loaded once per (RS + (TR-1)*ST) / (TR*ST) rows by the thread and
// the rest of its uses are register reads.  No LDS, no barriers: consecutive lanes read consecutive pieces of
// a row, and rows shared by neighbouring threads come from the vector L1.
//
// All loads of one input channel are issued together: rows outside the image are read from the nearest row
// inside and masked, so no branch stands between the loads.  The last piece of an output row is moved left to
// end with the row, so every store is a whole 16-byte piece; the columns two pieces share are computed twice,
// with the same result.
#include "cvx_device.h"

#include <cstring>
#include <type_traits>

namespace cvx {

namespace grp {

typedef uint32_t u32_a2 __attribute__((aligned(2)));

struct Geom {
    int tasks;                 // threads with work
    int chunks, row_groups;    // pieces of PX columns per output row, groups of TR output rows per plane
    int fb_per_group, filter_blocks;   // blocks of KF filters per group and in all
    int cg, kg;
    Div31 by_chunks, by_rows, by_fb, by_group;
};

// c + a.lo * b.lo + a.hi * b.hi in fp32 (a, b: packed pairs of bf16 / fp16).
template <int DT>
__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c)
{
    if constexpr (DT == DT_BF16) return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, b), c, false);
    else return __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, a), __builtin_bit_cast(f16x2, b), c, false);
}

// One output's sum over the taps inside the image, one product after another.
template <int DT, int RS, int ST>
__device__ __forceinline__ float plain_sum(const ConvArgs& a, int cg, int n, int c0, int k, int p, int q)
{
    float acc = 0.0f;
#pragma unroll 1
    for (int c = 0; c < cg; ++c)
#pragma unroll 1
        for (int r = 0; r < RS; ++r) {
            const int h = p * ST - a.pad_h + r;
            if (h < 0 || h >= a.H) continue;
#pragma unroll 1
            for (int s = 0; s < RS; ++s) {
                const int v = q * ST - a.pad_w + s;
                if (v < 0 || v >= a.W) continue;
                acc = fmaf(Elem<DT>::load(a.x, (((size_t)n * a.C + c0 + c) * a.H + h) * a.W + v),
                           Elem<DT>::load(a.w, (((size_t)k * cg + c) * RS + r) * RS + s), acc);
            }
        }
    return acc;
}

// KF filters x TR rows x PX columns per thread; RS x RS filter; stride ST.
template <int DT, int RS, int ST, int KF, int TR>
__global__ void __launch_bounds__(256) grouped_kernel(ConvArgs a, Geom g)
{
    constexpr bool F32 = DT == DT_F32;
    constexpr int PX = F32 ? 4 : 8;                      // output columns: 16 bytes of y
    constexpr int NEL = (PX - 1) * ST + RS;              // input columns they need
    constexpr int ND = F32 ? NEL : (NEL + 1) / 2;        // dwords of a row piece
    constexpr int NLD = F32 ? NEL : 2 * ND;              // elements loaded (one may be past the needed ones)
    constexpr int NROW = (TR - 1) * ST + RS;
    typedef typename Elem<DT>::type elem_t;
    typedef typename std::conditional<F32, uint32_t, u32_a2>::type dword_e;   // a dword at any element's alignment

    warm_kernel_arguments<sizeof(ConvArgs) + sizeof(Geom)>();
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= g.tasks) return;
    const int t1 = g.by_chunks.div(t), chunk = t - t1 * g.chunks;
    const int t2 = g.by_rows.div(t1), rg = t1 - t2 * g.row_groups;
    const int n = g.by_fb.div(t2), fb = t2 - n * g.filter_blocks;
    const int grp = g.by_group.div(fb);
    const int k0 = grp * g.kg + (fb - grp * g.fb_per_group) * KF;
    const int nk = min(KF, (grp + 1) * g.kg - k0);
    const int q0 = a.Wo >= PX ? min(chunk * PX, a.Wo - PX) : 0;
    const int p0 = rg * TR;
    const int h0 = p0 * ST - a.pad_h, w0 = q0 * ST - a.pad_w;

    const elem_t* __restrict__ xg = (const elem_t*)a.x;
    const elem_t* __restrict__ wg = (const elem_t*)a.w;
    const long long total = (long long)a.N * a.C * a.H * a.W;

    uint32_t keep[ND];                                   // columns inside the image
#pragma unroll
    for (int d = 0; d < ND; ++d) {
        if constexpr (F32) {
            const int c = w0 + d;
            keep[d] = c >= 0 && c < a.W ? 0xffffffffu : 0u;
        } else {
            const int c = w0 + 2 * d;
            keep[d] = (c >= 0 && c < a.W ? 0x0000ffffu : 0u) | (c + 1 >= 0 && c + 1 < a.W ? 0xffff0000u : 0u);
        }
    }
#pragma unroll
    for (int d = 0; d < ND; ++d) asm volatile("" : "+v"(keep[d]));   // held as a mask, not as a condition (which would take two scalar registers each)
    int hr[NROW];                                        // row to read (clamped into the image), and whether it counts
    bool live[NROW];
#pragma unroll
    for (int i = 0; i < NROW; ++i) {
        const int h = h0 + i;
        live[i] = h >= 0 && h < a.H;
        hr[i] = min(max(h, 0), a.H - 1) * a.W + w0;
    }

    float acc[KF][TR][PX];
#pragma unroll
    for (int f = 0; f < KF; ++f)
#pragma unroll
        for (int i = 0; i < TR; ++i)
#pragma unroll
            for (int q = 0; q < PX; ++q) acc[f][i][q] = 0.0f;

    // One input channel: its row pieces and the KF filters' taps of it, as loaded.
    constexpr int NW = RS * RS, WD = F32 ? NW : NW / 2;  // taps; whole dwords of them (16-bit types: plus one odd element)
    struct Chan {
        uint32_t x[NROW][ND];
        uint32_t w[KF][WD];
        uint16_t w_last[KF];
        bool edge;
    };
    auto fetch = [&](int c, Chan& r) __attribute__((always_inline)) {
        const long long plane = ((long long)n * a.C + grp * g.cg + c) * a.H * a.W;
#pragma unroll
        for (int f = 0; f < KF; ++f) {
            const elem_t* p = wg + ((size_t)(k0 + min(f, nk - 1)) * g.cg + c) * NW;
#pragma unroll
            for (int d = 0; d < WD; ++d) r.w[f][d] = ((const dword_e*)p)[d];
            if constexpr (!F32) r.w_last[f] = ((const uint16_t*)p)[NW - 1];
        }
        // Only the first row piece of the tensor can start before it and only the last ones can end past it: those
        // are read from where they fit, and moved into place before they are used.
        r.edge = plane + hr[0] < 0 || plane + hr[NROW - 1] + NLD > total;
#pragma unroll
        for (int i = 0; i < NROW; ++i) {
            const elem_t* p = xg + min(max(plane + hr[i], 0LL), total - NLD);
#pragma unroll
            for (int d = 0; d < ND; ++d) r.x[i][d] = ((const dword_e*)p)[d];
        }
    };
    auto settle = [&](int c, Chan& r) __attribute__((always_inline)) {
        if (!r.edge) return;
        const long long plane = ((long long)n * a.C + grp * g.cg + c) * a.H * a.W;
#pragma unroll
        for (int i = 0; i < NROW; ++i) {
            const long long off = plane + hr[i];
            // elements the piece was moved by (by NLD or more, nothing of it is in the image)
            int by = (int)min(max(off - min(max(off, 0LL), total - NLD), (long long)-NLD), (long long)NLD);
            for (; by < 0; ++by)
#pragma unroll
                for (int d = ND - 1; d >= 0; --d) r.x[i][d] = F32 ? (d ? r.x[i][d - 1] : 0u) : __builtin_amdgcn_alignbit(r.x[i][d], d ? r.x[i][d - 1] : 0u, 16);
            for (; by > 0; --by)
#pragma unroll
                for (int d = 0; d < ND; ++d) r.x[i][d] = F32 ? (d + 1 < ND ? r.x[i][d + 1] : 0u) : __builtin_amdgcn_alignbit(d + 1 < ND ? r.x[i][d + 1] : 0u, r.x[i][d], 16);
        }
    };
    auto multiply = [&](const Chan& r) __attribute__((always_inline)) {
        if constexpr (F32) {
#pragma unroll
            for (int i = 0; i < NROW; ++i) {
                float xr[NLD];
#pragma unroll
                for (int d = 0; d < ND; ++d) xr[d] = live[i] ? __uint_as_float(r.x[i][d] & keep[d]) : 0.0f;
#pragma unroll
                for (int tr = 0; tr < TR; ++tr) {
                    const int rr = i - tr * ST;
                    if (rr < 0 || rr >= RS) continue;
#pragma unroll
                    for (int f = 0; f < KF; ++f)
#pragma unroll
                        for (int s = 0; s < RS; ++s)
#pragma unroll
                            for (int q = 0; q < PX; ++q)
                                acc[f][tr][q] = fmaf(xr[q * ST + s], __uint_as_float(r.w[f][rr * RS + s]), acc[f][tr][q]);
                }
            }
        } else {
            // Two taps per instruction (v_dot2_f32_{bf16,f16}: both products and the fp32 accumulator), on the packed
            // pairs as they were loaded and on the same pairs shifted by one element.  The odd last tap of a filter
            // row shares its pair with the tap before it, whose weight is zero there.
            constexpr int NP = RS / 2 + 1;                           // pairs per filter row
            uint32_t wp[KF][RS][NP];
            auto w_at = [&](int f, int j) { return j == NW - 1 ? (uint32_t)r.w_last[f] : (r.w[f][j / 2] >> (16 * (j & 1))) & 0xffffu; };
#pragma unroll
            for (int f = 0; f < KF; ++f)
#pragma unroll
                for (int rr = 0; rr < RS; ++rr) {
#pragma unroll
                    for (int j = 0; j < RS / 2; ++j) wp[f][rr][j] = w_at(f, rr * RS + 2 * j) | (w_at(f, rr * RS + 2 * j + 1) << 16);
                    wp[f][rr][RS / 2] = w_at(f, rr * RS + RS - 1) << 16;
                }
#pragma unroll
            for (int i = 0; i < NROW; ++i) {
                uint32_t even[ND], odd[ND];                          // elements (2d, 2d+1) and (2d+1, 2d+2)
#pragma unroll
                for (int d = 0; d < ND; ++d) even[d] = live[i] ? r.x[i][d] & keep[d] : 0u;
#pragma unroll
                for (int d = 0; d < ND; ++d) odd[d] = d + 1 < ND ? __builtin_amdgcn_alignbit(even[d + 1], even[d], 16) : even[d] >> 16;
#pragma unroll
                for (int tr = 0; tr < TR; ++tr) {
                    const int rr = i - tr * ST;
                    if (rr < 0 || rr >= RS) continue;
#pragma unroll
                    for (int f = 0; f < KF; ++f)
#pragma unroll
                        for (int j = 0; j < NP; ++j)
#pragma unroll
                            for (int q = 0; q < PX; ++q) {
                                const int e = q * ST + (j < RS / 2 ? 2 * j : RS - 2);
                                acc[f][tr][q] = dot2<DT>((e & 1) ? odd[e / 2] : even[e / 2], wp[f][rr][j], acc[f][tr][q]);
                            }
                }
            }
        }
    };
    if constexpr (KF == 1) {
        // depthwise: one channel, registers kept for more waves
        for (int c = 0; c < g.cg; ++c) {
            Chan r;
            fetch(c, r);
            settle(c, r);
            multiply(r);
        }
    } else {
        // the next channel is in flight while one is multiplied
        Chan ra, rb;
        fetch(0, ra);
        for (int c = 0; c < g.cg; c += 2) {
            if (c + 1 < g.cg) fetch(c + 1, rb);
            settle(c, ra);
            multiply(ra);
            if (c + 1 >= g.cg) break;
            if (c + 2 < g.cg) fetch(c + 2, ra);
            settle(c + 1, rb);
            multiply(rb);
        }
    }

    const bool has_bn = a.bn_scale != nullptr;
    elem_t* __restrict__ yg = (elem_t*)a.y;
    float any = 0.0f;                                    // a NaN if one of the sums is
    auto write_out = [&](auto&& act_fn) __attribute__((always_inline)) {
#pragma unroll
        for (int f = 0; f < KF; ++f) {
            if (f >= nk) break;
            const ChannelAffine aff = channel_affine<DT>(a, k0 + f);
#pragma unroll
            for (int tr = 0; tr < TR; ++tr) {
                if (p0 + tr >= a.Ho) break;
                elem_t* dst = yg + (((size_t)n * a.K + k0 + f) * a.Ho + p0 + tr) * a.Wo + q0;
                float v[PX];
#pragma unroll
                for (int q = 0; q < PX; ++q) any += acc[f][tr][q];
#pragma unroll
                for (int q = 0; q < PX; ++q) v[q] = act_fn(has_bn ? fmaf(acc[f][tr][q], aff.mul, aff.add) : acc[f][tr][q] + aff.add);
                uint32_t o[4];
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    if constexpr (F32) o[d] = __float_as_uint(v[d]);
                    else o[d] = pack2<DT>(v[2 * d], v[2 * d + 1]);
                }
                if (a.Wo >= PX) {
#pragma unroll
                    for (int d = 0; d < 4; ++d) ((dword_e*)dst)[d] = o[d];
                } else {
#pragma unroll
                    for (int q = 0; q < PX; ++q)
                        if (q < a.Wo) {
                            if constexpr (F32) dst[q] = v[q];
                            else dst[q] = (elem_t)(o[q >> 1] >> ((q & 1) * 16));
                        }
                }
            }
        }
    };
    if (a.act == ACT_RELU) write_out([](float v) { return fmaxf(v, 0.0f); });
    else if (a.act == ACT_IDENTITY) write_out([](float v) { return v; });
    else if (a.act == ACT_LEAKY_RELU) write_out([&](float v) { return v > 0.0f ? v : a.alpha * v; });
    else write_out([&](float v) { return activate(v, a.act, a.alpha); });

    // The loops above multiply zeros that are no part of the convolution: columns and rows outside the image, and the
    // other tap of an odd tap's pair.  Against an infinite weight or input such a product is a NaN.  So outputs whose
    // sums hold a NaN (an infinity or a NaN is among the operands; nothing else makes one) are written again, summed one
    // tap at a time; finding them costs one addition for each output.
    if (any != any) {
#pragma unroll 1
        for (int f = 0; f < nk; ++f) {
            const ChannelAffine aff = channel_affine<DT>(a, k0 + f);
#pragma unroll 1
            for (int p = p0; p < min(p0 + TR, a.Ho); ++p)
#pragma unroll 1
                for (int q = q0; q < min(q0 + PX, a.Wo); ++q)
                    Elem<DT>::store(yg, (((size_t)n * a.K + k0 + f) * a.Ho + p) * a.Wo + q,
                                    finish(plain_sum<DT, RS, ST>(a, g.cg, n, grp * g.cg, k0 + f, p, q), aff, has_bn, a.act, a.alpha));
        }
    }
}

struct Variant {
    const char* name[3];       // by data type
    int RS, ST, KF, TR;
    void (*kern[3])(ConvArgs, Geom);
};

#define GRP_VARIANT(RS, ST, KF, TR)                                                                                              \
    {{"grouped_f32_" #RS "x" #RS "_s" #ST "_k" #KF "r" #TR, "grouped_f16_" #RS "x" #RS "_s" #ST "_k" #KF "r" #TR,                  \
      "grouped_bf16_" #RS "x" #RS "_s" #ST "_k" #KF "r" #TR},                                                                     \
     RS, ST, KF, TR,                                                                                                             \
     {grouped_kernel<DT_F32, RS, ST, KF, TR>, grouped_kernel<DT_F16, RS, ST, KF, TR>, grouped_kernel<DT_BF16, RS, ST, KF, TR>}}

// name: grouped_<type>_<filter>_s<stride>_k<filters per thread>r<rows per thread>; for each filter and stride the larger
// register tiles first
const Variant kVariants[] = {
    GRP_VARIANT(3, 1, 4, 2), GRP_VARIANT(3, 1, 4, 1), GRP_VARIANT(3, 1, 1, 4), GRP_VARIANT(3, 1, 1, 2), GRP_VARIANT(3, 1, 1, 1),
    GRP_VARIANT(3, 2, 4, 1), GRP_VARIANT(3, 2, 1, 2), GRP_VARIANT(3, 2, 1, 1),
    GRP_VARIANT(5, 1, 1, 4), GRP_VARIANT(5, 1, 1, 1), GRP_VARIANT(5, 2, 1, 2), GRP_VARIANT(5, 2, 1, 1),
};
constexpr int kNumVariants = sizeof(kVariants) / sizeof(kVariants[0]);

bool fill(const ConvArgs& a, const Variant& v, Geom* out)
{
    const int PX = a.dtype == DT_F32 ? 4 : 8;
    Geom g;
    memset(&g, 0, sizeof g);
    g.cg = a.C / a.groups;
    g.kg = a.K / a.groups;
    g.chunks = (a.Wo + PX - 1) / PX;
    g.row_groups = (a.Ho + v.TR - 1) / v.TR;
    g.fb_per_group = (g.kg + v.KF - 1) / v.KF;
    const long long fbs = (long long)g.fb_per_group * a.groups;
    const long long tasks = (long long)g.chunks * g.row_groups * fbs * a.N;
    if (fbs > 0x7fffffffLL || tasks > 0x7fffff00LL) return false;
    g.filter_blocks = (int)fbs;
    g.tasks = (int)tasks;
    g.by_chunks = div31(g.chunks);
    g.by_rows = div31(g.row_groups);
    g.by_fb = div31(g.filter_blocks);
    g.by_group = div31(g.fb_per_group);
    *out = g;
    return true;
}

}  // namespace grp

bool grouped_plan(const ConvArgs& a, const PlanEnv& env, LaunchPlan* out)
{
    static_assert(sizeof(grp::Geom) <= sizeof(out->geom), "geometry does not fit the plan");
    const int cg = a.C / a.groups, kg = a.K / a.groups;
    if (a.R != a.S || a.dil_h != 1 || a.dil_w != 1 || a.stride_h != a.stride_w) return false;
    if ((long long)a.H * a.W >= (1LL << 30)) return false;                  // row offsets inside a plane stay in int
    if ((long long)a.N * a.C * a.H * a.W < 32) return false;                // a row piece fits the tensor
    // Outputs a few pixels wide fill a corner of the 16-byte pieces, and most of their filters' taps lie in the padding, which
    // this kernel reads and multiplies like the rest and the direct kernel skips.  16-bit, direct against this: width 1
    // 5.3 and 28.0 us (14x168x1x1 K=10752 5x5, 3 channels), and 16 to 8 on the middle one of 135 drawn layers; width 2 and 3
    // slower with the fewest channels (1.0-1.4x), faster above; from width 4 on faster (1.4-3x).  fp32 pieces are half as wide: 260 drawn layers of width 1 take 0.2-1.0 of the time
    // on the direct kernel where the image is one pixel wide, or the filter 5x5, and 1.0-1.3 of it for 3x3 on two pixels.
    const long long work = (long long)a.N * a.K * a.Ho * a.Wo * cg * a.R * a.S;
    const bool direct_instead = a.dtype != DT_F32 || work < kTiledF32Work;    // else the tiled fp32 kernel
    const bool unit3 = a.stride_h == 1 && a.R == 3;
    const int few = a.dtype == DT_F32 || a.Wo >= 4 ? 1 : a.Wo == 3 ? (a.stride_h == 1 || a.R == 5 ? 1 : 3) : unit3 ? 2 : 3;
    const bool one = a.Wo == 1 && !(a.dtype == DT_F32 && a.W > 1 && (a.R == 3 || !direct_instead));
    // The direct kernel deals the channels of small problems over lanes from 8 on (4x40x17x17, 5 groups, stride 2: 4.4 us
    // there, 6.2 here).
    if (!env.pin && cg >= 8 && direct_instead && (long long)a.N * a.K * a.Ho * a.Wo <= kDirectSplitOutputs) return false;
    // 16-bit types with 8 or more channels per group go to the matrix pipe (8 channels: 6.3 against 15.7 us on
    // 15x96x19x19 at stride 2, 12.1 against 38 us on 8x320x51x51 with 16; with 4 channels 8.5 us here against 40 on
    // the direct kernel for 30x48x31x31); fp32 stays on the vector pipe up to 8.
    if (!env.pin && cg > (a.dtype == DT_F32 ? 8 : 7)) return false;
    const grp::Variant* bv = nullptr;
    grp::Geom bg;
    for (int i = 0; i < grp::kNumVariants; ++i) {
        const grp::Variant& v = grp::kVariants[i];
        if (v.RS != a.R || v.ST != a.stride_h) continue;
        grp::Geom g;
        if (!grp::fill(a, v, &g)) continue;
        if (env.pin) {
            if (strcmp(env.pin, v.name[a.dtype]) != 0) continue;
        } else {
            if (v.KF > 1 && kg == 1) continue;
            // The largest register tile that still gives the chip 160 threads per compute unit: below that the
            // longer chain of a thread costs more than the loads it spares (depthwise 3x3, us: 32x128x28x28 four
            // rows 6.4, two 6.9, one 7.5 with 448 threads per unit at four rows; 32x96x7x7 6.1, 4.0, 3.7 with 24).
            if (bv && bg.tasks >= 160LL * env.cus) continue;
        }
        bv = &v;
        bg = g;
    }
    if (!bv) return false;
    // (tiles of four filters, which only large problems run, gain from width 2 on whatever the channels, 1.1-3x over 8 drawn
    // layers, and with 6 channels of two pixels: 17x2128x2x2 K=34048 3x3 stride 2 40.5 us, 71.5 direct)
    const bool four = bv->KF == 4 && (a.Wo > 1 || (a.W > 1 && cg >= 6));
    if (!env.pin && !four && (one || cg < few)) return false;
    out->id = KID_GROUPED;
    out->name = bv->name[a.dtype];
    out->variant = (int)(bv - grp::kVariants);
    out->grid_x = (unsigned)((bg.tasks + 255) / 256);
    out->grid_y = 1;
    out->block = 256;
    out->lds = 0;
    {
        // fitted to 700 timed fp32 layers, met within 19 % rms: multiply-adds at 27 a clock and compute unit, a load of an
        // element by a thread each 25 ns / 1000, and a chain of the channels
        const double threads = (double)bg.tasks * cg, loads = ((bv->TR - 1) * bv->ST + bv->RS) * (3.0 * bv->ST + bv->RS) + bv->KF * bv->RS * bv->RS;
        out->us = 3.6 + threads * bv->KF * bv->TR * 4 * bv->RS * bv->RS / 27.5e6 + threads * loads / env.cus * 25e-6 + 0.2 * cg;
    }
    memcpy(out->geom, &bg, sizeof bg);
    return true;
}

hipError_t grouped_launch(const ConvArgs& a, const LaunchPlan& p, hipStream_t s)
{
    grp::Geom g;
    memcpy(&g, p.geom, sizeof g);
    hipLaunchKernelGGL(grp::kVariants[p.variant].kern[a.dtype], dim3(p.grid_x), dim3(p.block), 0, s, a, g);
    return hipGetLastError();
}

}  // namespace cvx
