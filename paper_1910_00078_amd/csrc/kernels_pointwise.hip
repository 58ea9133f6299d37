// Pointwise (1x1 filter, no padding, column stride 1 or 2) forward convolution on bf16 / fp16 MFMA for
// gfx950 (MI355X), with the bias / batch-norm / activation epilogue of Sec. V of the MIOpen paper
// applied to the accumulators before the single store.
//
// A 1x1 convolution is the GEMM  Y[n][k][pix] = sum_c Wt[k][c] * X[n][c][pix]  and, at the channel
// counts of residual networks, is bound by device-memory bandwidth, not by the matrix pipe.  The
// kernel is therefore organised around keeping the memory system busy without pause:
//
//   Persistent blocks   one block per compute unit; block b owns a contiguous span of the flattened
//                       (image, pixel) axis, so the blocks carry equal bytes, and walks it in pixel
//                       tiles.  The filters and epilogue constants are loaded into LDS once.
//   Direct-to-LDS loads two loader waves stream the input with global_load_lds (16 bytes per lane,
//                       no registers in between) into a ring of NS stage buffers, each CC channel
//                       rows x PT pixels in the tensor's own NCHW order.  The ring runs ahead of the
//                       multiply across tile boundaries; the loaders wait on their own load counter
//                       with an exact outstanding-load count, so NS-2 stages stay in flight.
//   Transposing reads   NCHW keeps pixels contiguous but the MFMA pixel operand wants 8 consecutive
//                       channels per lane.  ds_read_b64_tr_b16 does that exchange inside the LDS
//                       read (16 lanes x 4 pixels in, 4 channels x 1 pixel per lane out), so nothing
//                       is transposed in registers.  The 64-byte chunks of a stage row are XOR-
//                       swizzled with the row index so the four rows a read touches fall on
//                       different banks; the swizzle costs nothing, the loader just picks the global
//                       address that belongs at each LDS position.
//   Wave-private stores each multiply wave stages its 64-pixel x 64-filter results in its own LDS
//                       patch and writes them out itself as 128-byte rows; no block-wide barrier
//                       sits between the multiply and the store, and the loaders never wait for a
//                       store.
//   Chunks              the pixel axis is cut into chunks of 8 input pixels that lie in one line (a line is
//                       an image, or one needed image row under a stride).  A line's last chunk is moved back
//                       to end with the line, so no load leaves the tensor: its pixels are computed twice,
//                       with the same result.  Chunks then start at any 2-byte address, which the direct-to-LDS
//                       loads take at a lower rate that is still above device memory's.  Lines shorter than a
//                       chunk are left to the implicit-GEMM kernel.
//   Column stride 2     whole chunks are loaded (their lines are fetched anyway) and multiplied; the epilogue
//                       drops the odd columns.  Twice the matrix work is still below the memory time: against
//                       the implicit-GEMM kernel, which transposed both halves in registers,
//                       32x256x56x56 K=512 went from 99 to 28 us.
//   Ragged channels     the last stage's missing channel rows are read from 16 bytes of zeros.
#include "cvx_device.h"

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <type_traits>

namespace cvx {

namespace pw {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) unsigned char lds_byte;

struct Geom {
    int HW;            // input pixels per image
    int total_px;      // pixel slots: 8 x chunks
    int span;          // pixel slots per block, a multiple of the tile width
    int stages_per_tile;   // C / CC, rounded up
    int cpl, lpi;      // chunks per line, lines per image
    Div31 by_cpl, by_lpi, by_kblocks;
    int tail;          // first pixel of a line's last chunk
    int odd_tail;      // 1: that chunk's outputs are its odd pixels (column stride 2 on an odd image width)
    int x_line, y_line;    // input / output elements from one line to the next
    int y_aligned;     // 1: every chunk of y is 16 bytes on a 16-byte boundary
    int kblocks;       // filter blocks
    int x_streaming;   // 1: input loads carry the nontemporal hint
    int w_off, ca_off, out_off, ring_off;   // LDS byte offsets
};

// Transposing LDS read.  Within each group of 16 lanes, lane s supplies the address of 4 consecutive
// 16-bit elements; with K = s / 4 and M = 4 * (s % 4) + {0..3} naming those elements, lane i of the
// group receives the four elements (K = 0..3, M = i).  The low three address bits are ignored.
__device__ __forceinline__ u32x2 lds_read_tr16(const unsigned char* p)
{
    const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(lds_byte*)p);
    return __builtin_bit_cast(u32x2, v);
}

// All of a wave's LDS reads have returned; then the block barrier.  Deliberately not a fence: the
// loader waves keep device loads in flight across it and the multiply waves keep stores in flight.
__device__ __forceinline__ void stage_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <int N>
__device__ __forceinline__ void wait_loads_outstanding()
{
    static_assert(N >= 0 && N <= 63, "vmcnt is a 6-bit counter");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

constexpr int ND = 2;             // loader waves
constexpr int OPITCH = 136;       // bytes per filter row of a wave's output patch: 64 pixels + 4 (bank spread)

// What a loader lane reads for channels past the last one: 16 bytes of zeros.
static __device__ const uint32_t kZeros[4] __attribute__((aligned(16))) = {0u, 0u, 0u, 0u};

// WM x WN multiply waves, each TM pixel sub-tiles (32 pixels) x TN filter sub-tiles (32 filters);
// CC channels per stage; NS ring slots.
// SW: column stride.
// WS: the filters are not kept in LDS but streamed with the input, a ring slot holding both parts of a stage: for channel
// counts whose filters leave no room for a wide tile (41x758x29x29 K=213: 102 us with 32 resident filters a block, 51 with 128 streamed ones).
template <int DT, int WM, int WN, int TM, int TN, int CC, int NS, int SW, bool WS>
__global__ void __launch_bounds__((WM * WN + ND) * 64)
pointwise_kernel(ConvArgs a, Geom g)
{
    constexpr int NCW = WM * WN;
    constexpr int THREADS = (NCW + ND) * 64;
    constexpr int PT = WM * TM * 32;                 // pixels per tile
    constexpr int KT = WN * TN * 32;                 // filters per block
    constexpr int ROWB = PT * 2;                     // bytes per channel row of a stage
    constexpr int STAGE = CC * ROWB;
    constexpr int INSTR = STAGE / 1024;              // wave-wide 16-byte-per-lane loads per stage
    constexpr int U = INSTR / ND;                    // of which each loader wave issues this many
    constexpr int RPI = 1024 / ROWB;                 // channel rows one such load covers
    constexpr int KSTEPS = CC / 16;
    constexpr int WSTAGE = WS ? KT * CC * 2 : 0;     // streamed filters of a stage
    constexpr int SLOT = STAGE + WSTAGE;
    constexpr int UW = WSTAGE / 1024 / ND;           // and their loads per loader wave
    static_assert(WSTAGE % (1024 * ND) == 0 && (NS - 2) * (U + UW) <= 63, "whole loads, countable");
    static_assert(PT >= 128 && PT <= 512 && (PT & (PT - 1)) == 0, "swizzle needs >= 4 chunks of 64 bytes per row");
    static_assert(INSTR % ND == 0 && (ND * RPI) % 4 == 0, "a lane keeps one swizzle phase");
    static_assert(TM % 2 == 0, "output patches hold two pixel sub-tiles");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

    CVX_TRACE_MARK(0);
    warm_kernel_arguments<sizeof(ConvArgs) + sizeof(Geom)>();
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int HW = g.HW;
    // Blocks that share a span (and differ in the filter block) follow each other on one XCD, so that its L2
    // fetches their input once.
    int pb = blockIdx.x, kb = 0;
    if (g.kblocks > 1) {
        const int j = blockIdx.x >> 3, pj = g.by_kblocks.div(j);
        kb = j - pj * g.kblocks;
        pb = pj * 8 + (blockIdx.x & 7);
    }
    const int k0 = kb * KT;

    // this block's span of the flattened (image, line, chunk) axis
    const int Gb = pb * g.span;
    if (Gb >= g.total_px) return;                                    // whole block, before any barrier
    const int Ge = min(Gb + g.span, g.total_px);
    const int n_tiles = (Ge - Gb + PT - 1) / PT;
    const int SPT = g.stages_per_tile;
    const int T = n_tiles * SPT;                                     // stages this block multiplies

    unsigned char* ws = smem + g.w_off;               // written by the multiply waves' prologue
    float* cas = (float*)(smem + g.ca_off);
    unsigned char* ring = smem + g.ring_off;

    if (wave >= NCW) {
        // =========================================================================================
        // loader waves
        // =========================================================================================
        const int dw = wave - NCW;
        const uint16_t* __restrict__ xg = (const uint16_t*)a.x;
        // LDS position of this lane inside a load: channel row (relative) and 16-byte unit of the row
        const int lane_row = (lane * 16) / ROWB;
        const int u16 = ((lane * 16) % ROWB) >> 4;
        const int rowlow = (dw * RPI + lane_row) & 3;               // row & 3, the same for every load of this wave
        const int px = (((u16 >> 2) ^ rowlow) << 5) + ((u16 & 3) << 3);   // pixel of the tile that belongs here
        const int Glast = Ge - 8;                                    // last whole 8-pixel chunk of the span

        int ld_tile = 0, ld_st = 0, ld_slot = 0;
        long long goff = 0;
        auto issue_stage = [&]() __attribute__((always_inline)) {
            if (ld_st == 0) {
                // pixels past the span re-read its last chunk: every lane always loads, so the
                // outstanding-load arithmetic below is exact, and the address stays inside x
                const int q = min(Gb + ld_tile * PT + px, Glast) >> 3;
                const int line = g.by_cpl.div(q), j = q - line * g.cpl;
                const int n = g.by_lpi.div(line);
                goff = (long long)n * a.C * HW + (long long)(line - n * g.lpi) * g.x_line + (j == g.cpl - 1 ? g.tail : 8 * j);
            }
            const int c_lane = ld_st * CC + dw * RPI + lane_row;
            const uint16_t* src = xg + goff + (long long)c_lane * HW;
            lds_byte* dst = (lds_byte*)(ring + ld_slot * SLOT + dw * 1024);
            if ((ld_st + 1) * CC > a.C) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const void* p = c_lane + u * (ND * RPI) < a.C ? (const void*)(src + (long long)u * (ND * RPI) * HW) : (const void*)kZeros;
                    __builtin_amdgcn_global_load_lds(p, (__attribute__((address_space(3))) void*)(dst + u * ND * 1024), 16, 0, 0);
                }
            } else
            // The streaming hint keeps a large input from displacing the output lines waiting in L2; it
            // pays when the input is the larger tensor.
            if (g.x_streaming) {
#pragma unroll
                for (int u = 0; u < U; ++u)
                    __builtin_amdgcn_global_load_lds((const void*)(src + (long long)u * (ND * RPI) * HW),
                                                     (__attribute__((address_space(3))) void*)(dst + u * ND * 1024), 16, 0, 2);
            } else {
#pragma unroll
                for (int u = 0; u < U; ++u)
                    __builtin_amdgcn_global_load_lds((const void*)(src + (long long)u * (ND * RPI) * HW),
                                                     (__attribute__((address_space(3))) void*)(dst + u * ND * 1024), 16, 0, 0);
            }
            if constexpr (WS) {
                // [octet][filter] x 16 bytes, filter rows past K repeating the last.  A row's last, partial octet is
                // read as its last 8 channels (the multiply waves shift them down), so no load leaves the tensor.
                const uint16_t* __restrict__ wg = (const uint16_t*)a.w;
#pragma unroll
                for (int u = 0; u < UW; ++u) {
                    const int e = (u * ND + dw) * 64 + lane, kl = e % KT, c = ld_st * CC + e / KT * 8;
                    const uint16_t* row = wg + (size_t)min(k0 + kl, a.K - 1) * a.C;
                    const void* p = c < a.C ? (const void*)(row + min(c, a.C - 8)) : (const void*)kZeros;
                    __builtin_amdgcn_global_load_lds(p, (__attribute__((address_space(3))) void*)(dst + STAGE + u * ND * 1024), 16, 0, 0);
                }
            }
            if (++ld_st == SPT) { ld_st = 0; ++ld_tile; }
            if (++ld_slot == NS) ld_slot = 0;
        };

        const int ahead = min(NS - 1, T);
        for (int s = 0; s < ahead; ++s) issue_stage();
        CVX_TRACE_MARK_T(10, NCW * 64);
        if (ahead == NS - 1) wait_loads_outstanding<(NS - 2) * (U + UW)>();
        else wait_loads_outstanding<0>();
        CVX_TRACE_MARK_T(11, NCW * 64);
        stage_barrier();                                             // filters, constants and stage 0 are in LDS
        for (int t = 0; t < T; ++t) {
            // slot (t-1) % NS was multiplied in the previous pass; refill it with stage t+NS-1, then
            // wait until stage t+1 has landed (at most NS-2 younger stages still in flight)
            if (t + NS - 1 < T) {
                issue_stage();
                wait_loads_outstanding<(NS - 2) * (U + UW)>();
            } else {
                wait_loads_outstanding<0>();
            }
            stage_barrier();
        }
    } else {
        // =========================================================================================
        // multiply waves
        // =========================================================================================
        const int l32 = lane & 31, h = lane >> 5;
        const int gq = lane >> 4, s16 = lane & 15;
        const int wm = wave / WN, wn = wave % WN;
        const bool has_bn = a.bn_scale != nullptr;

        // pixel operand: byte offset inside a stage for sub-tile tm, k-step 0, first half
        int xa[TM];
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            const int jt = wm * TM + tm;
            xa[tm] = (8 * h + (s16 >> 2)) * ROWB + ((jt ^ (s16 >> 2)) << 6) + ((gq & 1) << 5) + ((s16 & 3) << 3);
        }
        const unsigned char* wl = ws + ((size_t)h * KT + (wn * TN) * 32 + l32) * 16;
        unsigned char* ow = smem + g.out_off + wave * (TN * 32 * OPITCH);

        // ---- once per block (the loaders are already streaming the input): filters into LDS as
        //      [channel octet][filter] x 16 bytes, by direct-to-LDS loads whose per-lane device address
        //      does the reordering, and the epilogue constants.  Filter rows past K repeat row K-1:
        //      they only feed output columns that are never stored.
        {
            const uint16_t* __restrict__ wg = (const uint16_t*)a.w;
            // chunks of 1 KiB: 64 (octet, filter) pairs; first those of whole octets
            const int whole = WS ? 0 : (a.C >> 3) * KT / 64, chunks = WS ? 0 : (SPT * CC >> 3) * KT / 64;
            int j = wave;
            for (; j < whole; j += NCW) {
                const int o = (j * 64 + lane) / KT, kl = (j * 64 + lane) % KT;
                const uint16_t* src = wg + ((size_t)min(k0 + kl, a.K - 1) * a.C + o * 8);
                __builtin_amdgcn_global_load_lds((const void*)src, (__attribute__((address_space(3))) void*)(lds_byte*)(ws + j * 1024),
                                                 16, 0, 0);
            }
            for (; j < chunks; j += NCW) {                           // channels past the last one: zeros
                const int o = (j * 64 + lane) / KT, kl = (j * 64 + lane) % KT;
                const uint16_t* src = wg + ((size_t)min(k0 + kl, a.K - 1) * a.C + o * 8);
                u32x4 v = {0u, 0u, 0u, 0u};
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (o * 8 + e < a.C) v[e >> 1] |= (uint32_t)src[e] << ((e & 1) * 16);
                *(u32x4*)(ws + j * 1024 + lane * 16) = v;
            }
            for (int kl = tid; kl < KT; kl += NCW * 64) {
                const ChannelAffine c1 = channel_affine<DT>(a, min(k0 + kl, a.K - 1));
                cas[2 * kl] = c1.mul;
                cas[2 * kl + 1] = c1.add;
            }
            wait_loads_outstanding<0>();
        }
        CVX_TRACE_MARK(1);
        stage_barrier();                                             // filters, constants and stage 0 are in LDS
        CVX_TRACE_MARK(2);
        ChannelAffine ca[TN];
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            ca[tn].mul = cas[2 * ((wn * TN + tn) * 32 + l32)];
            ca[tn].add = cas[2 * ((wn * TN + tn) * 32 + l32) + 1];
        }
        f32x16 acc[TM][TN];
        auto seed = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                for (int tn = 0; tn < TN; ++tn) {
                    const float sd = has_bn ? 0.0f : ca[tn].add;
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[tm][tn][r] = sd;
                }
        };
        seed();

        uint16_t* __restrict__ yg = (uint16_t*)a.y;
        // The wave's patch [TN*32 filters][64 pixel slots] -> device memory, 8 lanes per filter row, one chunk each
        // (16 bytes, 8 under a column stride of 2).  `tp` selects which pair of the wave's pixel sub-tiles it holds.
        typedef typename std::conditional<SW == 1, u32x4, u32x2>::type chunk_t;
        typedef chunk_t chunk_a2 __attribute__((aligned(2)));
        auto flush_patch = [&](int tile, int tp) __attribute__((always_inline)) {
            const int G = Gb + tile * PT + (wm * TM + tp * 2) * 32 + (lane & 7) * 8;
            const bool live = G < Ge;
            const int q = G >> 3;
            const int line = g.by_cpl.div(q), jc = q - line * g.cpl;
            const int n = g.by_lpi.div(line);
            const int HoWo = g.y_line * g.lpi;
            const int first = jc == g.cpl - 1 ? g.tail + g.odd_tail : 8 * jc;
            const size_t obase = ((size_t)n * a.K + k0 + wn * TN * 32) * HoWo + (line - n * g.lpi) * g.y_line + first / SW;
            chunk_t v[TN * 4];
#pragma unroll
            for (int i = 0; i < TN * 4; ++i) {
                const unsigned char* p = ow + (i * 8 + (lane >> 3)) * OPITCH + (lane & 7) * (16 / SW);
                const u32x2 lo = *(const u32x2*)p;
                if constexpr (SW == 1) {
                    const u32x2 hi = *(const u32x2*)(p + 8);
                    v[i] = u32x4{lo[0], lo[1], hi[0], hi[1]};
                } else {
                    v[i] = lo;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            // streaming store: the output is not read again by this kernel, and lines left dirty in
            // L2 would all have to be written back at the end of the kernel.  Only for whole aligned
            // pieces: lines written in parts are put together in L2.
            auto store_rows = [&](auto&& store) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < TN * 4; ++i) {
                    const int row = i * 8 + (lane >> 3);
                    if (live && k0 + wn * TN * 32 + row < a.K) store(v[i], yg + obase + (size_t)row * HoWo);
                }
            };
            if (SW == 1 && g.y_aligned) store_rows([](chunk_t q, uint16_t* dst) __attribute__((always_inline)) { __builtin_nontemporal_store(q, (chunk_t*)dst); });
            else store_rows([](chunk_t q, uint16_t* dst) __attribute__((always_inline)) { *(chunk_a2*)dst = q; });
        };
        // `convert` rounds two results to a packed pair and applies what the epilogue still owes them
        auto finish_tile = [&](int tile, auto&& convert) __attribute__((always_inline)) {
#pragma unroll
            for (int tp = 0; tp < TM / 2; ++tp) {
                int jc = 0;                                          // the patch's first chunk inside its line
                if constexpr (SW == 2) {
                    const int q = (Gb + tile * PT + (wm * TM + tp * 2) * 32) >> 3;
                    jc = q - g.by_cpl.div(q) * g.cpl;
                }
#pragma unroll
                for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4) {
                        const bool odd = SW == 2 && g.odd_tail && jc == g.cpl - 1;
#pragma unroll
                        for (int tn = 0; tn < TN; ++tn) {
                            const auto& t = acc[tp * 2 + t2][tn];
                            unsigned char* o = ow + (tn * 32 + l32) * OPITCH + (t2 * 32 + 8 * q4 + 4 * h) * 2 / SW;
                            if constexpr (SW == 1)
                                *(u32x2*)o = u32x2{convert(t[4 * q4], t[4 * q4 + 1], tn), convert(t[4 * q4 + 2], t[4 * q4 + 3], tn)};
                            else
                                *(uint32_t*)o = convert(odd ? t[4 * q4 + 1] : t[4 * q4], odd ? t[4 * q4 + 3] : t[4 * q4 + 2], tn);
                        }
                        if (SW == 2 && ++jc == g.cpl) jc = 0;
                    }
                flush_patch(tile, tp);
            }
        };
        auto finish_with = [&](int tile, auto&& act_fn) __attribute__((always_inline)) {
            finish_tile(tile, [&](float v0, float v1, int tn) __attribute__((always_inline)) {
                if (has_bn) {
                    v0 = fmaf(v0, ca[tn].mul, ca[tn].add);
                    v1 = fmaf(v1, ca[tn].mul, ca[tn].add);
                }
                return pack2<DT>(act_fn(v0), act_fn(v1));
            });
        };

        int st = 0, tile = 0, slot = 0;
        for (int t = 0; t < T; ++t) {
            const unsigned char* xs = ring + slot * SLOT;
            const unsigned char* wst = WS ? xs + STAGE + (h * KT + wn * TN * 32 + l32) * 16 : wl + (size_t)st * (CC / 8) * KT * 16;
            u32x4 fa[KSTEPS][TM], fb[KSTEPS][TN];
#pragma unroll
            for (int kk = 0; kk < KSTEPS; ++kk) {
#pragma unroll
                for (int tn = 0; tn < TN; ++tn) fb[kk][tn] = *(const u32x4*)(wst + (kk * 2 * KT + tn * 32) * 16);
#pragma unroll
                for (int tm = 0; tm < TM; ++tm) {
                    const u32x2 lo = lds_read_tr16(xs + xa[tm] + kk * 16 * ROWB);
                    const u32x2 hi = lds_read_tr16(xs + xa[tm] + kk * 16 * ROWB + 4 * ROWB);
                    fa[kk][tm] = u32x4{lo[0], lo[1], hi[0], hi[1]};
                }
            }
            if constexpr (WS) {
                const int c8 = a.C & ~7, sh = 16 * (8 - (a.C & 7));
                if (st == SPT - 1 && sh < 128) {                     // the partial octet's channels move down, zeros follow
#pragma unroll
                    for (int kk = 0; kk < KSTEPS; ++kk)
#pragma unroll
                        for (int tn = 0; tn < TN; ++tn) {
                            const u32x4 f = fb[kk][tn];
                            const uint64_t lo = (uint64_t)f[1] << 32 | f[0], hi = (uint64_t)f[3] << 32 | f[2];
                            const uint64_t nlo = sh < 64 ? lo >> sh | hi << (64 - sh) : hi >> (sh - 64), nhi = sh < 64 ? hi >> sh : 0ull;
                            if (st * CC + kk * 16 + 8 * h == c8)
                                fb[kk][tn] = u32x4{(uint32_t)nlo, (uint32_t)(nlo >> 32), (uint32_t)nhi, (uint32_t)(nhi >> 32)};
                        }
                }
            }
#pragma unroll
            for (int kk = 0; kk < KSTEPS; ++kk)
#pragma unroll
                for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                    for (int tn = 0; tn < TN; ++tn) acc[tm][tn] = mfma_32x32x16<DT>(fa[kk][tm], fb[kk][tn], acc[tm][tn]);

            if (++st == SPT) {
                st = 0;
                if (!has_bn && (a.act == ACT_RELU || a.act == ACT_IDENTITY)) {
                    // the bias is already in the accumulators: round, then ReLU on the packed pair, 1 instruction per value
                    const uint32_t floor2 = packed_floor(a.act == ACT_RELU);
                    finish_tile(tile, [&](float v0, float v1, int) __attribute__((always_inline)) { return max_packed(pack2<DT>(v0, v1), floor2); });
                } else if (a.act == ACT_RELU) finish_with(tile, [](float v) { return fmaxf(v, 0.0f); });
                else if (a.act == ACT_IDENTITY) finish_with(tile, [](float v) { return v; });
                else finish_with(tile, [&](float v) { return activate(v, a.act, a.alpha); });
                seed();
                ++tile;
                if (tile <= 6) CVX_TRACE_MARK(2 + tile);
            }
            if (++slot == NS) slot = 0;
            stage_barrier();
        }
        CVX_TRACE_MARK(15);
    }
}

// ------------------------------------------------------------------------------------------------
constexpr int LDS_LIMIT = 160 * 1024;

struct Variant {
    const char* name;                          // on whole images of aligned chunks
    const char* line_name;                     // on other lines
    int WM, WN, TM, TN, CC, NS;
    bool ws;                                   // filters streamed
    void (*kern[2][2])(ConvArgs, Geom);        // [fp16][column stride 2]
};

#define PW_VARIANT(nm, WM, WN, TM, TN, CC, NS, WS)                                              \
    {"pointwise_" nm, "pointwise_lines_" nm, WM, WN, TM, TN, CC, NS, WS,                                                            \
     {{pointwise_kernel<DT_BF16, WM, WN, TM, TN, CC, NS, 1, WS>, pointwise_kernel<DT_BF16, WM, WN, TM, TN, CC, NS, 2, WS>}, \
      {pointwise_kernel<DT_F16, WM, WN, TM, TN, CC, NS, 1, WS>, pointwise_kernel<DT_F16, WM, WN, TM, TN, CC, NS, 2, WS>}}}

// name: pointwise_ or pointwise_lines_<pixels per tile>x<filters per block>_c<channels per stage>_r<ring slots>[_w: filters streamed]
const Variant kVariants[] = {
    PW_VARIANT("256x64_c32_r5", 4, 1, 2, 2, 32, 5, false),
    PW_VARIANT("256x64_c32_r3", 4, 1, 2, 2, 32, 3, false),
    PW_VARIANT("128x128_c32_r6", 2, 2, 2, 2, 32, 6, false),
    PW_VARIANT("128x256_c32_r6", 1, 4, 4, 2, 32, 6, false),
    PW_VARIANT("128x64_c32_r6", 2, 1, 2, 2, 32, 6, false),
    PW_VARIANT("128x32_c32_r6", 2, 1, 2, 1, 32, 6, false),
    PW_VARIANT("128x128_c32_r6_w", 2, 2, 2, 2, 32, 6, true),
    PW_VARIANT("256x64_c32_r6_w", 4, 1, 2, 2, 32, 6, true),
};
constexpr int kNumVariants = sizeof(kVariants) / sizeof(kVariants[0]);

struct Plan {
    const Variant* v;
    Geom g;
    int blocks, lds;
    double us;             // estimated time
};

bool plan_variant(const ConvArgs& a, const Variant& v, int cus, Plan* out)
{
    const int PT = v.WM * v.TM * 32, KT = v.WN * v.TN * 32, NCW = v.WM * v.WN;
    const int SW = a.stride_w;
    Geom g;
    memset(&g, 0, sizeof g);
    g.HW = a.H * a.W;
    const bool rows = a.stride_w != 1 || a.stride_h != 1;              // lines are image rows
    const int slots = rows ? SW * a.Wo : g.HW;                        // of one line
    g.lpi = rows ? a.Ho : 1;
    g.cpl = (slots + 7) / 8;
    g.x_line = rows ? a.stride_h * a.W : 0;
    g.y_line = rows ? a.Wo : g.HW;
    // the last of SW * Wo columns may lie one past the row (odd width): the last chunk then starts a column earlier
    g.odd_tail = rows && SW == 2 && (a.W & 1);
    g.tail = slots - 8 - g.odd_tail;
    if (g.tail < 0) return false;
    g.y_aligned = SW == 1 && slots % 8 == 0;
    const long long total = (long long)a.N * g.lpi * g.cpl * 8;
    if (total >= (1LL << 30)) return false;                           // the flattened pixel index stays in int
    g.total_px = (int)total;
    g.stages_per_tile = (a.C + v.CC - 1) / v.CC;
    g.x_streaming = a.C > a.K ? 1 : 0;
    const long long wbytes = v.ws ? 0 : (long long)g.stages_per_tile * v.CC * KT * 2;
    const long long stage = (long long)v.CC * PT * 2, wstage = v.ws ? (long long)v.CC * KT * 2 : 0;
    long long off = 0;
    g.w_off = (int)off;            off += wbytes;
    g.ca_off = (int)off;           off += (long long)KT * 8;
    g.out_off = (int)off;          off += (long long)NCW * v.TN * 32 * OPITCH;
    off = (off + 1023) & ~1023LL;
    g.ring_off = (int)off;         off += (stage + wstage) * v.NS;
    if (off > LDS_LIMIT) return false;
    g.kblocks = (a.K + KT - 1) / KT;
    // Blocks get equal runs of whole tiles, as short as lets all of them run at once (one per compute unit): a nearly
    // empty last tile would still cost a block the full latency of its stages, while leaving a few compute units idle
    // costs nothing as long as the rest keep device memory busy.
    const long long tiles = (total + PT - 1) / PT;
    const long long per_block = (tiles * g.kblocks + cus - 1) / cus;
    long long blocks = (tiles + per_block - 1) / per_block;
    g.span = (int)(per_block * PT);
    g.by_cpl = div31(g.cpl);
    g.by_lpi = div31(g.lpi);
    g.by_kblocks = div31(g.kblocks);
    // Estimated time in us: the fill and drain (measured 3-4 us), the filters, and per tile the largest of what
    // device memory, the loaders and the multiply waves need (KB per us and cycles as measured on this chip).
    const double nblk = (double)blocks * g.kblocks, resident = nblk < cus ? nblk : cus;
    const double rate = 5500.0 / resident < 64.0 ? 5500.0 / resident : 64.0;        // KB per us and block, device memory
    const double x_kb = (double)g.stages_per_tile * stage / 1024.0, y_kb = (double)PT / SW * (a.K < KT ? a.K : KT) * 2 / 1024.0;
    // Few blocks of the wide streamed tile are chains of load latencies, twice as long where its pixels come in short runs:
    // 2x1712x40x40 K=27 stride (3, 1), 54 stages: 46.4 us, in 128x128 tiles 28.5; with many filter blocks the input comes
    // from L2 (2x1232x32x32 K=1472 stride (3, 1): 19.2, in 128x32 tiles 33.4)
    const bool chain = v.ws && PT == 256 && g.kblocks <= 4 && resident < cus / 2 && (a.stride_h > 1 ? a.W : g.HW) < 64;
    const double t_mem = (x_kb * (0.5 + 0.5 / g.kblocks) + y_kb) / rate, t_l2 = (x_kb / (g.y_aligned ? 64.0 : 45.0) + g.stages_per_tile * wstage / 1024.0 / 20.0) * (chain ? 2.0 : 1.0);
    const double t_mul = g.stages_per_tile * (v.CC / 16 * v.TM * v.TN * 32 / 0.6 + 250.0) / 2000.0 + 0.5 * v.TM * v.TN / 4;
    double tile = t_mem > t_l2 ? t_mem : t_l2;
    if (t_mul > tile) tile = t_mul;
    tile += 0.2 * (t_mem + t_l2 + t_mul - tile);                      // what overlaps incompletely
    out->us = (v.ws ? 4.0 : 3.0) + wbytes / 1024.0 / 50.0 + (double)((long long)(nblk + cus - 1) / cus) * per_block * tile;
    if (g.kblocks > 1) blocks = (blocks + 7) / 8 * 8;                  // whole groups of the 8 XCDs; spare blocks end at once
    out->v = &v;
    out->g = g;
    out->blocks = (int)(blocks * g.kblocks);
    out->lds = (int)off;
    return true;
}

bool choose(const ConvArgs& a, const PlanEnv& env, Plan* out)
{
    if (a.dtype != DT_BF16 && a.dtype != DT_F16) return false;
    if (a.groups != 1 || a.R != 1 || a.S != 1) return false;
    if (a.stride_w > 2 || a.pad_h != 0 || a.pad_w != 0) return false;
    const long long HW = (long long)a.H * a.W;
    if (HW > (1 << 24)) return false;
    if ((long long)a.N * HW * a.C >= (1LL << 31) || (long long)a.N * HW * a.K >= (1LL << 31)) return false;
    if (a.C < 8) return false;
    if (!env.aligned16) return false;
    bool found = false;
    Plan best;
    for (int i = 0; i < kNumVariants; ++i) {
        Plan p;
        if (!plan_variant(a, kVariants[i], env.cus, &p)) continue;
        if (env.pin) {                                               // developer pin: variant name
            if (strcmp(env.pin, kVariants[i].name) == 0 || strcmp(env.pin, kVariants[i].line_name) == 0) {
                *out = p;
                return true;
            }
            continue;
        }
        // four pixel sub-tiles a wave pay on aligned lines and full filter blocks only (8x112x51x51 K=496 stride 2: 12.4 us
        // against 8.6 on 128x128; 25x80x44x44 K=144: 10.6 against 9.4; 64x64x56x56 K=256: 27.6 against 27.4)
        if (kVariants[i].TM == 4 && (!p.g.y_aligned || a.K % (kVariants[i].WN * kVariants[i].TN * 32))) continue;
        if (!found || p.us < best.us) {
            best = p;
            found = true;
        }
    }
    if (found) *out = best;
    return found;
}

}  // namespace pw

#ifdef CVX_PHASE_TRACE
extern "C" int cvx_debug_set_phase_trace_pointwise(unsigned long long* device_buffer)
{
    return (int)hipMemcpyToSymbol(HIP_SYMBOL(g_phase_trace), &device_buffer, sizeof(device_buffer));
}
#endif

bool pointwise_plan(const ConvArgs& a, const PlanEnv& env, LaunchPlan* out)
{
    static_assert(sizeof(pw::Geom) <= sizeof(out->geom), "geometry does not fit the plan");
    pw::Plan p;
    if (!pw::choose(a, env, &p)) return false;
    out->id = KID_POINTWISE;
    out->name = a.stride_h == 1 && a.stride_w == 1 && p.g.y_aligned ? p.v->name : p.v->line_name;
    out->variant = (int)(p.v - pw::kVariants);
    out->grid_x = (unsigned)p.blocks;
    out->grid_y = 1;
    out->block = (unsigned)((p.v->WM * p.v->WN + pw::ND) * 64);
    out->lds = p.lds;
    out->us = p.us;
    memcpy(out->geom, &p.g, sizeof p.g);
    return true;
}

hipError_t pointwise_prepare()
{
    static const hipError_t status = [] {
        for (int i = 0; i < pw::kNumVariants; ++i) {
            const auto& k = pw::kVariants[i].kern;
            for (auto kern : {k[0][0], k[0][1], k[1][0], k[1][1]}) {
                hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, pw::LDS_LIMIT);
                if (e != hipSuccess) return e;
            }
        }
        return hipSuccess;
    }();
    return status;
}

hipError_t pointwise_launch(const ConvArgs& a, const LaunchPlan& p, hipStream_t s)
{
    hipError_t e = pointwise_prepare();
    if (e != hipSuccess) return e;
    const pw::Variant& v = pw::kVariants[p.variant];
    pw::Geom g;
    memcpy(&g, p.geom, sizeof g);
    auto kern = v.kern[a.dtype == DT_F16][a.stride_w == 2];
    hipLaunchKernelGGL(kern, dim3(p.grid_x), dim3(p.block), p.lds, s, a, g);
    return hipGetLastError();
}

}  // namespace cvx
