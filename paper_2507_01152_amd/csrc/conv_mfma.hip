// BF16 MFMA implicit-GEMM convolutions (forward, data gradient, weight
// gradient) with FP32 accumulation for gfx950, plus the element-wise kernels
// of the surrogate network.
//
// Tensors are NHWC bf16 with C a multiple of 8; weights are [Co][kh][kw][Ci]
// (K = kh*kw*Ci contiguous per output channel).  One GEMM kernel template
// serves the three products:
//   forward   C[pixel][co]       = sum_k im2col(x)[pixel][k] * W[co][k]
//   data grad C[in pixel][ci]    = sum_k gather(dy)[in pixel][k] * WT[ci][k]
//                                  (k = (r, s, co); WT = [Ci][kh][kw][Co])
//   weight gr C[co][(r, s, ci)]  = sum_pixels dy[pixel][co] * x(shifted)[pixel][ci]
// A block tile (BM x BN) is built from 4 waves, each owning FM x FN tiles of
// v_mfma_f32_16x16x32_bf16.  The forward / data-gradient operands are
// contiguous along K: they go from global memory straight into a three-stage
// LDS ring by DMA (global_load_lds, 16 bytes a lane, two K steps ahead; no
// staging registers), in unpadded 64-byte rows whose 16-byte chunks are
// XOR-swizzled so the MFMA operand reads are free of bank conflicts.  Where the
// channel count is a multiple of 32 each K step is one tap's 32 channels, and
// the gather addresses are set once per tap.  The weight-gradient operands are
// contiguous along the channel (M / N) axis and are transposed into
// double-buffered LDS (rows padded to 80 bytes) through registers.  The weight
// gradient splits K (pixels) over blocks and sums the partial tiles in a fixed
// order (deterministic).
// A conv may read its input through a nearest-neighbour x2 upsampling
// (decoder layers): the gather maps (h, w) to (h / 2, w / 2).
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <cstring>
#include <type_traits>

#include "surrogate_internal.h"

namespace sg {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // 16-byte staging chunk

constexpr int kThreads = 256;

// conv epilogue activation: 0 none, 1 ReLU, 2 leaky ReLU (slope kLeakySlope)
__device__ __forceinline__ float activate(float y, int act)
{
    if (act == 1) return fmaxf(y, 0.f);
    if (act == 2) return y > 0.f ? y : kLeakySlope * y;
    return y;
}
// the same with the activation known at compile time (epilogue loops instantiated per activation,
// so no per-element branch)
template <int ACT>
__device__ __forceinline__ float activate_c(float y)
{
    if constexpr (ACT == 1) return fmaxf(y, 0.f);
    else if constexpr (ACT == 2) return y > 0.f ? y : kLeakySlope * y;
    else return y;
}
constexpr int kBK = 32;           // K per MFMA step
constexpr int kBKP = kBK + 8;     // padded LDS row (bf16)

__device__ __forceinline__ uint16_t f2bf(float f)
{
    // round to nearest even (finite inputs)
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float bf2f(uint16_t b)
{
    return __uint_as_float((uint32_t)b << 16);
}

typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
typedef float f32x2v __attribute__((ext_vector_type(2)));
// two floats to packed bf16 (lo in bits 0..15) by the hardware conversion, round to nearest even:
// the bits of f2bf for finite inputs (checked on gfx950 over random finite patterns, exact ties,
// denormals and values next to the largest finite), one instruction for the pair
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    const f32x2v v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2v));
}
// bf16(a + b) for the two bf16 halves of each of two packed words
__device__ __forceinline__ uint32_t add_bf16x2(uint32_t a, uint32_t b)
{
    return pack_bf16x2(__uint_as_float(a << 16) + __uint_as_float(b << 16),
                       __uint_as_float(a & 0xFFFF0000u) + __uint_as_float(b & 0xFFFF0000u));
}

enum Mode { kFwd = 0, kDgrad = 1, kWgrad = 2 };

// LDS DMA operand rows are 64 bytes (four 16-byte K chunks) with no padding; K chunk q of row
// r sits in slot q ^ swz(r).  The 16 rows read by one MFMA operand load then put their chunks
// in 16 distinct 16-byte bank groups of 256 bytes (and any 8 consecutive rows in 8 of 128).
__device__ __forceinline__ int swz(int r) { return ((r >> 2) ^ (r >> 1)) & 3; }
// source of the DMA loads of padding and out-of-tile chunks (the DMA writes what it reads):
// 4096 bf16, so that a padding chunk can be advanced by any channel offset below C (C <= 4096)
__device__ __attribute__((aligned(16))) uint16_t g_zero_buf[4096];
// one 16-byte global -> LDS DMA load per lane: lane i of the wave writes dst_wave + 16 i, where
// dst_wave must be the same for the whole wave (it goes through M0).  A function of its own: the
// builtin called straight from a lambda inside a kernel template leaves that kernel without a
// host launch stub, with no diagnostic.
__device__ __forceinline__ void dma16(const uint16_t* src, uint16_t* dst_wave)
{
    __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void*)dst_wave, 16, 0, 0);
}
// s_waitcnt immediate with expcnt and lgkmcnt at their maxima: OR in a vmcnt below 16
constexpr int kWaitVm0 = 0x0F70;
constexpr int kWaitLgkm0 = 0xC07F;   // lgkmcnt 0, vmcnt and expcnt at their maxima

template <int MODE, int BM, int BN, int WM, int WN>
__global__ __launch_bounds__(kThreads) void k_conv_gemm(ConvGeom g0, ConvArgs a)
{
    ConvGeom g = g0;
    if (MODE == kDgrad && g0.par == 4) {   // parity class blockIdx.z of a stride-2 data gradient
        const int par = blockIdx.z, pa = par >> 1, pb = par & 1;
        g.par = par;
        g.Hc = g0.hc4[par];
        g.Wc = g0.wc4[par];
        g.f_hw = g0.f_hw4[par];
        g.f_w = g0.f_w4[par];
        g.M = (g0.Kw / ((int64_t)g0.Ho * g0.Wo)) * g.Hc * g.Wc;
        g.K = (pa + 1) * (pb + 1) * g0.Co;
        if ((int64_t)blockIdx.x * BM >= g.M) return;   // this class has fewer row tiles
    }
    constexpr int TM = BM / WM, TN = BN / WN;
    constexpr int FM = TM / 16, FN = TN / 16;
    static_assert(WM * WN == 4, "four waves");
    static_assert(FM >= 1 && FN >= 1, "tile");
    // staged per K step: K-contiguous operands in (row, 8 k) 16-byte chunks
    // (one per register); the weight gradient's in tasks of 8 rows x 4 k, four
    // 16-byte (8 rows, k) chunks per task, transposed in registers into one
    // 8-byte (row, 4 k) LDS store per row
    constexpr int CA = (MODE == kWgrad) ? (BM / 8) * (kBK / 4) : BM * (kBK / 8);
    constexpr int CB = (MODE == kWgrad) ? (BN / 8) * (kBK / 4) : BN * (kBK / 8);
    constexpr int RPC = (MODE == kWgrad) ? 4 : 1;   // registers per chunk or task
    constexpr int PA = RPC * ((CA + kThreads - 1) / kThreads);
    constexpr int PB = RPC * ((CB + kThreads - 1) / kThreads);
    constexpr int AM8 = BM / 8, BN8 = BN / 8;   // weight-gradient row groups

    // operand tiles: the K-contiguous products fill a three-stage ring of unpadded 64-byte rows
    // straight from global memory (LDS DMA); the weight gradient double-buffers padded rows
    // through registers.  The forward epilogue reuses the space for its output tile.
    constexpr bool DMA = MODE != kWgrad;
    constexpr int NS = DMA ? 3 : 2, RL = DMA ? kBK : kBKP;   // stages, LDS row length
    constexpr int SMEM_OPS = NS * (BM + BN) * RL, SMEM_OUT = (MODE == kFwd) ? BM * (BN + 8) : 0;
    __shared__ __attribute__((aligned(16))) uint16_t smem[SMEM_OPS > SMEM_OUT ? SMEM_OPS : SMEM_OUT];
    uint16_t (*sA)[BM * RL] = reinterpret_cast<uint16_t (*)[BM * RL]>(smem);
    uint16_t (*sB)[BN * RL] = reinterpret_cast<uint16_t (*)[BN * RL]>(smem + NS * BM * RL);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    const int m_base = (int)blockIdx.x * BM;    // M < 2^31
    const int n_base = blockIdx.y * BN;
    const uint16_t* __restrict__ A = a.a;
    const uint16_t* __restrict__ B = a.b;
    const u32x4 zero = {0u, 0u, 0u, 0u};

    // K range of this block (split-K for the weight gradient)
    int64_t k_begin = 0, k_end = (MODE == kWgrad) ? g.Kw : g.K;
    if constexpr (MODE == kWgrad) {
        k_begin = (int64_t)blockIdx.z * a.k_chunk;
        k_end = min(k_end, k_begin + a.k_chunk);
    }
    const int nk = (int)((k_end - k_begin + kBK - 1) / kBK);
    const int Hin = g.up ? 2 * g.H : g.H, Win = g.up ? 2 * g.W : g.W;

    // ---- per-thread chunk bookkeeping, fixed over the K loop ----
    // K-contiguous modes: chunk c = tid + i * 256 -> LDS row c / 4, 16-byte slot c % 4, which holds
    // K chunk k8 = slot ^ swz(row); swz depends on row bits 1..3 only, so k8 is fixed per thread
    const int k8 = DMA ? (tid & 3) ^ swz(tid >> 2) : tid & 3;
    int a_hb[PA], a_wb[PA];       // forward: ho*s - pad, wo*s - pad; data grad: h + pad, w + pad
    int64_t a_base[PA];           // element offset of the row's image (or -1: row outside M)
    // weight gradient: fixed channel group of A (dy) and of B (x)
    const int wg_m0 = m_base + (tid % AM8) * 8;
    const int wg_n0 = n_base + (tid % BN8) * 8;
    int wg_r = 0, wg_s = 0, wg_ci0 = 0;
    if constexpr (MODE == kWgrad) {
        if (wg_n0 < g.N) {
            const int t = (int)fdiv((uint32_t)wg_n0, g.f_c);
            wg_ci0 = wg_n0 - t * g.C;
            wg_r = (int)fdiv((uint32_t)t, g.f_kw);
            wg_s = t - wg_r * g.kw;
        }
    } else {
#pragma unroll
        for (int i = 0; i < PA; ++i) {
            const int row = (tid >> 2) + i * (kThreads / 4);
            const int m = m_base + row;
            a_base[i] = -1;
            a_hb[i] = a_wb[i] = 0;
            if (row < BM && m < g.M) {
                if constexpr (MODE == kFwd) {
                    const int n = (int)fdiv((uint32_t)m, g.f_howo);
                    const int rem = m - n * g.Ho * g.Wo;
                    const int ho = (int)fdiv((uint32_t)rem, g.f_wo);
                    const int wo = rem - ho * g.Wo;
                    a_hb[i] = ho * g.stride - g.pad;
                    a_wb[i] = wo * g.stride - g.pad;
                    a_base[i] = (int64_t)n * g.H * g.W * g.C;
                } else {
                    // pixel (h, w) of image n; a parity class counts only its own pixels; an upsampled input's
                    // rows are quads, the four fine pixels of one stored pixel
                    const bool pc = g.par >= 0;
                    const int q = g.up ? m >> 2 : m;
                    const int n = (int)fdiv((uint32_t)q, g.f_hw);
                    const int rem = q - n * (pc ? g.Hc * g.Wc : g.H * g.W);
                    const int qh = (int)fdiv((uint32_t)rem, g.f_w);
                    const int qw = rem - qh * (pc ? g.Wc : g.W);
                    const int h = pc ? 2 * qh + (g.par >> 1) : (g.up ? 2 * qh + ((m >> 1) & 1) : qh);
                    const int w = pc ? 2 * qw + (g.par & 1) : (g.up ? 2 * qw + (m & 1) : qw);
                    a_hb[i] = h + g.pad;
                    a_wb[i] = w + g.pad;
                    a_base[i] = (int64_t)n * g.Ho * g.Wo * g.Co;
                }
            }
        }
    }

    u32x4 ra[PA], rb[PB];

    auto load_tiles = [&](int64_t k0) __attribute__((always_inline)) {
        if constexpr (MODE == kWgrad) {
#pragma unroll
            for (int i = 0; i < PA; ++i) {
                const int c = tid + (i / 4) * kThreads;   // task: rows wg_m0.., k = 4 (c / AM8) + i % 4
                const int64_t k = k0 + 4 * (c / AM8) + (i & 3);
                ra[i] = (c < CA && wg_m0 < g.M && k < k_end)
                            ? *reinterpret_cast<const u32x4*>(A + k * g.Co + wg_m0)
                            : zero;
            }
#pragma unroll
            for (int i = 0; i < PB; ++i) {
                const int c = tid + (i / 4) * kThreads;
                const int64_t k = k0 + 4 * (c / BN8) + (i & 3);
                rb[i] = zero;
                if (c < CB && wg_n0 < g.N && k < k_end) {
                    const int p = (int)k;
                    const int n = (int)fdiv((uint32_t)p, g.f_howo);
                    const int rem = p - n * g.Ho * g.Wo;
                    const int ho = (int)fdiv((uint32_t)rem, g.f_wo);
                    const int wo = rem - ho * g.Wo;
                    int hi = ho * g.stride - g.pad + wg_r, wi = wo * g.stride - g.pad + wg_s;
                    if (hi >= 0 && wi >= 0 && hi < Hin && wi < Win) {
                        if (g.up) {
                            hi >>= 1;
                            wi >>= 1;
                        }
                        rb[i] = *reinterpret_cast<const u32x4*>(B + (((int64_t)n * g.H + hi) * g.W + wi) * g.C + wg_ci0);
                    }
                }
            }
            return;
        }
        // K-contiguous: one tap / channel split per K step (k8 fixed per thread)
        const int k = (int)k0 + k8 * 8;
        const bool kin = k < g.K;
        int r = 0, s = 0, c0 = 0, kf = k;   // kf: the column of B (all taps)
        if (kin) {
            const FastDiv fc = (MODE == kFwd) ? g.f_c : g.f_co;
            const int cc = (MODE == kFwd) ? g.C : g.Co;
            const int t = (int)fdiv((uint32_t)k, fc);
            c0 = k - t * cc;
            if (MODE == kDgrad && g.par >= 0) {
                // class taps: rows r in {1} (even h) or {0, 2} (odd h), columns s likewise, row-major
                const int pa = g.par >> 1, pb = g.par & 1;
                const int tr = pb ? t >> 1 : t, ts = pb ? t & 1 : 0;
                r = pa ? 2 * tr : 1;
                s = pb ? 2 * ts : 1;
                kf = (r * 3 + s) * cc + c0;
            } else {
                r = (int)fdiv((uint32_t)t, g.f_kw);
                s = t - r * g.kw;
            }
        }
#pragma unroll
        for (int i = 0; i < PA; ++i) {
            ra[i] = zero;
            if (!kin || a_base[i] < 0) continue;
            if constexpr (MODE == kFwd) {
                int hi = a_hb[i] + r, wi = a_wb[i] + s;
                if (hi < 0 || wi < 0 || hi >= Hin || wi >= Win) continue;
                if (g.up) {
                    hi >>= 1;
                    wi >>= 1;
                }
                ra[i] = *reinterpret_cast<const u32x4*>(A + a_base[i] + ((int64_t)hi * g.W + wi) * g.C + c0);
            } else {
                const int hh = a_hb[i] - r, ww = a_wb[i] - s;
                if (hh < 0 || ww < 0) continue;
                const int ho = (int)fdiv((uint32_t)hh, g.f_stride), wo = (int)fdiv((uint32_t)ww, g.f_stride);
                if (ho * g.stride != hh || wo * g.stride != ww || ho >= g.Ho || wo >= g.Wo) continue;
                ra[i] = *reinterpret_cast<const u32x4*>(A + a_base[i] + ((int64_t)ho * g.Wo + wo) * g.Co + c0);
            }
        }
#pragma unroll
        for (int i = 0; i < PB; ++i) {
            const int col = n_base + (tid >> 2) + i * (kThreads / 4);
            rb[i] = (kin && (tid >> 2) + i * (kThreads / 4) < BN && col < g.N)
                        ? *reinterpret_cast<const u32x4*>(B + (int64_t)col * g.kb + kf)
                        : zero;
        }
    };
    // one stage of the LDS-DMA ring: each lane fetches its 16-byte chunk (a zero chunk where the
    // operand is padding or past the tile) into slot c of the stage; the 64 lanes of a wave fill
    // 64 consecutive slots, so the LDS address passed is the wave's first slot, a scalar.
    // The zero buffer's address is taken once (readfirstlane returns int: each half goes through
    // uint32_t, or the low half sign-extends).
    const uint64_t zp = reinterpret_cast<uint64_t>(g_zero_buf);
    const uint32_t zhi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(zp >> 32));
    const uint32_t zlo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)zp);
    const uint16_t* zsrc = reinterpret_cast<const uint16_t*>(((uint64_t)zhi << 32) | zlo);
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    const FastDiv fcc = (MODE == kFwd) ? g.f_c : g.f_co;
    const int cc = (MODE == kFwd) ? g.C : g.Co;   // channels of one tap along K
    // tap (r, s) of tap index t, and the column of B where the tap's channels start
    auto tap_of = [&](int t, int& r, int& s, int& kfb) __attribute__((always_inline)) {
        if (MODE == kDgrad && g.par >= 0) {
            // class taps: rows r in {1} (even h) or {0, 2} (odd h), columns s likewise, row-major
            const int pa = g.par >> 1, pb = g.par & 1;
            const int tr = pb ? t >> 1 : t, ts = pb ? t & 1 : 0;
            r = pa ? 2 * tr : 1;
            s = pb ? 2 * ts : 1;
            kfb = (r * 3 + s) * cc;
        } else {
            r = (int)fdiv((uint32_t)t, g.f_kw);
            s = t - r * g.kw;
            kfb = t * cc;
        }
    };
    // element offset of tap (r, s), channel c0, inside row i's image; false where it is padding
    auto a_tap = [&](int i, int r, int s, int c0, int& off) __attribute__((always_inline)) -> bool {
        if constexpr (MODE == kFwd) {
            const int hi = a_hb[i] + r, wi = a_wb[i] + s;
            off = ((hi >> g.up) * g.W + (wi >> g.up)) * g.C + c0;
            return a_base[i] >= 0 && (unsigned)hi < (unsigned)Hin && (unsigned)wi < (unsigned)Win;
        } else {
            const int hh = a_hb[i] - r, ww = a_wb[i] - s;
            const int ho = (int)fdiv((uint32_t)hh, g.f_stride), wo = (int)fdiv((uint32_t)ww, g.f_stride);
            off = (ho * g.Wo + wo) * g.Co + c0;
            return a_base[i] >= 0 && hh >= 0 && ww >= 0 && ho * g.stride == hh && wo * g.stride == ww &&
                   ho < g.Ho && wo < g.Wo;
        }
    };
    // general K steps (C not a multiple of 32: a step's chunks may fall in different taps, or past K)
    auto issue_stage = [&](int k0, int st) __attribute__((always_inline)) {
        const int k = k0 + k8 * 8;
        const bool kin = k < g.K;
        int r = 0, s = 0, c0 = 0, kf = k;
        if (kin) {
            const int t = (int)fdiv((uint32_t)k, fcc);
            c0 = k - t * cc;
            int kfb;
            tap_of(t, r, s, kfb);
            kf = kfb + c0;
        }
#pragma unroll
        for (int i = 0; i < PA; ++i) {
            if ((i + 1) * kThreads > CA && wv * 64 + i * kThreads >= CA) continue;   // CA is a multiple of 64
            int off;
            const bool ok = a_tap(i, r, s, c0, off) && kin;
            dma16(ok ? A + a_base[i] + off : zsrc, &sA[st][(wv * 64 + i * kThreads) * 8]);
        }
#pragma unroll
        for (int i = 0; i < PB; ++i) {
            if ((i + 1) * kThreads > CB && wv * 64 + i * kThreads >= CB) continue;
            const int col = n_base + ((tid + i * kThreads) >> 2);
            dma16((kin && col < g.N) ? B + (int64_t)col * g.kb + kf : zsrc, &sB[st][(wv * 64 + i * kThreads) * 8]);
        }
    };
    // tap steps (C a multiple of 32: each K step is 32 channels of one tap, and K = nk * 32): the
    // chunk pointers are set once per tap (pointing at channel 0 plus this lane's 8 k, or into the
    // zero buffer) and a step adds its channel offset
    const uint16_t* tpa[PA];
    const uint16_t* tpb[PB];
    int cur_t = 0, tap_k = 0;   // the current tap and its first K
    auto issue_tap = [&](int k0, int st) __attribute__((always_inline)) {
        const int c0 = k0 - tap_k;   // K steps come in order: the next tap starts after cc channels
        if (c0 == cc || k0 == 0) {
            const int t = k0 == 0 ? 0 : cur_t + 1;
            cur_t = t;
            tap_k = k0;
            int r, s, kfb;
            tap_of(t, r, s, kfb);
#pragma unroll
            for (int i = 0; i < PA; ++i) {
                if ((i + 1) * kThreads > CA && wv * 64 + i * kThreads >= CA) continue;
                int off;
                const bool ok = a_tap(i, r, s, 0, off);
                tpa[i] = (ok ? A + a_base[i] + off : zsrc) + k8 * 8;
            }
#pragma unroll
            for (int i = 0; i < PB; ++i) {
                if ((i + 1) * kThreads > CB && wv * 64 + i * kThreads >= CB) continue;
                const int col = n_base + ((tid + i * kThreads) >> 2);
                tpb[i] = (col < g.N ? B + (int64_t)col * g.kb + kfb : zsrc) + k8 * 8;
            }
        }
#pragma unroll
        for (int i = 0; i < PA; ++i) {
            if ((i + 1) * kThreads > CA && wv * 64 + i * kThreads >= CA) continue;
            dma16(tpa[i] + (k0 - tap_k), &sA[st][(wv * 64 + i * kThreads) * 8]);
        }
#pragma unroll
        for (int i = 0; i < PB; ++i) {
            if ((i + 1) * kThreads > CB && wv * 64 + i * kThreads >= CB) continue;
            dma16(tpb[i] + (k0 - tap_k), &sB[st][(wv * 64 + i * kThreads) * 8]);
        }
    };
    // four (8 rows, k) chunks of consecutive k -> row j's 4 k as one 8-byte value
    auto transpose_store = [&](uint16_t* dst, const u32x4* r, int row0, int kk) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int w = j >> 1;
            const uint32_t lo = (j & 1) ? ((r[0][w] >> 16) | (r[1][w] & 0xFFFF0000u))
                                        : ((r[0][w] & 0xFFFFu) | (r[1][w] << 16));
            const uint32_t hi = (j & 1) ? ((r[2][w] >> 16) | (r[3][w] & 0xFFFF0000u))
                                        : ((r[2][w] & 0xFFFFu) | (r[3][w] << 16));
            *reinterpret_cast<uint2*>(&dst[(row0 + j) * kBKP + kk]) = make_uint2(lo, hi);
        }
    };
    auto store_tiles = [&](int buf) __attribute__((always_inline)) {
        if constexpr (MODE == kWgrad) {
#pragma unroll
            for (int i = 0; i < PA / 4; ++i) {
                const int c = tid + i * kThreads;
                if (c < CA) transpose_store(sA[buf], ra + 4 * i, (c % AM8) * 8, 4 * (c / AM8));
            }
#pragma unroll
            for (int i = 0; i < PB / 4; ++i) {
                const int c = tid + i * kThreads;
                if (c < CB) transpose_store(sB[buf], rb + 4 * i, (c % BN8) * 8, 4 * (c / BN8));
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < PA; ++i) {
            const int c = tid + i * kThreads;
            if (c >= CA) continue;
            *reinterpret_cast<u32x4*>(&sA[buf][(c >> 2) * kBKP + k8 * 8]) = ra[i];
        }
#pragma unroll
        for (int i = 0; i < PB; ++i) {
            const int c = tid + i * kThreads;
            if (c >= CB) continue;
            *reinterpret_cast<u32x4*>(&sB[buf][(c >> 2) * kBKP + k8 * 8]) = rb[i];
        }
    };

    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // the forward epilogue's bias, read once here (in the epilogue a load after a possibly
    // aliasing store would be repeated, each waiting for memory)
    float bias_r[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) {
        const int col = n_base + wn * TN + j * 16 + (lane & 15);
        bias_r[j] = (MODE == kFwd && a.bias && col < g.N) ? a.bias[col] : 0.f;
    }

    const int frow = lane & 15, fk = (lane >> 4) * 8;
    if constexpr (DMA) {
        // a wave waits for its own DMA of stage kt (vmcnt counts in issue order: at most the next
        // stage's loads may remain), then the barrier makes every wave's chunks visible and
        // retires the reads of the stage the next issue overwrites.  LW is the fewest DMA loads
        // any wave issues per stage (wave 3's, whose first chunk is 192); a wave with more waits
        // for part of the next stage too.  The barrier is the bare s_barrier: __syncthreads()
        // would add a wait for every outstanding load (vmcnt(0)) and drain the ring; the empty
        // asm statements keep the compiler from moving LDS accesses across it.
        constexpr int LW = ((CA - 192 + kThreads - 1) / kThreads) + (CB > 192 ? (CB - 192 + kThreads - 1) / kThreads : 0);
        static_assert(LW >= 1 && LW < 16, "per-wave DMA loads per stage");
        const int rd = frow * kBK + (((lane >> 4) ^ swz(frow)) * 8);
        // (one instantiation of the loop per kind of step, and no test that the tile's size decides: with those
        // branches inside, 128 -> 64 channels upsampled on 131072 pixels took 30.7 us forward and 38 us backward,
        // now 29.2 and 34.5)
        auto k_loop = [&](auto issue) __attribute__((always_inline)) {
        if (nk > 0) issue(0, 0);
        if (nk > 1) issue(kBK, 1);
        int st = 0, st2 = 2;   // stages of step kt and of step kt + 2
        for (int kt = 0; kt < nk; ++kt) {
            if (kt + 1 < nk) __builtin_amdgcn_s_waitcnt(kWaitVm0 | LW);
            else __builtin_amdgcn_s_waitcnt(kWaitVm0);
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (kt + 2 < nk) issue((kt + 2) * kBK, st2);
            bf16x8 fa[FM], fb[FN];
#pragma unroll
            for (int i = 0; i < FM; ++i)
                fa[i] = *reinterpret_cast<const bf16x8*>(&sA[st][(wm * TM + i * 16) * kBK + rd]);
#pragma unroll
            for (int j = 0; j < FN; ++j)
                fb[j] = *reinterpret_cast<const bf16x8*>(&sB[st][(wn * TN + j * 16) * kBK + rd]);
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
            st = st == 2 ? 0 : st + 1;
            st2 = st2 == 2 ? 0 : st2 + 1;
        }
        };
        if (cc % kBK == 0) k_loop(issue_tap);
        else k_loop(issue_stage);
    } else {
    if (nk > 0) {
        load_tiles(k_begin);
        store_tiles(0);
    }
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        const int buf = kt & 1;
        if (kt + 1 < nk) load_tiles(k_begin + (int64_t)(kt + 1) * kBK);
        bf16x8 fa[FM], fb[FN];
#pragma unroll
        for (int i = 0; i < FM; ++i)
            fa[i] = *reinterpret_cast<const bf16x8*>(&sA[buf][(wm * TM + i * 16 + frow) * RL + fk]);
#pragma unroll
        for (int j = 0; j < FN; ++j)
            fb[j] = *reinterpret_cast<const bf16x8*>(&sB[buf][(wn * TN + j * 16 + frow) * RL + fk]);
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
        if (kt + 1 < nk) store_tiles(buf ^ 1);
        __syncthreads();
    }
    }

    // epilogue: lane holds rows 4*(lane/16) + r, column lane % 16 of each tile
    if constexpr (MODE == kFwd) {
        // the bf16 outputs go through an LDS tile [BM][BN + 8] to 16-byte stores; the skip tensor's
        // chunks are all loaded before the first store (a load issued after a store waits for it:
        // one memory round trip per element otherwise)
        constexpr int TP = BN + 8;
        uint16_t* sT = smem;
        __syncthreads();   // every wave is done with the operand tiles
        // (one instantiation per activation; a lane's rows r, r + 1 share one bf16 conversion)
        auto write_tile = [&](auto act_c) __attribute__((always_inline)) {
            constexpr int ACT = decltype(act_c)::value;
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    const int cl = wn * TN + j * 16 + (lane & 15), col = n_base + cl;
#pragma unroll
                    for (int r = 0; r < 4; r += 2) {
                        const int rl = wm * TM + i * 16 + (lane >> 4) * 4 + r;
                        const float y0 = activate_c<ACT>(acc[i][j][r] + bias_r[j]);
                        const float y1 = activate_c<ACT>(acc[i][j][r + 1] + bias_r[j]);
                        const uint32_t pk = pack_bf16x2(y0, y1);
                        sT[rl * TP + cl] = (uint16_t)pk;
                        sT[(rl + 1) * TP + cl] = (uint16_t)(pk >> 16);
                        if (a.out_f32) {
                            const int64_t row = (int64_t)m_base + rl;
                            if (row < g.M && col < g.N) a.out_f32[row * g.Co + col] = y0;
                            if (row + 1 < g.M && col < g.N) a.out_f32[(row + 1) * g.Co + col] = y1;
                        }
                    }
                }
        };
        if (a.relu == 1) write_tile(std::integral_constant<int, 1>{});
        else if (a.relu == 2) write_tile(std::integral_constant<int, 2>{});
        else write_tile(std::integral_constant<int, 0>{});
        __syncthreads();
        constexpr int CH = BM * BN / 8, CPT = (CH + kThreads - 1) / kThreads;   // 16-byte chunks
        const int ld2 = a.ld_out2 ? a.ld_out2 : g.Co;
        // chunk u of this thread: tile row rl, columns 8 c8.. (Co is a multiple of 8, so a chunk is
        // wholly inside or past column N); separate loops with and without the skip tensor, so the
        // stores of the plain one wait for no load
        if (a.skip && a.out2_bf16) {
            u32x4 kv[CPT];
#pragma unroll
            for (int u = 0; u < CPT; ++u) {
                const int c = tid + u * kThreads, rl = c / (BN / 8), c8 = c % (BN / 8);
                const int64_t row = (int64_t)m_base + rl;
                const int col = n_base + c8 * 8;
                kv[u] = (c < CH && row < g.M && col < g.N)
                            ? *reinterpret_cast<const u32x4*>(a.skip + row * g.Co + col)
                            : zero;
            }
#pragma unroll
            for (int u = 0; u < CPT; ++u) {
                const int c = tid + u * kThreads, rl = c / (BN / 8), c8 = c % (BN / 8);
                const int64_t row = (int64_t)m_base + rl;
                const int col = n_base + c8 * 8;
                if (c >= CH || row >= g.M || col >= g.N) continue;
                const u32x4 v = *reinterpret_cast<const u32x4*>(&sT[rl * TP + c8 * 8]);
                if (a.out_bf16) *reinterpret_cast<u32x4*>(a.out_bf16 + row * g.Co + col) = v;
                u32x4 o;
#pragma unroll
                for (int q = 0; q < 4; ++q) o[q] = add_bf16x2(v[q], kv[u][q]);
                *reinterpret_cast<u32x4*>(a.out2_bf16 + row * ld2 + col) = o;
            }
        } else if (a.out_bf16) {
#pragma unroll
            for (int u = 0; u < CPT; ++u) {
                const int c = tid + u * kThreads, rl = c / (BN / 8), c8 = c % (BN / 8);
                const int64_t row = (int64_t)m_base + rl;
                const int col = n_base + c8 * 8;
                if (c >= CH || row >= g.M || col >= g.N) continue;
                *reinterpret_cast<u32x4*>(a.out_bf16 + row * g.Co + col) =
                    *reinterpret_cast<const u32x4*>(&sT[rl * TP + c8 * 8]);
            }
        }
        return;
    }
    // data and weight gradients: FP32 straight from the accumulators.  Output pixel of row r of row
    // tile i (a parity class's rows are a quarter of the pixels), -1 past the last row:
    auto pixel = [&](int i, int r) __attribute__((always_inline)) -> int64_t {
        const int64_t row = (int64_t)m_base + wm * TM + i * 16 + (lane >> 4) * 4 + r;
        if (row >= g.M) return -1;
        if constexpr (MODE == kDgrad) {
            if (g.par >= 0) {
                const int n = (int)fdiv((uint32_t)row, g.f_hw);
                const int rem = (int)row - n * g.Hc * g.Wc;
                const int qh = (int)fdiv((uint32_t)rem, g.f_w);
                const int qw = rem - qh * g.Wc;
                return ((int64_t)n * g.H + 2 * qh + (g.par >> 1)) * g.W + 2 * qw + (g.par & 1);
            }
        }
        return row;
    };
    if (MODE == kDgrad && g.up) {
        // a lane's four rows are one stored pixel's quad: summed here, so the fine gradient (67 MB for 131072
        // pixels of 128 channels) never leaves the registers; written out and summed by a kernel of its own, the
        // layer of 32768 stored pixels took 41 + 16 us, with this epilogue 38
        float pre[FM][FN];
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const int64_t row = (int64_t)m_base + wm * TM + i * 16 + (lane >> 4) * 4;   // M is a multiple of 4
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const int col = n_base + wn * TN + j * 16 + (lane & 15);
                pre[i][j] = (a.add && col < g.N && row < g.M) ? a.add[(row >> 2) * g.C + col] : 0.f;
            }
        }
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const int64_t row = (int64_t)m_base + wm * TM + i * 16 + (lane >> 4) * 4;
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const int col = n_base + wn * TN + j * 16 + (lane & 15);
                const float v = (acc[i][j][0] + acc[i][j][1]) + (acc[i][j][2] + acc[i][j][3]);
                if (col < g.N && row < g.M) a.out_f32[(row >> 2) * g.C + col] = a.add ? pre[i][j] + v : v;
            }
        }
        return;
    }
    if (MODE == kDgrad && a.add) {
        // per row tile, the old values are all loaded before the tile's first store (a load issued
        // after a store waits for it)
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            int64_t px[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) px[r] = pixel(i, r);
            float pre[FN][4];
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const int col = n_base + wn * TN + j * 16 + (lane & 15);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    pre[j][r] = (col < g.N && px[r] >= 0) ? a.add[px[r] * g.C + col] : 0.f;
            }
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const int col = n_base + wn * TN + j * 16 + (lane & 15);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (col < g.N && px[r] >= 0) a.out_f32[px[r] * g.C + col] = pre[j][r] + acc[i][j][r];
            }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t px = pixel(i, r);
            if (px < 0) continue;
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const int col = n_base + wn * TN + j * 16 + (lane & 15);
                if (col >= g.N) continue;
                if constexpr (MODE == kDgrad)
                    a.out_f32[px * g.C + col] = acc[i][j][r];
                else
                    a.out_f32[(int64_t)blockIdx.z * g.M * g.N + px * g.N + col] = acc[i][j][r];
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Direct 3x3 convolution (stride 1, pad 1) for few channels.  A block of TH / 2
// waves computes a TH x 32 pixel output tile of one image for all CO output
// channels.  The
// input tile with its one-pixel halo ((TH + 2) x 34 pixels, zero outside the image;
// with upsampling, fine pixel (h, w) reads stored pixel (h / 2, w / 2)) and
// all weights are staged in LDS once (by DMA, every chunk in flight at once),
// and the MFMA operands are read from there, so each input pixel leaves global
// memory once per tile instead of once per tap.  LDS pixel and weight rows are odd multiples of 16 bytes, so
// neighbouring rows start in different bank groups (the bank conflicts left take
// 7-25 % of the kernels' time by the counters).  The output tile is staged through LDS for 16-byte stores; the skip sum and a 1x1 head
// with one output can be fused.
// 16 x 32 tiles (eight waves): against 8 x 32 ones, the weights staged per
// block serve twice the pixels and the halo adds 1/8 instead of 1/4 of the
// input rows (the 1024-frame forward's tiled layers took 3.3 instead of
// 3.6 ms; 32-row tiles were slower again)
constexpr int kTileH = 16, kTileW = 32;

template <int C, int CO, bool UP, bool DIL = false, bool ACC = false, int TH = kTileH>
__global__ __launch_bounds__(32 * TH) void k_conv3x3_tile(ConvGeom g, ConvArgs a)
{
    // DIL: the input is dy of a stride-2 conv dilated by zeros: virtual pixel (h, w) is stored pixel
    // (h / 2, w / 2) when both are even, else 0 (the data gradient of that conv as a stride-1 conv)
    // UP: the input is read upsampled x2; the tile stages the stored pixels it
    // covers (fine halo pixel (hy, wx) of the (TH + 2) x 34 window is stored pixel
    // ((hy + 1) / 2, (wx + 1) / 2) of a (TH / 2 + 2) x 18 window, tile origins being even)
    constexpr int NT = 32 * TH;   // threads: TH / 2 waves of two output rows each
    constexpr int HP = UP ? TH / 2 + 2 : TH + 2, WP = UP ? kTileW / 2 + 2 : kTileW + 2;
    constexpr int C8 = C / 8;
    constexpr int PS = (C8 % 2 == 0) ? C + 8 : C;   // LDS pixel stride (bf16)
    constexpr int K8 = 9 * C8;                       // 8-wide K groups
    constexpr int NKS = (K8 + 3) / 4;                // MFMA K steps of 32
    constexpr int KP = NKS * 32 + 8;                 // LDS weight row (bf16), zero beyond K
    constexpr int FN = CO / 16;
    constexpr int CO8 = CO / 8;
    // staged by LDS DMA in 16-byte slots, whole waves at a time: the regions are rounded up to
    // 64 slots (512 bf16), the slots past the data (and the pad slot of each pixel and weight
    // row) filled from the zero buffer
    constexpr int SPP = PS / 8, KPS = KP / 8;        // slots per staged pixel, per weight row
    constexpr int NXS = HP * WP * SPP, NWS = CO * KPS;
    constexpr int XS = (NXS + 63) / 64 * 512, OS = TH * kTileW * CO;
    __shared__ __attribute__((aligned(16))) uint16_t sX[XS > OS ? XS : OS];
    __shared__ __attribute__((aligned(16))) uint16_t sW[(NWS + 63) / 64 * 512];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lr = lane & 15, lk = lane >> 4;
    const int tiles_x = (g.Wo + kTileW - 1) / kTileW, tiles_y = (g.Ho + TH - 1) / TH;
    // neighbouring tiles on the same XCD (blocks are dealt round-robin over 8)
    int64_t b = blockIdx.x;
    const int64_t nb = gridDim.x;
    if ((nb & 7) == 0) b = (b & 7) * (nb >> 3) + (b >> 3);
    const int64_t per_img = (int64_t)tiles_x * tiles_y;
    const int64_t n = b / per_img;
    const int t_in = (int)(b - n * per_img);
    const int ty = t_in / tiles_x, tx = t_in - ty * tiles_x;
    const int ho0 = ty * TH, wo0 = tx * kTileW;
    const int Hin = g.up ? 2 * g.H : g.H, Win = g.up ? 2 * g.W : g.W;
    const u32x4 zero = {0u, 0u, 0u, 0u};
    // the epilogue's bias, read here, where its latency overlaps the staging (in the epilogue a
    // load after a possibly aliasing store would be repeated, each waiting for memory)
    float bias_r[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) bias_r[j] = a.bias ? a.bias[16 * j + lr] : 0.f;

    // staging: every slot of the halo tile and of the weights is one DMA load, all in flight
    // together (no staging registers); halo slot j is pixel j / SPP, channel group j % SPP (the
    // pad group where that is C8), weight slot j is row j / KPS, K group j % KPS
    const uint64_t zp = reinterpret_cast<uint64_t>(g_zero_buf);
    const uint32_t zhi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(zp >> 32));
    const uint32_t zlo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)zp);
    const uint16_t* zsrc = reinterpret_cast<const uint16_t*>(((uint64_t)zhi << 32) | zlo);
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    // (each source is one select between the operand and the zero buffer, computed without early
    // returns: with divergent returns the compiler reused the zero pointer's register on the
    // padding lanes' path and those lanes loaded from a garbage address)
    auto x_src = [&](int j) __attribute__((always_inline)) -> const uint16_t* {
        const int pix = j / SPP, c8 = j - pix * SPP;
        const int hy = pix / WP, wx = pix - hy * WP;
        bool ok = j < NXS && c8 < C8;
        int hi, wi;
        if constexpr (UP) {   // stored pixels (ho0 / 2 - 1 + hy, wo0 / 2 - 1 + wx), zero outside
            hi = ho0 / 2 - 1 + hy;
            wi = wo0 / 2 - 1 + wx;
            ok = ok && (unsigned)hi < (unsigned)g.H && (unsigned)wi < (unsigned)g.W;
        } else if constexpr (DIL) {
            const int h2 = ho0 - 1 + hy, w2 = wo0 - 1 + wx;
            ok = ok && h2 >= 0 && w2 >= 0 && !(h2 & 1) && !(w2 & 1) && (h2 >> 1) < g.H && (w2 >> 1) < g.W;
            hi = h2 >> 1;
            wi = w2 >> 1;
        } else {
            const int h2 = ho0 - 1 + hy, w2 = wo0 - 1 + wx;
            ok = ok && (unsigned)h2 < (unsigned)Hin && (unsigned)w2 < (unsigned)Win;
            hi = h2 >> g.up;
            wi = w2 >> g.up;
        }
        const int64_t off = ((n * g.H + hi) * g.W + wi) * C + c8 * 8;
        return ok ? a.a + off : zsrc;
    };
    auto w_src = [&](int j) __attribute__((always_inline)) -> const uint16_t* {
        const int co = j / KPS, k8 = j - co * KPS;
        // k8 = tap * C8 + channel group; mirrored: tap 8 - tap of the transposed copy
        const int ks = a.flip ? (8 - k8 / C8) * C8 + k8 % C8 : k8;
        return (j < NWS && k8 < K8) ? a.b + (int64_t)co * (9 * C) + ks * 8 : zsrc;
    };
#pragma unroll
    for (int u = 0; u < (NWS + NT - 1) / NT; ++u) {
        const int base = wv * 64 + NT * u;   // first slot of this wave's load
        if (base < NWS) dma16(w_src(base + lane), &sW[base * 8]);
    }
#pragma unroll
    for (int u = 0; u < (NXS + NT - 1) / NT; ++u) {
        const int base = wv * 64 + NT * u;
        if (base < NXS) dma16(x_src(base + lane), &sX[base * 8]);
    }
    __builtin_amdgcn_s_waitcnt(kWaitVm0);
    __syncthreads();

    f32x4 acc[4][FN];
#pragma unroll
    for (int gi = 0; gi < 4; ++gi)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[gi][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // operand of row group gi (output rows rr = 2 wave + gi / 2, columns cc = 16 (gi % 2) + lr) at
    // tap (r, s): staged pixel (sy, sx) = (rr + r, cc + s), or with UP ((rr + r + 1) / 2,
    // (cc + s + 1) / 2) = (wave + (gi / 2 + r + 1) / 2, 8 (gi % 2) + lr / 2 + (lr % 2 + s + 1) / 2).
    // Either way the LDS offset is a per-lane part fixed over the K loop plus a per-step part that
    // depends on gi only through gi / 2.
    int gofs[4];
#pragma unroll
    for (int gi = 0; gi < 4; ++gi)
        gofs[gi] = UP ? (wave * WP + (gi & 1) * 8 + (lr >> 1)) * PS
                      : ((2 * wave + (gi >> 1)) * WP + (gi & 1) * 16 + lr) * PS;
#pragma unroll 3
    for (int ks = 0; ks < NKS; ++ks) {
        const int k8 = ks * 4 + lk;
        int r = 0, s = 0, c0 = 0;
        if (k8 < K8) {   // beyond K the weights are zero; read tap 0
            const int tap = k8 / C8;
            c0 = (k8 - tap * C8) * 8;
            r = tap / 3;
            s = tap - r * 3;
        }
        int tofs[2];
        if constexpr (UP) {
            const int sxo = ((lr & 1) + s + 1) >> 1;
            tofs[0] = (((r + 1) >> 1) * WP + sxo) * PS + c0;
            tofs[1] = (((r + 2) >> 1) * WP + sxo) * PS + c0;
        } else {
            tofs[0] = tofs[1] = (r * WP + s) * PS + c0;
        }
        bf16x8 fb[FN];
#pragma unroll
        for (int j = 0; j < FN; ++j) fb[j] = *reinterpret_cast<const bf16x8*>(&sW[(16 * j + lr) * KP + k8 * 8]);
#pragma unroll
        for (int gi = 0; gi < 4; ++gi) {
            const bf16x8 fa = *reinterpret_cast<const bf16x8*>(&sX[gofs[gi] + tofs[gi >> 1]]);
#pragma unroll
            for (int j = 0; j < FN; ++j)
                acc[gi][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fb[j], acc[gi][j], 0, 0, 0);
        }
    }
    __syncthreads();   // sX is reused for the output tile

    uint16_t* sO = sX;   // [TH * kTileW][CO]
    const bool pool = a.out_f32 && a.pool2;
    if (pool) {
        // data gradient of an upsampled input: each 2 x 2 output block summed into one pixel of the
        // half-size out_f32, as (top pair) + (bottom pair).  Wave w holds output rows 2 w (row tile
        // gi = h) and 2 w + 1 (gi = h + 2) of column half h; a lane the column pairs (q, q + 1), q = 0, 2.
        const int Hc = g.Ho >> 1, Wc = g.Wo >> 1, hc = (ho0 >> 1) + wave;
        float pv[ACC ? FN : 1][2][2];   // ACC: the old values, all loaded before the stores
        if constexpr (ACC) {
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int pr = 0; pr < 2; ++pr) {
                        const int wc = ((wo0 + h * 16 + 4 * lk) >> 1) + pr;
                        pv[j][h][pr] = (hc < Hc && wc < Wc) ? a.add[((n * Hc + hc) * Wc + wc) * CO + 16 * j + lr]
                                                            : 0.f;
                    }
        }
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int pr = 0; pr < 2; ++pr) {
                    const int wc = ((wo0 + h * 16 + 4 * lk) >> 1) + pr;
                    const float y00 = activate(acc[h][j][2 * pr] + bias_r[j], a.relu);
                    const float y01 = activate(acc[h][j][2 * pr + 1] + bias_r[j], a.relu);
                    const float y10 = activate(acc[h + 2][j][2 * pr] + bias_r[j], a.relu);
                    const float y11 = activate(acc[h + 2][j][2 * pr + 1] + bias_r[j], a.relu);
                    float sum = (y00 + y01) + (y10 + y11);
                    if constexpr (ACC) sum = pv[j][h][pr] + sum;
                    if (hc < Hc && wc < Wc) a.out_f32[((n * Hc + hc) * Wc + wc) * CO + 16 * j + lr] = sum;
                    // (for dpre: [TH / 2 * kTileW / 2][CO])
                    sO[(wave * (kTileW / 2) + h * 8 + 2 * lk + pr) * CO + 16 * j + lr] = f2bf(sum);
                }
    }
    // (one instantiation of the loop per activation; two outputs of a lane, neighbouring pixels of
    // one channel, share one bf16 conversion)
    auto write_tile = [&](auto act_c) __attribute__((always_inline)) {
        constexpr int ACT = decltype(act_c)::value;
#pragma unroll
    for (int gi = 0; gi < 4; ++gi) {
        const int rr = 2 * wave + (gi >> 1), ho = ho0 + rr;
        // ACC (a.add is added to the FP32 output): its values for this row group, all loaded before the
        // stores (a load issued after a store waits for it)
        float prev[ACC ? FN : 1][4];
        if constexpr (ACC) {
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int wo = wo0 + (gi & 1) * 16 + 4 * lk + q;
                    prev[j][q] = (ho < g.Ho && wo < g.Wo)
                                     ? a.add[((n * g.Ho + ho) * g.Wo + wo) * CO + 16 * j + lr]
                                     : 0.f;
                }
        }
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const int co = 16 * j + lr;
#pragma unroll
            for (int q = 0; q < 4; q += 2) {
                const int cc = (gi & 1) * 16 + 4 * lk + q;
                float y0 = activate_c<ACT>(acc[gi][j][q] + bias_r[j]);
                float y1 = activate_c<ACT>(acc[gi][j][q + 1] + bias_r[j]);
                if constexpr (ACC) {
                    y0 = prev[j][q] + y0;
                    y1 = prev[j][q + 1] + y1;
                }
                const uint32_t pk = pack_bf16x2(y0, y1);
                sO[(rr * kTileW + cc) * CO + co] = (uint16_t)pk;
                sO[(rr * kTileW + cc + 1) * CO + co] = (uint16_t)(pk >> 16);
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int wo = wo0 + cc + t;
                    if (a.out_f32 && ho < g.Ho && wo < g.Wo)
                        a.out_f32[((n * g.Ho + ho) * g.Wo + wo) * CO + co] = t ? y1 : y0;
                }
            }
        }
    }
    };
    if (pool) {
    } else if (a.relu == 1) write_tile(std::integral_constant<int, 1>{});
    else if (a.relu == 2) write_tile(std::integral_constant<int, 2>{});
    else write_tile(std::integral_constant<int, 0>{});
    __syncthreads();
    if (a.dpre) {
        // the masked gradient of the layer below, bf16(out_f32 [mask > 0]), and this block's column sums of it.  A
        // pass of its own (k_mask_colsum) reads out_f32 again: 16 -> 16 channels on 2097152 pixels 38 + 55 us, here 65
        const int tw = pool ? kTileW / 2 : kTileW, th = pool ? TH / 2 : TH;
        const int Hp = pool ? g.Ho >> 1 : g.Ho, Wp = pool ? g.Wo >> 1 : g.Wo;
        const int hp0 = pool ? ho0 >> 1 : ho0, wp0 = pool ? wo0 >> 1 : wo0;
        const int c8 = tid % CO8 * 8;   // the same for every chunk of a thread
        int64_t op[CO8];
        u32x4 mv[CO8];
#pragma unroll
        for (int u = 0; u < CO8; ++u) {
            const int pix = (tid + NT * u) / CO8, rr = pix / tw, h = hp0 + rr, w = wp0 + pix - rr * tw;
            const bool in = (int)(rr < th) & (int)(h < Hp) & (int)(w < Wp);
            op[u] = in ? (((int64_t)n * Hp + h) * Wp + w) * CO + c8 : -1;
            mv[u] = in ? *reinterpret_cast<const u32x4*>(a.mask + op[u]) : zero;
        }
        float sum[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) sum[q] = 0.f;
#pragma unroll
        for (int u = 0; u < CO8; ++u) {
            if (op[u] < 0) continue;
            u32x4 v = *reinterpret_cast<const u32x4*>(&sO[(tid + NT * u) / CO8 * CO + c8]);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float lo = __uint_as_float(mv[u][q] << 16), hi = __uint_as_float(mv[u][q] & 0xFFFF0000u);
                v[q] = (lo > 0.f ? v[q] & 0xFFFFu : 0u) | (hi > 0.f ? v[q] & 0xFFFF0000u : 0u);
                sum[2 * q] += __uint_as_float(v[q] << 16);
                sum[2 * q + 1] += __uint_as_float(v[q] & 0xFFFF0000u);
            }
            *reinterpret_cast<u32x4*>(a.dpre + op[u]) = v;
        }
        float* red = reinterpret_cast<float*>(sW);   // [waves][CO] (the weights were last read before the barriers above)
        static_assert(sizeof(sW) >= NT / 64 * CO * sizeof(float), "column sums in the weights' space");
#pragma unroll
        for (int q = 0; q < 8; ++q) {
#pragma unroll
            for (int m = CO8; m < 64; m <<= 1) sum[q] += __shfl_xor(sum[q], m);
            if (lane < CO8) red[wave * CO + c8 + q] = sum[q];
        }
        __syncthreads();
        if (tid < CO) {
            float t = 0.f;
            for (int w = 0; w < NT / 64; ++w) t += red[w * CO + tid];
            a.colsum[(int64_t)blockIdx.x * CO + tid] = t;
        }
        return;
    }
    const int ld2 = a.ld_out2 ? a.ld_out2 : CO;
    // 16-byte output chunks: thread tid takes chunks tid + NT u; the skip tensor's chunks are all
    // loaded before the first store
    static_assert(TH * kTileW == NT, "one output pixel per thread and channel group");
    // one extra chunk per pixel (the depth integral into S0): pixel tid's, loaded with the skip
    // chunks before the first store
    const bool extra1 = a.extra && a.out2_bf16 && a.extra_c == 8;
    const int64_t op_t = (n * g.Ho + ho0 + tid / kTileW) * g.Wo + wo0 + tid % kTileW;
    const bool in_t = ho0 + tid / kTileW < g.Ho && wo0 + tid % kTileW < g.Wo;
    const u32x4 ev = (extra1 && in_t) ? *reinterpret_cast<const u32x4*>(a.extra + op_t * 8) : zero;
    u32x4 kv[CO8];
#pragma unroll
    for (int u = 0; u < CO8; ++u) {
        const int i = tid + NT * u, c8 = i % CO8, pix = i / CO8;
        const int rr = pix / kTileW, cc = pix - rr * kTileW;
        const int ho = ho0 + rr, wo = wo0 + cc;
        kv[u] = (a.skip && a.out2_bf16 && ho < g.Ho && wo < g.Wo)
                    ? *reinterpret_cast<const u32x4*>(a.skip + ((n * g.Ho + ho) * g.Wo + wo) * CO + c8 * 8)
                    : zero;
    }
#pragma unroll
    for (int u = 0; u < CO8; ++u) {
        const int i = tid + NT * u, c8 = i % CO8, pix = i / CO8;
        const int rr = pix / kTileW, cc = pix - rr * kTileW;
        const int ho = ho0 + rr, wo = wo0 + cc;
        if (ho >= g.Ho || wo >= g.Wo) continue;
        const int64_t op = (n * g.Ho + ho) * g.Wo + wo;
        const u32x4 v = *reinterpret_cast<const u32x4*>(&sO[pix * CO + c8 * 8]);
        if (a.out_bf16) *reinterpret_cast<u32x4*>(a.out_bf16 + op * CO + c8 * 8) = v;
        if (a.skip && a.out2_bf16) {
            const u32x4 k = kv[u];
            u32x4 o;
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j] = add_bf16x2(v[j], k[j]);
            *reinterpret_cast<u32x4*>(a.out2_bf16 + op * ld2 + c8 * 8) = o;
        }
    }
    if (extra1) {
        if (in_t) *reinterpret_cast<u32x4*>(a.out2_bf16 + op_t * ld2 + CO) = ev;
    } else if (a.extra && a.out2_bf16) {
        const int E8 = a.extra_c / 8;
        for (int i = tid; i < TH * kTileW * E8; i += NT) {
            const int e8 = i % E8, pix = i / E8;
            const int rr = pix / kTileW, cc = pix - rr * kTileW;
            const int ho = ho0 + rr, wo = wo0 + cc;
            if (ho >= g.Ho || wo >= g.Wo) continue;
            const int64_t op = (n * g.Ho + ho) * g.Wo + wo;
            *reinterpret_cast<u32x4*>(a.out2_bf16 + op * ld2 + CO + e8 * 8) =
                *reinterpret_cast<const u32x4*>(a.extra + op * a.extra_c + e8 * 8);
        }
    }
    if (a.head_out && tid < TH * kTileW) {
        const int rr = tid / kTileW, cc = tid - rr * kTileW;
        const int ho = ho0 + rr, wo = wo0 + cc;
        if (ho < g.Ho && wo < g.Wo) {
            float sum = 0.f;
#pragma unroll
            for (int co = 0; co < CO; ++co) sum += bf2f(a.head_w[co]) * bf2f(sO[tid * CO + co]);
            a.head_out[(n * g.Ho + ho) * g.Wo + wo] = sum + a.head_b[0];
        }
    }
}

// 3x3 convolution (stride 1, pad 1) of many channels: a block computes 16 x 16 output pixels of one image for
// 64 output channels.  The im2col GEMM fetches every input pixel nine times from L2 (453 MB for 128 -> 64
// channels on 131072 pixels, at 15 TB/s: that, not the matrix cores, bounds it); here the tile's input with its
// halo is fetched once into LDS (all C channels; with UP the stored pixels, 10 x 10 of them) and only the
// weights stream, 64 K of the 64 channels a step, through a three-stage ring of LDS DMA.  Eight waves of 64
// pixels x 32 channels; K runs over taps and channels in the GEMM's order, so the results are its bits.  No unit
// is full: LDS (six reads for eight products) is busy 45-61 % of the time in large launches, the matrix cores 36-54 %,
// the VALU 35-43 %, and the rest is the steps' latency; on 131072 pixels LDS and matrix cores are both under 30 %.
// 131072 pixels of 128 -> 64 upsampled 28.4 -> 23.5 us, of 64 -> 64 22.6 -> 15.8 us.
// MODE kDgrad, the data gradient of such a layer: a is dy, b the [Ci][9][Co] copy, tap (r, s) reads dy at
// (2 - r, 2 - s) of the halo; FP32 output plus add, with pool2 (an upsampled input's gradient) summed over 2 x 2
// pixels, a lane's four sums.  Against the GEMM, 131072 pixels: 64 -> 64 28.0 -> 20.5 us, 128 -> 64 upsampled 38.1 ->
// 26.0 us (with stores that test the image's edge one by one it was no faster than the GEMM).
// The 16 rows of an MFMA operand are 2 x 8 pixels in 2 x 2 quads (row 4 q + 2 dy + dx): with UP four of them read
// one or two stored pixels.
constexpr int kHaloK = 64, kHaloThreads = 512;   // (kHaloT, kHaloN: conv_rules.h)

template <int MODE, int C, bool UP>
__global__ __launch_bounds__(kHaloThreads, 4) void k_conv3x3_halo(ConvGeom g, ConvArgs a)
{
    constexpr int XC = UP ? kHaloT / 2 + 2 : kHaloT + 2, C8 = C / 8;   // staged rows and columns
    constexpr int NX = XC * XC * C8, NXP = (NX + 63) / 64 * 64;        // 16-byte chunks of the halo
    constexpr int SW = kHaloN * kHaloK;                                // bf16 of a weight stage
    constexpr int TP = kHaloN + 8;                                     // row of the output tile
    constexpr int OPS = NXP * 8 + 3 * SW, OUT = MODE == kFwd ? kHaloT * kHaloT * TP : 0;
    static_assert(C % kHaloK == 0 && (kHaloN * kHaloK) / 8 == kHaloThreads, "one weight chunk per thread and step");
    __shared__ __attribute__((aligned(16))) uint16_t smem[OPS > OUT ? OPS : OUT];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lk = lane >> 4, wm = wv >> 1, wn = wv & 1;
    // blocks of one pixel tile (its channel groups) follow each other on one XCD
    uint32_t b = blockIdx.x;
    const uint32_t nblk = gridDim.x;
    if ((nblk & 7) == 0) b = (b & 7) * (nblk >> 3) + (b >> 3);
    const uint32_t ng = (uint32_t)g.Co / kHaloN;
    const uint32_t tile = b / ng;
    const int n_base = (int)(b - tile * ng) * kHaloN;
    const int tiles_x = (g.Wo + kHaloT - 1) / kHaloT, tiles_y = (g.Ho + kHaloT - 1) / kHaloT;
    const int n = (int)(tile / (uint32_t)(tiles_x * tiles_y)), t_in = (int)tile - n * tiles_x * tiles_y;
    const int ho0 = t_in / tiles_x * kHaloT, wo0 = t_in % tiles_x * kHaloT;
    const uint64_t zp = reinterpret_cast<uint64_t>(g_zero_buf);
    const uint32_t zhi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(zp >> 32));
    const uint32_t zlo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)zp);
    const uint16_t* zsrc = reinterpret_cast<const uint16_t*>(((uint64_t)zhi << 32) | zlo);
    // chunk q of staged pixel (r, c) sits in slot q ^ key: the 2 x 8 pixels of an operand read then lie in 16
    // distinct 16-byte groups of 256 bytes
    auto key = [](int r, int c) { return C8 == 8 ? ((c >> 1) & 3) | ((r & 1) << 2) : (c & 7) | ((r & 1) << 3); };
    const int h0 = (UP ? ho0 / 2 : ho0) - 1, w0 = (UP ? wo0 / 2 : wo0) - 1;
    const uint16_t* xb = a.a + (((int64_t)n * g.H + h0) * g.W + w0) * C;
#pragma unroll
    for (int k = 0; k < (NXP + kHaloThreads - 1) / kHaloThreads; ++k) {
        if ((k + 1) * kHaloThreads > NXP && wv * 64 + k * kHaloThreads >= NXP) continue;
        const int i = tid + k * kHaloThreads, px = i / C8, r = px / XC, c = px - r * XC;
        const int q = (i % C8) ^ key(r, c);
        const bool ok = (int)(i < NX) & (int)((unsigned)(h0 + r) < (unsigned)g.H) & (int)((unsigned)(w0 + c) < (unsigned)g.W);
        dma16(ok ? xb + (int64_t)(r * g.W + c) * C + q * 8 : zsrc, smem + (wv * 64 + k * kHaloThreads) * 8);
    }
    // weight stage: row tid / 8 (output channel), chunk q in slot q ^ (row / 2 % 8)
    const uint16_t* wsrc = a.b + (int64_t)(n_base + (tid >> 3)) * g.kb + ((tid & 7) ^ ((tid >> 4) & 7)) * 8;
    uint16_t* sW = smem + NXP * 8;
    auto issue = [&](int kt, int st) __attribute__((always_inline)) { dma16(wsrc + kt * kHaloK, sW + st * SW + wv * 512); };
    float bias_r[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) bias_r[j] = (MODE == kFwd && a.bias) ? a.bias[n_base + wn * 32 + j * 16 + lr] : 0.f;
    f32x4 acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // row tile i of the wave: output rows 4 wm + 2 (i / 2) + rb, columns 8 (i % 2) + cl
    const int rb = (lr >> 1) & 1, cl = 2 * (lr >> 2) + (lr & 1);
    const uint16_t* wrow = sW + (wn * 32 + lr) * kHaloK;
    constexpr int NK = 9 * C / kHaloK, KT = C / kHaloK;   // steps, and steps per tap
    issue(0, 0);
    issue(1, 1);
    int st = 0, st2 = 2, kt = 0;
#pragma unroll 1
    for (int t = 0; t < 9; ++t) {
        const int r = MODE == kDgrad ? 2 - t / 3 : t / 3, s = MODE == kDgrad ? 2 - t % 3 : t % 3;
        // staged pixel of row tile 0 and its key; those of the others follow (i % 2: 8 columns on, UP 4; i / 2: 2
        // rows on, UP 1)
        const int sr = UP ? 2 * wm + ((rb + r + 1) >> 1) : 4 * wm + rb + r;
        const int sc = UP ? (cl + s + 1) >> 1 : cl + s;
        const int kx = key(sr, sc) ^ lk;
        const uint16_t* xrow = smem + (sr * XC + sc) * C;
#pragma unroll
        for (int kc = 0; kc < KT; ++kc, ++kt) {
            if (kt + 1 < NK) __builtin_amdgcn_s_waitcnt(kWaitVm0 | 1);   // this step's stage (and the halo) has landed
            else __builtin_amdgcn_s_waitcnt(kWaitVm0);
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (kt + 2 < NK) issue(kt + 2, st2);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                bf16x8 fa[4], fb[2];
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    fb[j] = *reinterpret_cast<const bf16x8*>(wrow + st * SW + j * 16 * kHaloK + (((u * 4 + lk) ^ (lr >> 1)) * 8));
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    constexpr int B8 = C8 == 8 ? 1 : 2;   // key bit of column bit 2 (UP)
                    const int ko = UP ? ((i & 1) << B8) ^ ((i >> 1) << (B8 + 1)) : 0;
                    fa[i] = *reinterpret_cast<const bf16x8*>(xrow + ((i >> 1) * (UP ? 1 : 2) * XC + (i & 1) * (UP ? 4 : 8)) * C +
                                                             ((kx ^ ko ^ ((kc * 2 + u) * 4)) * 8));
                }
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
            }
            st = st == 2 ? 0 : st + 1;
            st2 = st2 == 2 ? 0 : st2 + 1;
        }
    }
    // lane (lr, lk), element e of acc[i][j]: output pixel (4 wm + 2 (i / 2) + e / 2, 8 (i % 2) + 2 lk + e % 2),
    // channel n_base + 32 wn + 16 j + lr
    if constexpr (MODE == kDgrad) {
        // (whole tiles only, so no store is conditional; what is added is all loaded before the first store)
        const int64_t Co = g.Co;
        const int ch = n_base + wn * 32 + lr;
        if (a.pool2) {
            const int W2 = g.Wo >> 1;
            const int64_t o0 = (((int64_t)n * (g.Ho >> 1) + ho0 / 2 + 2 * wm) * W2 + wo0 / 2 + lk) * Co + ch;
            float pre[4][2];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    pre[i][j] = a.add ? a.add[o0 + ((i >> 1) * W2 + 4 * (i & 1)) * Co + 16 * j] : 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const float v = (acc[i][j][0] + acc[i][j][1]) + (acc[i][j][2] + acc[i][j][3]);
                    a.out_f32[o0 + ((i >> 1) * W2 + 4 * (i & 1)) * Co + 16 * j] = a.add ? pre[i][j] + v : v;
                }
            return;
        }
        const int64_t o0 = (((int64_t)n * g.Ho + ho0 + 4 * wm) * g.Wo + wo0 + 2 * lk) * Co + ch;
        auto at = [&](int i, int j, int e) __attribute__((always_inline)) {
            return o0 + ((2 * (i >> 1) + (e >> 1)) * g.Wo + 8 * (i & 1) + (e & 1)) * Co + 16 * j;
        };
        if (a.add) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[i][j][e] = a.add[at(i, j, e)] + acc[i][j][e];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) a.out_f32[at(i, j, e)] = acc[i][j][e];
        return;
    }
    uint16_t* sT = smem;
    __syncthreads();
    auto write_tile = [&](auto act_c) __attribute__((always_inline)) {
        constexpr int ACT = decltype(act_c)::value;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int co = wn * 32 + j * 16 + lr;
#pragma unroll
                for (int e = 0; e < 4; e += 2) {
                    const int rr = 4 * wm + 2 * (i >> 1) + (e >> 1), cc = 8 * (i & 1) + 2 * lk;
                    const float y0 = activate_c<ACT>(acc[i][j][e] + bias_r[j]);
                    const float y1 = activate_c<ACT>(acc[i][j][e + 1] + bias_r[j]);
                    const uint32_t pk = pack_bf16x2(y0, y1);
                    sT[(rr * kHaloT + cc) * TP + co] = (uint16_t)pk;
                    sT[(rr * kHaloT + cc + 1) * TP + co] = (uint16_t)(pk >> 16);
                    if (a.out_f32) {
                        const int ho = ho0 + rr, wo = wo0 + cc;
                        float* o = a.out_f32 + (((int64_t)n * g.Ho + ho) * g.Wo + wo) * g.Co + n_base + co;
                        if (ho < g.Ho && wo < g.Wo) o[0] = y0;
                        if (ho < g.Ho && wo + 1 < g.Wo) o[g.Co] = y1;
                    }
                }
            }
    };
    if (a.relu == 1) write_tile(std::integral_constant<int, 1>{});
    else if (a.relu == 2) write_tile(std::integral_constant<int, 2>{});
    else write_tile(std::integral_constant<int, 0>{});
    __syncthreads();
    // 16-byte chunks; the skip tensor's are all loaded before the first store (a load after a store waits)
    constexpr int CPT = kHaloT * kHaloT * kHaloN / 8 / kHaloThreads;
    const int ld2 = a.ld_out2 ? a.ld_out2 : g.Co;
    const bool skip = a.skip && a.out2_bf16;
    const int c8 = tid % (kHaloN / 8) * 8;
    u32x4 kv[CPT];
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
        const int px = (tid + u * kHaloThreads) / (kHaloN / 8), ho = ho0 + px / kHaloT, wo = wo0 + px % kHaloT;
        kv[u] = u32x4{0u, 0u, 0u, 0u};
        if (skip && ho < g.Ho && wo < g.Wo)
            kv[u] = *reinterpret_cast<const u32x4*>(a.skip + (((int64_t)n * g.Ho + ho) * g.Wo + wo) * g.Co + n_base + c8);
    }
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
        const int px = (tid + u * kHaloThreads) / (kHaloN / 8), ho = ho0 + px / kHaloT, wo = wo0 + px % kHaloT;
        if (ho >= g.Ho || wo >= g.Wo) continue;
        const int64_t op = ((int64_t)n * g.Ho + ho) * g.Wo + wo;
        const u32x4 v = *reinterpret_cast<const u32x4*>(&sT[px * TP + c8]);
        if (a.out_bf16) *reinterpret_cast<u32x4*>(a.out_bf16 + op * g.Co + n_base + c8) = v;
        if (skip) {
            u32x4 o;
#pragma unroll
            for (int q = 0; q < 4; ++q) o[q] = add_bf16x2(v[q], kv[u][q]);
            *reinterpret_cast<u32x4*>(a.out2_bf16 + op * ld2 + n_base + c8) = o;
        }
    }
}

// Two 3x3 convolutions (stride 1, pad 1, ReLU) in one pass, for inference, where nothing reads the tensor between
// them: the first (C -> CM channels; UP: its input read upsampled x2, its output added to skip) and the second
// ((CM + EX) -> CO; EX further input channels come from extra).  These layers are bound by memory, and the tensor
// between is written and read once per pass otherwise (64 to 96 bytes a pixel).  A block stages the first input's
// tile with a halo of two pixels and both weights (DMA), computes the 18 x 34 pixels of the tensor between that
// its 16 x 32 outputs need into LDS (bf16, zero outside the image, the second conv's padding) and continues from
// there; the halo costs a fifth of the first conv again.  K order and roundings are k_conv3x3_tile's: same bits.
// 33554432 pixels, 8 -> 16 -> 16 channels: 333 + 453 us as two passes, 549 us here; 32 upsampled -> 16 (+ 8) -> 16
// and the head: 759 + 545 and 54 us for the clamp, 1140 us here.  Bound by LDS reads (a 16-channel product
// needs one each; LDS busy 72-77 % of the time, nearly half of that bank conflicts) and by the VALU (73-76 %).
// 64 upsampled -> 32 -> 32 on a quarter of the pixels takes 131 KB of LDS, one block per compute unit, and is
// slower (893 against 386 + 266 us), so those stay apart.
template <int C, bool UP, int CM, int EX, int CO>
__global__ __launch_bounds__(512, 4) void k_conv3x3_pair(PairArgs a)
{
    constexpr int TH = 16, TW = 32, NT = 512, IW = TW + 2, NP = (TH + 2) * IW;   // NP: pixels between
    constexpr int HP = UP ? TH / 2 + 2 : TH + 4, WP = UP ? TW / 2 + 2 : TW + 4;  // staged input pixels
    constexpr int C8 = C / 8, PS = C8 % 2 == 0 ? C + 8 : C, K8 = 9 * C8, NKS = (K8 + 3) / 4, KP = NKS * 32 + 8;
    constexpr int CT = CM + EX, T8 = CT / 8, PT = T8 % 2 == 0 ? CT + 8 : CT, L8 = 9 * T8, NLS = (L8 + 3) / 4,
                  LP = NLS * 32 + 8;
    constexpr int FM = CM / 16, FO = CO / 16, NF = (NP + 127) / 128;   // NF: row tiles of a wave in the first conv
    constexpr int SPP = PS / 8, KPS = KP / 8, LPS = LP / 8;
    constexpr int NXS = HP * WP * SPP, NWS = CM * KPS, NVS = CO * LPS;   // 16-byte slots
    constexpr int XS = (NXS + 63) / 64 * 512, WS = (NWS + 63) / 64 * 512, VS = (NVS + 63) / 64 * 512;
    constexpr int OS = TH * TW * CO;
    __shared__ __attribute__((aligned(16))) uint16_t sX[XS + WS > OS ? XS + WS : OS];   // input, weights; then output
    __shared__ __attribute__((aligned(16))) uint16_t sV[VS];
    __shared__ __attribute__((aligned(16))) uint16_t sT[NP * PT];
    uint16_t* sW = sX + XS;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lr = lane & 15, lk = lane >> 4;
    const int Ho = a.H, Wo = a.W, Hs = UP ? Ho >> 1 : Ho, Ws = UP ? Wo >> 1 : Wo;
    const int tiles_x = (Wo + TW - 1) / TW, tiles_y = (Ho + TH - 1) / TH;
    uint32_t b = blockIdx.x;   // neighbouring tiles on the same XCD
    const uint32_t nb = gridDim.x;
    if ((nb & 7) == 0) b = (b & 7) * (nb >> 3) + (b >> 3);
    const int n = (int)(b / (uint32_t)(tiles_x * tiles_y)), t_in = (int)b - n * tiles_x * tiles_y;
    const int ho0 = t_in / tiles_x * TH, wo0 = t_in % tiles_x * TW;
    const u32x4 zero = {0u, 0u, 0u, 0u};
    float bias1[FM], bias2[FO];
#pragma unroll
    for (int j = 0; j < FM; ++j) bias1[j] = a.b1[16 * j + lr];
#pragma unroll
    for (int j = 0; j < FO; ++j) bias2[j] = a.b2[16 * j + lr];
    const uint64_t zp = reinterpret_cast<uint64_t>(g_zero_buf);
    const uint32_t zhi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(zp >> 32));
    const uint32_t zlo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)zp);
    const uint16_t* zsrc = reinterpret_cast<const uint16_t*>(((uint64_t)zhi << 32) | zlo);
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    const int h0 = UP ? ho0 / 2 - 1 : ho0 - 2, w0 = UP ? wo0 / 2 - 1 : wo0 - 2;
#pragma unroll
    for (int u = 0; u < (NXS + NT - 1) / NT; ++u) {
        const int base = wv * 64 + NT * u, j = base + lane;
        const int pix = j / SPP, c8 = j - pix * SPP, hy = pix / WP, wx = pix - hy * WP;
        const bool ok = (int)(j < NXS) & (int)(c8 < C8) & (int)((unsigned)(h0 + hy) < (unsigned)Hs) &
                        (int)((unsigned)(w0 + wx) < (unsigned)Ws);
        const int64_t off = (((int64_t)n * Hs + h0 + hy) * Ws + w0 + wx) * C + c8 * 8;
        if (base < NXS) dma16(ok ? a.x + off : zsrc, &sX[base * 8]);
    }
    auto weights = [&](const uint16_t* w, uint16_t* dst, auto slots_c, auto row_c, auto k8_c) __attribute__((always_inline)) {
        constexpr int SL = decltype(slots_c)::value, RS = decltype(row_c)::value, KK = decltype(k8_c)::value;
#pragma unroll
        for (int u = 0; u < (SL + NT - 1) / NT; ++u) {
            const int base = wv * 64 + NT * u, j = base + lane, co = j / RS, k8 = j - co * RS;
            const bool ok = (int)(j < SL) & (int)(k8 < KK);
            if (base < SL) dma16(ok ? w + (int64_t)co * (8 * KK) + k8 * 8 : zsrc, dst + base * 8);
        }
    };
    weights(a.w1, sW, std::integral_constant<int, NWS>{}, std::integral_constant<int, KPS>{}, std::integral_constant<int, K8>{});
    weights(a.w2, sV, std::integral_constant<int, NVS>{}, std::integral_constant<int, LPS>{}, std::integral_constant<int, L8>{});
    // chunks of the tensor between that this thread completes (skip and extra, zero outside the image), their
    // loads in flight with the DMA; pixel p of it is (ho0 - 1 + p / IW, wo0 - 1 + p % IW)
    constexpr int M8 = CM / 8, SI = (NP * M8 + NT - 1) / NT, EI = EX ? (NP * (EX / 8) + NT - 1) / NT : 0;
    static_assert(EX == 0 || EX == 8, "one further chunk per pixel");
    auto inside = [&](int p, int64_t& px) __attribute__((always_inline)) -> bool {
        const int h = ho0 - 1 + p / IW, w = wo0 - 1 + p % IW;
        px = ((int64_t)n * Ho + h) * Wo + w;
        return (int)(p < NP) & (int)((unsigned)h < (unsigned)Ho) & (int)((unsigned)w < (unsigned)Wo);
    };
    u32x4 kv[UP ? SI : 1], ev[EX ? EI : 1];
    if constexpr (UP) {
#pragma unroll
        for (int u = 0; u < SI; ++u) {
            const int i = tid + NT * u;
            int64_t px;
            kv[u] = inside(i / M8, px) ? *reinterpret_cast<const u32x4*>(a.skip + px * CM + i % M8 * 8) : zero;
        }
    }
    if constexpr (EX) {
#pragma unroll
        for (int u = 0; u < EI; ++u) {
            int64_t px;
            ev[u] = inside(tid + NT * u, px) ? *reinterpret_cast<const u32x4*>(a.extra + px * EX) : zero;
        }
    }
    __builtin_amdgcn_s_waitcnt(kWaitVm0);
    __syncthreads();
    // first conv: wave w takes the row tiles w, w + 8, ... of 16 consecutive pixels between
    {
        f32x4 acc[NF][FM];
        int pr[NF], pc[NF];   // row and column of this lane's pixel (past the last: the last)
#pragma unroll
        for (int i = 0; i < NF; ++i) {
            const int p = min((wave + 8 * i) * 16 + lr, NP - 1);
            pr[i] = p / IW;
            pc[i] = p - pr[i] * IW;
#pragma unroll
            for (int j = 0; j < FM; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll 3
        for (int ks = 0; ks < NKS; ++ks) {
            const int k8 = ks * 4 + lk;
            int r = 0, s = 0, c0 = 0;
            if (k8 < K8) {   // beyond K the weights are zero; read tap 0
                const int tap = k8 / C8;
                c0 = (k8 - tap * C8) * 8;
                r = tap / 3;
                s = tap - r * 3;
            }
            bf16x8 fb[FM];
#pragma unroll
            for (int j = 0; j < FM; ++j) fb[j] = *reinterpret_cast<const bf16x8*>(&sW[(16 * j + lr) * KP + k8 * 8]);
#pragma unroll
            for (int i = 0; i < NF; ++i) {
                const int q = UP ? ((pr[i] + r) >> 1) * WP + ((pc[i] + s) >> 1) : (pr[i] + r) * WP + pc[i] + s;
                const bf16x8 fa = *reinterpret_cast<const bf16x8*>(&sX[q * PS + c0]);
#pragma unroll
                for (int j = 0; j < FM; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fb[j], acc[i][j], 0, 0, 0);
            }
        }
#pragma unroll
        for (int i = 0; i < NF; ++i)
#pragma unroll
            for (int j = 0; j < FM; ++j)
#pragma unroll
                for (int q = 0; q < 4; q += 2) {
                    const int p = (wave + 8 * i) * 16 + 4 * lk + q;
                    const uint32_t pk = pack_bf16x2(fmaxf(acc[i][j][q] + bias1[j], 0.f), fmaxf(acc[i][j][q + 1] + bias1[j], 0.f));
                    if (p < NP) {   // NP is even
                        sT[p * PT + 16 * j + lr] = (uint16_t)pk;
                        sT[(p + 1) * PT + 16 * j + lr] = (uint16_t)(pk >> 16);
                    }
                }
    }
    static_assert(NP % 2 == 0, "pairs of pixels");
    __syncthreads();
#pragma unroll
    for (int u = 0; u < SI; ++u) {
        const int i = tid + NT * u, p = i / M8;
        int64_t px;
        const bool in = inside(p, px);
        if (p >= NP || (!UP && in)) continue;
        u32x4* t = reinterpret_cast<u32x4*>(&sT[p * PT + i % M8 * 8]);
        u32x4 o = zero;
        if constexpr (UP) {
            if (in) {
                const u32x4 v = *t;
#pragma unroll
                for (int q = 0; q < 4; ++q) o[q] = add_bf16x2(v[q], kv[u][q]);
            }
        }
        *t = o;
    }
    if constexpr (EX) {
#pragma unroll
        for (int u = 0; u < EI; ++u)
            if (tid + NT * u < NP) *reinterpret_cast<u32x4*>(&sT[(tid + NT * u) * PT + CM]) = ev[u];
    }
    __syncthreads();
    // second conv, as k_conv3x3_tile from its staged halo tile
    f32x4 acc[4][FO];
#pragma unroll
    for (int gi = 0; gi < 4; ++gi)
#pragma unroll
        for (int j = 0; j < FO; ++j) acc[gi][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 3
    for (int ks = 0; ks < NLS; ++ks) {
        const int k8 = ks * 4 + lk;
        int tofs = 0;
        if (k8 < L8) {
            const int tap = k8 / T8, r = tap / 3;
            tofs = (r * IW + tap - r * 3) * PT + (k8 - tap * T8) * 8;
        }
        bf16x8 fb[FO];
#pragma unroll
        for (int j = 0; j < FO; ++j) fb[j] = *reinterpret_cast<const bf16x8*>(&sV[(16 * j + lr) * LP + k8 * 8]);
#pragma unroll
        for (int gi = 0; gi < 4; ++gi) {
            const bf16x8 fa = *reinterpret_cast<const bf16x8*>(
                &sT[((2 * wave + (gi >> 1)) * IW + (gi & 1) * 16 + lr) * PT + tofs]);
#pragma unroll
            for (int j = 0; j < FO; ++j)
                acc[gi][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fb[j], acc[gi][j], 0, 0, 0);
        }
    }
    uint16_t* sO = sX;   // [TH * TW][CO] (the input and its weights were last read before the barriers above)
#pragma unroll
    for (int gi = 0; gi < 4; ++gi)
#pragma unroll
        for (int j = 0; j < FO; ++j)
#pragma unroll
            for (int q = 0; q < 4; q += 2) {
                const int o = ((2 * wave + (gi >> 1)) * TW + (gi & 1) * 16 + 4 * lk + q) * CO + 16 * j + lr;
                const uint32_t pk = pack_bf16x2(fmaxf(acc[gi][j][q] + bias2[j], 0.f), fmaxf(acc[gi][j][q + 1] + bias2[j], 0.f));
                sO[o] = (uint16_t)pk;
                sO[o + CO] = (uint16_t)(pk >> 16);
            }
    __syncthreads();
    if (a.out) {
        constexpr int O8 = CO / 8;
#pragma unroll
        for (int u = 0; u < O8; ++u) {
            const int i = tid + NT * u, pix = i / O8, ho = ho0 + pix / TW, wo = wo0 + pix % TW;
            if (ho < Ho && wo < Wo)
                *reinterpret_cast<u32x4*>(a.out + (((int64_t)n * Ho + ho) * Wo + wo) * CO + i % O8 * 8) =
                    *reinterpret_cast<const u32x4*>(&sO[pix * CO + i % O8 * 8]);
        }
    }
    if constexpr (CO == 16) {
        if (a.head_out) {   // the 1x1 head with one output, clamped to [0, 1]
            const int ho = ho0 + tid / TW, wo = wo0 + tid % TW;
            if (ho < Ho && wo < Wo) {
                float sum = 0.f;
#pragma unroll
                for (int co = 0; co < CO; ++co) sum += bf2f(a.head_w[co]) * bf2f(sO[tid * CO + co]);
                const float y = fminf(fmaxf(sum + a.head_b[0], 0.f), 1.f);
                const int64_t px = ((int64_t)n * Ho + ho) * Wo + wo;
                a.head_out[px] = y;
                if (a.head_bf16) a.head_bf16[px] = f2bf(y);
            }
        }
    }
}

// Direct 3x3 weight gradient (pad 1; stride 1, or 2 with S2): dW[co][r][s][ci] = sum over
// output pixels p of dy[p][co] x[p + (r - 1, s - 1)][ci], for a group of CI in
// {8, 16, 24, 32} input and CO in {16, 32} output channels (block y: input
// group, block z: output group, of a layer with g.C and g.Co channels).  The
// contraction runs over pixels while memory holds channels together: a block
// copies, per tile of 8 (stride 2: 4) x 32 output pixels, the halo of x and the
// tile of dy as they are into LDS (DMA, the next tile's while this one is
// multiplied; UP: the stored pixels only, fine pixel (h, w) being stored pixel
// (h / 2, w / 2)) and reads the MFMA operands transposed from there
// (ds_read_b64_tr_b16: four pixels of a lane's channel; lanes 16 k .. 16 k + 15
// of a wave hold the addresses of pixels 8 k + i / 4 and channels 4 (i % 4)).
// The three column shifts of a row come from one set of reads by byte alignment.
// A wave owns RW output rows and all 9 CI CO sums; at the end the four waves'
// sums are added in wave order through LDS.
// Bound by the latency between a tile's phases at one to two and a half waves per SIMD, not by memory: with 64
// training pairs LDS is busy 10-14 % of the time, the VALU 15-31 %, the matrix cores 6-37 %.
// With register transposes into channel planes (4-byte LDS stores, three of
// them for each operand read, and 11 million bank-conflict cycles) 128 -> 64
// channels on 131072 pixels, read upsampled, took 42 us, 64 -> 64 channels on
// 131072 pixels 31 us and 32 -> 16 on 2097152 pixels, upsampled, 51 us; now 24,
// 21 and 25 us.
constexpr int kWgW = 32;                              // output columns per tile
constexpr int kWgH = 8, kWgH2 = 4;                    // output rows per tile, stride 1 and 2
template <int CI, int CO, bool UP, bool S2>
struct WgTile {
    static constexpr int TH = S2 ? kWgH2 : kWgH, RW = TH / 4;
    static constexpr int XR = UP ? TH / 2 + 2 : (S2 ? 2 * TH + 1 : TH + 2);        // staged rows of x
    static constexpr int XC = UP ? kWgW / 2 + 2 : (S2 ? 2 * kWgW + 2 : kWgW + 2);  // and columns (the first at -1)
    static constexpr int XN = XR * XC * (CI / 8), DN = TH * kWgW * (CO / 8);       // 16-byte chunks
    static constexpr int XNP = (XN + 63) / 64 * 64;   // whole waves; dy follows, so reads past x stay in the stage
    static constexpr int STAGE = (XNP + DN) * 8;      // bf16
};

// Work groups per compute unit by the registers a thread needs: 9, 18 or 36 quads of sums and the tile's
// operands (direct: stride 1, not upsampled, the most operands).  With 2 for all, 16 x 16 groups took 30.3
// instead of 29.8 us (2097152 pixels), upsampled 32 x 16 ones 27.8 instead of 25.4; 3 for direct 24 x 16 ones
// would spill (47.5 instead of 45.9 us).
constexpr int wgrad_blocks_per_cu(int ci, int co, bool direct)
{
    const int groups = (ci + 15) / 16 * (co / 16);
    return groups == 1 ? 4 : (groups == 2 && !(direct && ci > 16) ? 3 : 2);
}

template <int CI, int CO, bool UP, bool S2>
__global__ __launch_bounds__(256, wgrad_blocks_per_cu(CI, CO, !UP && !S2)) void k_wgrad3x3_tile(ConvGeom g, const uint16_t* __restrict__ x,
                                                          const uint16_t* __restrict__ dy, float* __restrict__ part)
{
    static_assert(!(UP && S2), "stride 2 reads its input directly");
    using T = WgTile<CI, CO, UP, S2>;
    constexpr int NB = (CI + 15) / 16, ND = CO / 16, NA = 9 * NB * ND;
    constexpr int CI8 = CI / 8, CO8 = CO / 8, RW = T::RW, XC = T::XC;
    constexpr int XI = (T::XNP + 255) / 256, DI = (T::DN + 255) / 256;   // DMA loads per thread and stage
    static_assert(T::DN % 256 == 0, "whole blocks of dy chunks");
    static_assert(!S2 || CI <= 16, "stride 2 reads every other pixel: 64-byte ones would use half of the LDS banks");
    __shared__ __attribute__((aligned(16))) uint16_t smem[T::STAGE];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lk = lane >> 4;
    const int tiles_x = (g.Wo + kWgW - 1) / kWgW, tiles_y = (g.Ho + T::TH - 1) / T::TH;
    const uint32_t per_img = (uint32_t)tiles_x * tiles_y;
    const uint32_t total = (uint32_t)(g.Kw / ((int64_t)g.Ho * g.Wo)) * per_img;   // <= Kw = N * Ho * Wo < 2^31
    const uint16_t* xg = x + blockIdx.y * CI;    // the block's input channel group
    const uint16_t* dyg = dy + blockIdx.z * CO;  // and output channel group
    const uint64_t zp = reinterpret_cast<uint64_t>(g_zero_buf);
    const uint32_t zhi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(zp >> 32));
    const uint32_t zlo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)zp);
    const uint16_t* zsrc = reinterpret_cast<const uint16_t*>(((uint64_t)zhi << 32) | zlo);
    // this thread's chunks: row and column in the tile (rows past the staged ones: none), channel offset
    int xy[XI];
#pragma unroll
    for (int k = 0; k < XI; ++k) {
        const int px = (tid + 256 * k) / CI8;
        xy[k] = ((px / XC) << 16) | (px % XC);
    }
    auto issue = [&](uint32_t t) __attribute__((always_inline)) {
        const uint32_t n = t / per_img, t_in = t - n * per_img;
        const int ty = (int)(t_in / (uint32_t)tiles_x), tx = (int)t_in - ty * tiles_x;
        const int ho0 = ty * T::TH, wo0 = tx * kWgW;
        const int h0 = (UP ? ho0 >> 1 : (S2 ? 2 * ho0 : ho0)) - 1, w0 = (UP ? wo0 >> 1 : (S2 ? 2 * wo0 : wo0)) - 1;
        const uint16_t* xb = xg + (((int64_t)n * g.H + h0) * g.W + w0) * g.C;
        const uint16_t* db = dyg + (((int64_t)n * g.Ho + ho0) * g.Wo + wo0) * g.Co;
#pragma unroll
        for (int k = 0; k < XI; ++k) {
            if (wave * 64 + 256 * k >= T::XNP) continue;
            const int r = xy[k] >> 16, c = xy[k] & 0xFFFF;
            const int q = (tid + 256 * k) % CI8;
            const bool ok = (int)((unsigned)(h0 + r) < (unsigned)g.H) & (int)((unsigned)(w0 + c) < (unsigned)g.W) &
                            (int)(256 * k + 255 < T::XN || tid + 256 * k < T::XN);
            dma16(ok ? xb + (int64_t)(r * g.W + c) * g.C + q * 8 : zsrc, smem + (wave * 64 + 256 * k) * 8);
        }
#pragma unroll
        for (int k = 0; k < DI; ++k) {
            const int r = (tid + 256 * k) / (CO8 * kWgW), c = tid / CO8 % kWgW;
            const bool ok = (int)(ho0 + r < g.Ho) & (int)(wo0 + c < g.Wo);
            dma16(ok ? db + (int64_t)(r * g.Wo + c) * g.Co + (tid % CO8) * 8 : zsrc,
                  smem + (T::XNP + wave * 64 + 256 * k) * 8);
        }
    };
    f32x4 acc[9][ND][NB];
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int d = 0; d < ND; ++d)
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[t][d][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    // operand addresses (bf16 elements of a stage): lane i of a group reads pixel i / 4, channels 4 (i % 4)
    const int r0 = wave * RW, pi = lr >> 2, pc = (lr & 3) * 4;
    const int a_d = T::XNP * 8 + (r0 * kWgW + 8 * lk + pi) * CO + pc;
    const int a_x = ((UP ? r0 / 2 : (S2 ? 2 * r0 : r0)) * XC + (UP ? 4 : (S2 ? 16 : 8)) * lk + (S2 ? 2 : 1) * pi) * CI + pc;
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    auto tr = [&](const uint16_t* p) __attribute__((always_inline)) -> uint2 {
        return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                             (__attribute__((address_space(3))) s16x4*)p));
    };
    constexpr int NXR = UP ? RW / 2 + 2 : (S2 ? 2 * RW + 1 : RW + 2);   // staged rows the wave's outputs read
    constexpr int NR = UP ? 2 : (S2 ? 5 : 3);                           // reads per staged row and 16 channels
    constexpr int P = (S2 ? 2 : 1) * CI;                                // elements between a lane's pixels
    uint2 rd[RW][ND][2], rx[NXR][NB][NR];
    auto read = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int rs = 0; rs < RW; ++rs)
#pragma unroll
            for (int d = 0; d < ND; ++d)
#pragma unroll
                for (int m = 0; m < 2; ++m) rd[rs][d][m] = tr(smem + a_d + (rs * kWgW + 4 * m) * CO + d * 16);
#pragma unroll
        for (int xr = 0; xr < NXR; ++xr)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const uint16_t* p = smem + a_x + xr * XC * CI + b * 16;
#pragma unroll
                for (int m = 0; m < NR; ++m) rx[xr][b][m] = tr(m < 3 ? p + 4 * m * P : p + CI + 4 * (m - 3) * P);
            }
    };
    auto multiply = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int xr = 0; xr < NXR; ++xr)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const uint2 u = rx[xr][b][0], v = rx[xr][b][1];
                u32x4 sh[3];
                if constexpr (UP) {
                    // stored columns a(-1) .. a4 of the lane's fine columns 0 .. 7 (a0 a0 a1 a1 a2 a2 a3 a3)
                    const uint32_t m = __builtin_amdgcn_alignbyte(u.y, u.x, 2u), q = __builtin_amdgcn_alignbyte(v.x, u.y, 2u);
                    sh[0] = u32x4{u.x, m, u.y, q};
                    sh[1] = u32x4{__builtin_amdgcn_perm(u.x, u.x, 0x07060706u), __builtin_amdgcn_perm(u.y, u.y, 0x05040504u),
                                  __builtin_amdgcn_perm(u.y, u.y, 0x07060706u), __builtin_amdgcn_perm(v.x, v.x, 0x05040504u)};
                    sh[2] = u32x4{m, u.y, q, v.x};
                } else {
                    const uint2 w = rx[xr][b][2];
                    const u32x4 sft = {__builtin_amdgcn_alignbyte(u.y, u.x, 2u), __builtin_amdgcn_alignbyte(v.x, u.y, 2u),
                                       __builtin_amdgcn_alignbyte(v.y, v.x, 2u), __builtin_amdgcn_alignbyte(w.x, v.y, 2u)};
                    sh[0] = u32x4{u.x, u.y, v.x, v.y};
                    if constexpr (S2) {
                        sh[1] = u32x4{rx[xr][b][3].x, rx[xr][b][3].y, rx[xr][b][4].x, rx[xr][b][4].y};
                        sh[2] = sft;
                    } else {
                        sh[1] = sft;
                        sh[2] = u32x4{u.y, v.x, v.y, w.x};
                    }
                }
#pragma unroll
                for (int dc = 0; dc < 3; ++dc)
#pragma unroll
                    for (int rs = 0; rs < RW; ++rs)
#pragma unroll
                        for (int dr = 0; dr < 3; ++dr) {
                            // staged row (from the wave's first) of output row rs, tap row dr
                            const int row = UP ? (rs + dr + 1) / 2 : (S2 ? 2 * rs + dr : rs + dr);
                            if (row != xr) continue;
#pragma unroll
                            for (int d = 0; d < ND; ++d) {
                                const u32x4 fa = {rd[rs][d][0].x, rd[rs][d][0].y, rd[rs][d][1].x, rd[rs][d][1].y};
                                acc[3 * dr + dc][d][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                    __builtin_bit_cast(bf16x8, fa), __builtin_bit_cast(bf16x8, sh[dc]),
                                    acc[3 * dr + dc][d][b], 0, 0, 0);
                            }
                        }
            }
    };
    // A stage is read after every wave's own DMA has landed (vmcnt) and the barrier; a wave takes its operands
    // of the whole tile into registers, so after the next barrier the next tile is fetched into the same stage
    // while this one is multiplied.  (With a second stage instead, the compiler waits for the fetch in flight
    // before the first LDS read.)  The empty asm statements keep LDS accesses on their side of the barriers
    auto barrier = [&]() __attribute__((always_inline)) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    if (blockIdx.x < total) issue(blockIdx.x);
    for (uint32_t t = blockIdx.x; t < total; t += gridDim.x) {
        __builtin_amdgcn_s_waitcnt(kWaitVm0);
        barrier();
        read();
        __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
        barrier();
        if (t + gridDim.x < total) issue(t + gridDim.x);
        multiply();
    }
    // sums of the four waves, in wave order: RC of the NA accumulator quads at a time pass through LDS, a
    // quad as 16 bytes per lane (no bank conflicts); lane (lr, lk), element q is co = 16 d + 4 lk + q,
    // ci = 16 b + lr.  The blocks with this blockIdx.x (one per channel-group pair) fill partial blockIdx.x
    // of the whole dW
    constexpr int RC = (int)(sizeof(smem) / 4096) < NA ? (int)(sizeof(smem) / 4096) : NA;
    f32x4* red = reinterpret_cast<f32x4*>(smem);
    float* pb = part + (int64_t)blockIdx.x * ((int64_t)g.Co * 9 * g.C);
    const f32x4* fl = &acc[0][0][0];
#pragma unroll
    for (int c0 = 0; c0 < NA; c0 += RC) {
        __syncthreads();
#pragma unroll
        for (int j = 0; j < RC; ++j)
            if (c0 + j < NA) red[(wave * RC + j) * 64 + lane] = fl[c0 + j];
        __syncthreads();
        for (int j = wave; j < RC && c0 + j < NA; j += 4) {
            f32x4 v = red[j * 64 + lane];
#pragma unroll
            for (int w = 1; w < 4; ++w) v += red[(w * RC + j) * 64 + lane];
            const int id = c0 + j, b = id % NB, d = id / NB % ND, tap = id / (NB * ND);
            const int ci = b * 16 + lr;
            if (ci >= CI) continue;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                pb[((int64_t)(blockIdx.z * CO + d * 16 + 4 * lk + q) * 9 + tap) * g.C + blockIdx.y * CI + ci] = v[q];
        }
    }
}

// Backward of the 1x1 map p = W x (W: KC x C, bf16) feeding the depth
// integral and of the skip sum next to it, from the gradient gs [pixel][ld]
// whose first C channels belong to u + x (u: a conv's output): the gradient at
// x, g[pixel][c] = gs[pixel][c] + sum_k dp[pixel][k] W[k][c] (FP32 sum over
// k), u's masked gradient dpre = bf16(gs [u > 0]), the per-block partials of
// dW[k][c] = sum over pixels of dp[pixel][k] x[pixel][c] and, in bias_part,
// of dpre's column sums.  Four threads share a pixel, each
// owning C / 4 channels, so a thread keeps KC x C / 4 accumulators; the
// pixels are dealt out in a fixed order and reduced in a fixed order.
// Bound by memory: gs copied to g, g read and written again and gs read a
// third time for dpre, 2097152 pixels took 119 (with the integral) + 60 + 60 us, now 65 + 103.
constexpr int kProjBlocks = 1024;
template <int KC, int C>
__global__ __launch_bounds__(256) void k_proj_bwd(const uint16_t* __restrict__ dp, const uint16_t* __restrict__ x,
                                                  const uint16_t* __restrict__ w, const float* __restrict__ gs, int ld,
                                                  const uint16_t* __restrict__ u, float* __restrict__ g,
                                                  uint16_t* __restrict__ dpre, int64_t P, float* __restrict__ part,
                                                  float* __restrict__ bias_part)
{
    constexpr int CQ = C / 4;
    static_assert(C == 16 && KC == 8, "four 4-channel groups per thread quad; 8 map channels");
    __shared__ float red[4][KC * C], redb[4][C];
    float bsum[CQ] = {0.f, 0.f, 0.f, 0.f};
    const int q = threadIdx.x & 3, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    float wr[KC][CQ], acc[KC][CQ];
#pragma unroll
    for (int k = 0; k < KC; ++k)
#pragma unroll
        for (int j = 0; j < CQ; ++j) {
            wr[k][j] = bf2f(w[k * C + q * CQ + j]);
            acc[k][j] = 0.f;
        }
    const int64_t stride = (int64_t)gridDim.x * 64;
    for (int64_t p = (int64_t)blockIdx.x * 64 + (threadIdx.x >> 2); p < P; p += stride) {
        const u32x4 dv = *reinterpret_cast<const u32x4*>(dp + p * KC);
        float d[KC];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            d[2 * j] = __uint_as_float(dv[j] << 16);
            d[2 * j + 1] = __uint_as_float(dv[j] & 0xFFFF0000u);
        }
        float xs[CQ];
        const uint16_t* xp = x + p * C + q * CQ;
#pragma unroll
        for (int j = 0; j < CQ; j += 4) {
            const uint2 v = *reinterpret_cast<const uint2*>(xp + j);
            xs[j] = __uint_as_float(v.x << 16);
            xs[j + 1] = __uint_as_float(v.x & 0xFFFF0000u);
            xs[j + 2] = __uint_as_float(v.y << 16);
            xs[j + 3] = __uint_as_float(v.y & 0xFFFF0000u);
        }
        const float4 gv = *reinterpret_cast<const float4*>(gs + p * ld + q * CQ);
        const uint2 uv = *reinterpret_cast<const uint2*>(u + p * C + q * CQ);
        const float gsv[CQ] = {gv.x, gv.y, gv.z, gv.w};
        const float us[CQ] = {__uint_as_float(uv.x << 16), __uint_as_float(uv.x & 0xFFFF0000u),
                              __uint_as_float(uv.y << 16), __uint_as_float(uv.y & 0xFFFF0000u)};
        float go[CQ];
        uint32_t b[CQ];
#pragma unroll
        for (int e = 0; e < CQ; ++e) {
            float t = 0.f;
#pragma unroll
            for (int k = 0; k < KC; ++k) t = fmaf(d[k], wr[k][e], t);
            go[e] = gsv[e] + t;
            b[e] = f2bf(us[e] > 0.f ? gsv[e] : 0.f);
            bsum[e] += bf2f((uint16_t)b[e]);
        }
        *reinterpret_cast<float4*>(g + p * C + q * CQ) = make_float4(go[0], go[1], go[2], go[3]);
        *reinterpret_cast<uint2*>(dpre + p * C + q * CQ) = make_uint2(b[0] | (b[1] << 16), b[2] | (b[3] << 16));
#pragma unroll
        for (int k = 0; k < KC; ++k)
#pragma unroll
            for (int j = 0; j < CQ; ++j) acc[k][j] = fmaf(d[k], xs[j], acc[k][j]);
    }
    // the 16 threads of a wave with the same channel group, then the four waves
#pragma unroll
    for (int k = 0; k < KC; ++k)
#pragma unroll
        for (int j = 0; j < CQ; ++j) {
            float v = acc[k][j];
#pragma unroll
            for (int m = 4; m < 64; m <<= 1) v += __shfl_xor(v, m);
            if (lane < 4) red[wave][k * C + q * CQ + j] = v;
        }
#pragma unroll
    for (int j = 0; j < CQ; ++j) {
        float v = bsum[j];
#pragma unroll
        for (int m = 4; m < 64; m <<= 1) v += __shfl_xor(v, m);
        if (lane < 4) redb[wave][q * CQ + j] = v;
    }
    __syncthreads();
    if (threadIdx.x < C)
        bias_part[(int64_t)blockIdx.x * C + threadIdx.x] =
            ((redb[0][threadIdx.x] + redb[1][threadIdx.x]) + redb[2][threadIdx.x]) + redb[3][threadIdx.x];
    for (int i = threadIdx.x; i < KC * C; i += 256)
        part[(int64_t)blockIdx.x * (KC * C) + i] = ((red[0][i] + red[1][i]) + red[2][i]) + red[3][i];
}

// ---------------------------------------------------------------------------
// element-wise / reduction kernels

__global__ void k_to_bf16(const float* x, uint16_t* out, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        out[i] = f2bf(x[i]);
}

// Frames replaced after an audit: frame pairs[k].y of out (and, unless null, of its bf16 copy) becomes frame
// pairs[k].x of src, for every k in one launch (blockIdx.x = k).  Bound by the copy's
// memory traffic; launched frame by frame, 256 of 1024 frames of 128 x 256 added 1.75 ms to an inference, now 0.10
__global__ __launch_bounds__(256) void k_replace_frames(const float* __restrict__ src, const int2* __restrict__ pairs,
                                                        int64_t frame, float* __restrict__ out,
                                                        uint16_t* __restrict__ out_bf16)
{
    const int2 p = pairs[blockIdx.x];
    const float* a = src + p.x * frame;
    const int64_t o = p.y * frame;
    for (int64_t i = (int64_t)blockIdx.y * 256 + threadIdx.x; i < frame; i += (int64_t)gridDim.y * 256) {
        const float v = a[i];
        out[o + i] = v;
        if (out_bf16) out_bf16[o + i] = f2bf(v);
    }
}

// Masked output gradient and bias-gradient partials in one pass over a
// [rows][C] matrix: out = bf16(g * [y > 0]) (y may be null: no mask; out may
// be null: g is already bf16 in gb), part[block][c] = sum of the block's rows
// of out.  Thread t owns column t % C for every (256 / C)-th row; the threads
// of a column are summed in a fixed order (deterministic).
__global__ __launch_bounds__(256) void k_mask_colsum(const float* g, int ldg, const uint16_t* gb, const uint16_t* y,
                                                     uint16_t* out, int64_t rows, int C, int64_t rows_per_block,
                                                     float* part, float slope)
{
    // a thread owns one 8-channel chunk of rows r_off, r_off + RP, ... (C multiple of 8, <= 256)
    __shared__ float red[256 * 8];
    const int C8 = C / 8;
    const int RP = 256 / C8;
    const int c8 = threadIdx.x % C8;
    const int r_off = threadIdx.x / C8;
    const int64_t r0 = (int64_t)blockIdx.x * rows_per_block;
    const int64_t r1 = min(rows, r0 + rows_per_block);
    float sum[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) sum[j] = 0.f;
    if (r_off < RP) {
        // kMaskRows rows per thread at a time, all their loads issued before their stores (a load
        // issued after a store waits for it); the sums take the rows in order
        constexpr int kMaskRows = 4;
        for (int64_t rb = r0 + r_off; rb < r1; rb += kMaskRows * RP) {
            u32x4 b[kMaskRows];
            if (gb) {
#pragma unroll
                for (int k = 0; k < kMaskRows; ++k) {
                    const int64_t r = rb + k * RP;
                    b[k] = r < r1 ? *reinterpret_cast<const u32x4*>(gb + r * C + c8 * 8) : u32x4{0u, 0u, 0u, 0u};
                }
            } else {
                float4 g0[kMaskRows], g1[kMaskRows];
                u32x4 yv[kMaskRows];
#pragma unroll
                for (int k = 0; k < kMaskRows; ++k) {
                    const int64_t r = rb + k * RP;
                    yv[k] = u32x4{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};   // no mask: bf16 1.0
                    g0[k] = g1[k] = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (r < r1) {
                        g0[k] = *reinterpret_cast<const float4*>(g + r * ldg + c8 * 8);
                        g1[k] = *reinterpret_cast<const float4*>(g + r * ldg + c8 * 8 + 4);
                        if (y) yv[k] = *reinterpret_cast<const u32x4*>(y + r * C + c8 * 8);
                    }
                }
#pragma unroll
                for (int k = 0; k < kMaskRows; ++k) {
                    const float gv[8] = {g0[k].x, g0[k].y, g0[k].z, g0[k].w, g1[k].x, g1[k].y, g1[k].z, g1[k].w};
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float ylo = __uint_as_float(yv[k][j] << 16), yhi = __uint_as_float(yv[k][j] & 0xFFFF0000u);
                        const uint16_t lo = f2bf(ylo > 0.f ? gv[2 * j] : (slope != 0.f ? slope * gv[2 * j] : 0.f));
                        const uint16_t hi =
                            f2bf(yhi > 0.f ? gv[2 * j + 1] : (slope != 0.f ? slope * gv[2 * j + 1] : 0.f));
                        b[k][j] = (uint32_t)lo | ((uint32_t)hi << 16);
                    }
                }
#pragma unroll
                for (int k = 0; k < kMaskRows; ++k) {
                    const int64_t r = rb + k * RP;
                    if (out && r < r1) *reinterpret_cast<u32x4*>(out + r * C + c8 * 8) = b[k];
                }
            }
#pragma unroll
            for (int k = 0; k < kMaskRows; ++k) {
                if (rb + k * RP >= r1) break;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    sum[2 * j] += __uint_as_float(b[k][j] << 16);
                    sum[2 * j + 1] += __uint_as_float(b[k][j] & 0xFFFF0000u);
                }
            }
        }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) red[threadIdx.x * 8 + j] = sum[j];
    __syncthreads();
    if ((int)threadIdx.x < C) {
        const int k8 = threadIdx.x / 8, j = threadIdx.x % 8;
        float t = 0.f;
        for (int q = 0; q < RP; ++q) t += red[(q * C8 + k8) * 8 + j];
        part[(int64_t)blockIdx.x * C + threadIdx.x] = t;
    }
}

// out[i] = sum_s part[s][i] in fixed order
// Depth integral along the beam.  A block owns 32 neighbouring columns (in
// frame-major order) and splits their rows into 8 segments, one thread per
// (segment, column): each thread first sums its segment, the segment totals
// meet in LDS, and a second pass over the segment writes the running sums
// from the totals of the segments above (below, for the backward).  A wave
// covers 32 columns of two segments, so each row access is contiguous.
// Eight channels per pixel (kScanC).
constexpr int kScanC = 8;
constexpr int kScanCols = 32, kScanSeg = 8;
constexpr int kScanRows = 4;   // rows whose loads are issued together

// the 1x1 map p = b + w e of one pixel (e: 16 bf16 channels as two 16-byte chunks); w, b in LDS
__device__ __forceinline__ void depth_map(const u32x4& a0, const u32x4& a1, const float* wf, const float* bf,
                                          float* p)
{
    asm volatile("" ::: "memory");   // weights stay in LDS (broadcast reads), not in registers
    float xc[16];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        xc[2 * j] = __uint_as_float(a0[j] << 16);
        xc[2 * j + 1] = __uint_as_float(a0[j] & 0xFFFF0000u);
        xc[8 + 2 * j] = __uint_as_float(a1[j] << 16);
        xc[8 + 2 * j + 1] = __uint_as_float(a1[j] & 0xFFFF0000u);
    }
#pragma unroll
    for (int k = 0; k < kScanC; ++k) {
        float acc = bf[k];
#pragma unroll
        for (int c = 0; c < 16; ++c) acc = fmaf(wf[k * 16 + c], xc[c], acc);
        p[k] = acc;
    }
}

// out[n][y][x][c_off + k] = bf16(scale * sum_{v < y} p_k(n, v, x)) with the
// 1x1 map p_k = b[k] + sum_c w[k][c] e[n][v][x][c] of the bf16 tensor e
// [N][H][W][16] (w bf16 [8][16], b FP32), evaluated in FP32 per pixel.
__global__ __launch_bounds__(256) void k_depth_map_scan_fwd(const uint16_t* __restrict__ e,
                                                            const uint16_t* __restrict__ w,
                                                            const float* __restrict__ b, uint16_t* __restrict__ out,
                                                            int N, int H, int W, float scale, int ld, int c_off)
{
    __shared__ float sw[kScanC * 16];
    __shared__ float sb[kScanC];
    __shared__ float tot[kScanSeg][kScanC][kScanCols + 1];
    if (threadIdx.x < kScanC * 16) sw[threadIdx.x] = bf2f(w[threadIdx.x]);
    if (threadIdx.x < kScanC) sb[threadIdx.x] = b[threadIdx.x];
    __syncthreads();
    const int c = threadIdx.x % kScanCols, sg = threadIdx.x / kScanCols;
    const int64_t col = (int64_t)blockIdx.x * kScanCols + c;
    const bool live = col < (int64_t)N * W;
    const int64_t n = live ? col / W : 0;
    const int x = live ? (int)(col - n * W) : 0;
    const int seg = (H + kScanSeg - 1) / kScanSeg;
    const int ya = live ? min(sg * seg, H) : 0, yb = live ? min(ya + seg, H) : 0;
    const float* wf = sw;
    const float* bf = sb;
    float sum[kScanC], p[kScanC];
#pragma unroll
    for (int k = 0; k < kScanC; ++k) sum[k] = 0.f;
    const uint16_t* ec = e + (n * H * W + x) * 16;   // column base; row stride W * 16
    for (int y0 = ya; y0 < yb; y0 += kScanRows) {
        u32x4 a0[kScanRows], a1[kScanRows];
#pragma unroll
        for (int q = 0; q < kScanRows; ++q) {
            const int64_t o = (int64_t)min(y0 + q, yb - 1) * W * 16;
            a0[q] = *reinterpret_cast<const u32x4*>(ec + o);
            a1[q] = *reinterpret_cast<const u32x4*>(ec + o + 8);
        }
#pragma unroll
        for (int q = 0; q < kScanRows; ++q) {
            if (y0 + q >= yb) break;
            depth_map(a0[q], a1[q], wf, bf, p);
#pragma unroll
            for (int k = 0; k < kScanC; ++k) sum[k] += p[k];
        }
    }
#pragma unroll
    for (int k = 0; k < kScanC; ++k) tot[sg][k][c] = sum[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kScanC; ++k) {
        float o = 0.f;
        for (int q = 0; q < sg; ++q) o += tot[q][k][c];
        sum[k] = o;   // running sum over the rows above this segment
    }
    uint16_t* oc = out + (n * H * W + x) * ld + c_off;
    for (int y0 = ya; y0 < yb; y0 += kScanRows) {
        u32x4 a0[kScanRows], a1[kScanRows];
#pragma unroll
        for (int q = 0; q < kScanRows; ++q) {
            const int64_t o = (int64_t)min(y0 + q, yb - 1) * W * 16;
            a0[q] = *reinterpret_cast<const u32x4*>(ec + o);
            a1[q] = *reinterpret_cast<const u32x4*>(ec + o + 8);
        }
#pragma unroll
        for (int q = 0; q < kScanRows; ++q) {
            const int y = y0 + q;
            if (y >= yb) break;
            u32x4 ov;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                ov[j] = (uint32_t)f2bf(scale * sum[2 * j]) | ((uint32_t)f2bf(scale * sum[2 * j + 1]) << 16);
            *reinterpret_cast<u32x4*>(oc + (int64_t)y * W * ld) = ov;
            depth_map(a0[q], a1[q], wf, bf, p);
#pragma unroll
            for (int k = 0; k < kScanC; ++k) sum[k] += p[k];
        }
    }
}

// k_depth_map_scan_fwd for columns of at most kScan1Seg * kScan1Rows rows, reading e once: a block
// owns kScan1Cols neighbouring columns split into kScan1Seg segments of at most kScan1Rows rows, one
// thread per (segment, column), which keeps its rows' maps p in registers between the segment sum
// and the running sums (the two-pass kernel reads e again for those).
constexpr int kScan1Cols = 8, kScan1Seg = 32, kScan1Rows = 8;
__global__ __launch_bounds__(256) void k_depth_map_scan_fwd1(const uint16_t* __restrict__ e,
                                                             const uint16_t* __restrict__ w,
                                                             const float* __restrict__ b, uint16_t* __restrict__ out,
                                                             int N, int H, int W, float scale, int ld, int c_off)
{
    static_assert(kScan1Cols * kScan1Seg == 256, "one thread per (segment, column)");
    __shared__ float sw[kScanC * 16];
    __shared__ float sb[kScanC];
    __shared__ float tot[kScan1Seg][kScanC][kScan1Cols + 1];
    if (threadIdx.x < kScanC * 16) sw[threadIdx.x] = bf2f(w[threadIdx.x]);
    if (threadIdx.x < kScanC) sb[threadIdx.x] = b[threadIdx.x];
    __syncthreads();
    const int c = threadIdx.x % kScan1Cols, sg = threadIdx.x / kScan1Cols;
    const int64_t col = (int64_t)blockIdx.x * kScan1Cols + c;
    const bool live = col < (int64_t)N * W;
    const int64_t n = live ? col / W : 0;
    const int x = live ? (int)(col - n * W) : 0;
    const int seg = (H + kScan1Seg - 1) / kScan1Seg;   // <= kScan1Rows (host check)
    const int ya = live ? min(sg * seg, H) : 0, yb = live ? min(ya + seg, H) : 0;
    const uint16_t* ec = e + (n * H * W + x) * 16;   // column base; row stride W * 16
    u32x4 a0[kScan1Rows], a1[kScan1Rows];
#pragma unroll
    for (int q = 0; q < kScan1Rows; ++q) {   // every row's loads before any use
        const int64_t o = (int64_t)min(ya + q, max(yb - 1, 0)) * W * 16;
        a0[q] = *reinterpret_cast<const u32x4*>(ec + o);
        a1[q] = *reinterpret_cast<const u32x4*>(ec + o + 8);
    }
    float pr[kScan1Rows][kScanC], sum[kScanC];
#pragma unroll
    for (int k = 0; k < kScanC; ++k) sum[k] = 0.f;
#pragma unroll
    for (int q = 0; q < kScan1Rows; ++q) {
        depth_map(a0[q], a1[q], sw, sb, pr[q]);
        if (ya + q < yb) {
#pragma unroll
            for (int k = 0; k < kScanC; ++k) sum[k] += pr[q][k];
        }
    }
#pragma unroll
    for (int k = 0; k < kScanC; ++k) tot[sg][k][c] = sum[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kScanC; ++k) {
        float o = 0.f;
        for (int q = 0; q < sg; ++q) o += tot[q][k][c];
        sum[k] = o;   // running sum over the rows above this segment
    }
    uint16_t* oc = out + (n * H * W + x) * ld + c_off;
#pragma unroll
    for (int q = 0; q < kScan1Rows; ++q) {
        const int y = ya + q;
        if (y >= yb) break;
        u32x4 ov;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            ov[j] = (uint32_t)f2bf(scale * sum[2 * j]) | ((uint32_t)f2bf(scale * sum[2 * j + 1]) << 16);
        *reinterpret_cast<u32x4*>(oc + (int64_t)y * W * ld) = ov;
#pragma unroll
        for (int k = 0; k < kScanC; ++k) sum[k] += pr[q][k];
    }
}

// Backward of k_depth_map_scan_fwd after the 1x1 map, through a tensor g
// [pixel][ld] (FP32) whose channels [c_off, c_off + 8) are the integral's
// gradient:  dp[n][v][x][k] = bf16(scale * sum_{y > v} g[n][y][x][c_off + k])
// and per-block column sums of the bf16 dp (bias gradient partials) in
// part[block][8].
__global__ __launch_bounds__(256) void k_depth_scan_bwd(const float* __restrict__ g, int ld, int c_off,
                                                        uint16_t* __restrict__ dp, float* __restrict__ part, int N,
                                                        int H, int W, float scale)
{
    __shared__ float tot[kScanSeg][kScanC][kScanCols + 1];
    __shared__ float red[kScanC][256];
    const int c = threadIdx.x % kScanCols, sg = threadIdx.x / kScanCols;
    const int64_t col = (int64_t)blockIdx.x * kScanCols + c;
    const bool live = col < (int64_t)N * W;
    const int64_t n = live ? col / W : 0;
    const int x = live ? (int)(col - n * W) : 0;
    const int seg = (H + kScanSeg - 1) / kScanSeg;
    const int ya = live ? min(sg * seg, H) : 0, yb = live ? min(ya + seg, H) : 0;
    const int64_t pc = n * H * W + x;   // column's pixel index at row 0; row stride W
    float sum[kScanC], bsum[kScanC];
#pragma unroll
    for (int k = 0; k < kScanC; ++k) {
        sum[k] = 0.f;
        bsum[k] = 0.f;
    }
    for (int y0 = ya; y0 < yb; y0 += kScanRows) {
        float4 ga[kScanRows][2];
#pragma unroll
        for (int q = 0; q < kScanRows; ++q) {
            const int64_t px = pc + (int64_t)min(y0 + q, yb - 1) * W;
            ga[q][0] = *reinterpret_cast<const float4*>(g + px * ld + c_off);
            ga[q][1] = *reinterpret_cast<const float4*>(g + px * ld + c_off + 4);
        }
#pragma unroll
        for (int q = 0; q < kScanRows; ++q) {
            if (y0 + q >= yb) break;
            sum[0] += ga[q][0].x; sum[1] += ga[q][0].y; sum[2] += ga[q][0].z; sum[3] += ga[q][0].w;
            sum[4] += ga[q][1].x; sum[5] += ga[q][1].y; sum[6] += ga[q][1].z; sum[7] += ga[q][1].w;
        }
    }
#pragma unroll
    for (int k = 0; k < kScanC; ++k) tot[sg][k][c] = sum[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kScanC; ++k) {
        float o = 0.f;
        for (int q = kScanSeg - 1; q > sg; --q) o += tot[q][k][c];
        sum[k] = o;   // running sum over the rows below this segment
    }
    for (int y0 = yb - 1; y0 >= ya; y0 -= kScanRows) {
        float4 ga[kScanRows][2];
#pragma unroll
        for (int q = 0; q < kScanRows; ++q) {
            const int64_t px = pc + (int64_t)max(y0 - q, ya) * W;
            ga[q][0] = *reinterpret_cast<const float4*>(g + px * ld + c_off);
            ga[q][1] = *reinterpret_cast<const float4*>(g + px * ld + c_off + 4);
        }
#pragma unroll
        for (int q = 0; q < kScanRows; ++q) {
            const int y = y0 - q;
            if (y < ya) break;
            const int64_t px = pc + (int64_t)y * W;
            u32x4 o;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint16_t lo = f2bf(scale * sum[2 * j]), hi = f2bf(scale * sum[2 * j + 1]);
                bsum[2 * j] += bf2f(lo);
                bsum[2 * j + 1] += bf2f(hi);
                o[j] = (uint32_t)lo | ((uint32_t)hi << 16);
            }
            *reinterpret_cast<u32x4*>(dp + px * kScanC) = o;
            sum[0] += ga[q][0].x; sum[1] += ga[q][0].y; sum[2] += ga[q][0].z; sum[3] += ga[q][0].w;
            sum[4] += ga[q][1].x; sum[5] += ga[q][1].y; sum[6] += ga[q][1].z; sum[7] += ga[q][1].w;
        }
    }
#pragma unroll
    for (int k = 0; k < kScanC; ++k) red[k][threadIdx.x] = bsum[k];
    __syncthreads();
    if (threadIdx.x < kScanC) {   // fixed order over the block's threads
        float t = 0.f;
        for (int i = 0; i < 256; ++i) t += red[threadIdx.x][i];
        part[(int64_t)blockIdx.x * kScanC + threadIdx.x] = t;
    }
}

// out[i] = sum over z of part[z][i]; one thread per output, rows in order
// (for many outputs and few rows)
__global__ void k_sum_parts(const float* part, int64_t n, int splits, float* out)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        float s = 0.f;
        int z = 0;
        for (; z + 8 <= splits; z += 8) {   // eight loads in flight, added in order
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = part[(int64_t)(z + j) * n + i];
#pragma unroll
            for (int j = 0; j < 8; ++j) s += v[j];
        }
        for (; z < splits; ++z) s += part[(int64_t)z * n + i];
        out[i] = s;
    }
}

// the same sum for few outputs and many rows: thread (ty, tx) of a block sums
// rows ty, ty + G, ... of output blockIdx.x * ob + tx (G = 256 / ob), then
// the G partial sums are added in order (fixed order, deterministic)
__global__ __launch_bounds__(256) void k_sum_parts_grouped(const float* part, int64_t n, int splits, float* out,
                                                           int ob)
{
    __shared__ float red[256];
    const int tx = threadIdx.x % ob, ty = threadIdx.x / ob;
    const int G = 256 / ob;
    const int64_t i = (int64_t)blockIdx.x * ob + tx;
    float s = 0.f;
    if (i < n) {
        int z = ty;
        for (; z + 7 * G < splits; z += 8 * G) {   // eight loads in flight, added in order
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = part[(int64_t)(z + j * G) * n + i];
#pragma unroll
            for (int j = 0; j < 8; ++j) s += v[j];
        }
        for (; z < splits; z += G) s += part[(int64_t)z * n + i];
    }
    red[threadIdx.x] = s;
    __syncthreads();
    if (ty == 0 && i < n) {
        float t = 0.f;
        for (int j = 0; j < G; ++j) t += red[j * ob + tx];
        out[i] = t;
    }
}

// Several reductions of per-block partials in one launch: block b computes output i of the segment
// holding it, out[out_off + i] = sum over z < splits of part[part_off + z n + i], added as
// k_sum_parts_grouped adds one output (thread t sums z = t, t + 256, ... in order, then the 256
// thread sums in order), so the results equal separate reduce_parts calls
__global__ __launch_bounds__(256) void k_reduce_segments(const float* __restrict__ part, float* __restrict__ out,
                                                         ReduceSegs t)
{
    __shared__ float red[256];
    int k = 0;
    while (k + 1 < t.count && t.s[k + 1].first <= (int)blockIdx.x) ++k;
    const ReduceSeg sg = t.s[k];
    const int64_t i = (int64_t)blockIdx.x - sg.first;
    const float* p = part + sg.part_off + i;
    float v = 0.f;
    for (int z = threadIdx.x; z < sg.splits; z += 256) v += p[(int64_t)z * sg.n];
    red[threadIdx.x] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        float a = 0.f;
        for (int j = 0; j < 256; ++j) a += red[j];
        out[sg.out_off + i] = a;
    }
}

// head backward (C = 16): dx[p][c] = w[c] g[p] (FP32), the layer's masked gradient dpre = bf16(dx [x > 0]), and
// per-block partials of dw[c] = sum_p x[p][c] g[p] (c < 16), db = sum_p g[p] (entry 16) and, in bias_part, of the
// column sums of dpre.  Bound by memory (132 bytes a pixel: g, x, dx and dpre; 3.8 TB/s); dpre in a pass of
// its own (k_mask_colsum), 2097152 pixels took 54 + 55 us, now 73.
__global__ __launch_bounds__(256) void k_head_bwd(const uint16_t* __restrict__ x, const uint16_t* __restrict__ w,
                                                  const float* __restrict__ g, float* __restrict__ dx,
                                                  uint16_t* __restrict__ dpre, int64_t P, int64_t rows_per_block,
                                                  float* __restrict__ part, float* __restrict__ bias_part)
{
    constexpr int NR = 33;   // dw, db, column sums of dpre
    __shared__ float red[NR][257];   // (a row more than the threads: the sums below read NR different banks)
    float wf[16], acc[NR];
#pragma unroll
    for (int c = 0; c < 16; ++c) wf[c] = bf2f(w[c]);
#pragma unroll
    for (int c = 0; c < NR; ++c) acc[c] = 0.f;
    const int64_t p0 = (int64_t)blockIdx.x * rows_per_block;
    const int64_t p1 = min(P, p0 + rows_per_block);
    for (int64_t p = p0 + threadIdx.x; p < p1; p += blockDim.x) {
        const float gp = g[p];
        const u32x4 v[2] = {*reinterpret_cast<const u32x4*>(x + p * 16), *reinterpret_cast<const u32x4*>(x + p * 16 + 8)};
        u32x4 o[2];
        float d[16];
#pragma unroll
        for (int c = 0; c < 16; c += 2) {
            const uint32_t u = v[c / 8][c % 8 / 2];
            const float xl = __uint_as_float(u << 16), xh = __uint_as_float(u & 0xFFFF0000u);
            acc[c] += xl * gp;
            acc[c + 1] += xh * gp;
            d[c] = wf[c] * gp;
            d[c + 1] = wf[c + 1] * gp;
            const uint32_t b = (uint32_t)f2bf(xl > 0.f ? d[c] : 0.f) | ((uint32_t)f2bf(xh > 0.f ? d[c + 1] : 0.f) << 16);
            o[c / 8][c % 8 / 2] = b;
            acc[17 + c] += __uint_as_float(b << 16);
            acc[18 + c] += __uint_as_float(b & 0xFFFF0000u);
        }
        acc[16] += gp;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<float4*>(dx + p * 16 + 4 * q) = make_float4(d[4 * q], d[4 * q + 1], d[4 * q + 2], d[4 * q + 3]);
        *reinterpret_cast<u32x4*>(dpre + p * 16) = o[0];
        *reinterpret_cast<u32x4*>(dpre + p * 16 + 8) = o[1];
    }
#pragma unroll
    for (int c = 0; c < NR; ++c) red[c][threadIdx.x] = acc[c];
    __syncthreads();
    if (threadIdx.x < NR) {
        float t = 0.f;
        for (int j = 0; j < 256; ++j) t += red[threadIdx.x][j];
        if (threadIdx.x < 17) part[(int64_t)blockIdx.x * 17 + threadIdx.x] = t;
        else bias_part[(int64_t)blockIdx.x * 16 + threadIdx.x - 17] = t;
    }
}

// Discriminator input of two sets of P pixels: z[i] = (x[p] channels 0..3,
// bf16(img), 0, 0, 0) with img = y_real[p] for i = p < P and y_fake[p] for
// i = P + p (the same encoded input x[p] in both sets)
__global__ void k_disc_input(const uint16_t* x, const float* y_real, const float* y_fake, uint16_t* z, int64_t P)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < 2 * P; i += (int64_t)gridDim.x * blockDim.x) {
        const bool fake = i >= P;
        const int64_t p = fake ? i - P : i;
        const uint2 xv = *reinterpret_cast<const uint2*>(x + p * 8);
        const float img = fake ? y_fake[p] : y_real[p];
        uint4 o;
        o.x = xv.x;
        o.y = xv.y;
        o.z = (uint32_t)f2bf(img);
        o.w = 0u;
        *reinterpret_cast<uint4*>(z + i * 8) = o;
    }
}

// Binary cross-entropy on the logits l = logits[r * ld] of rows r < P_total:
// rows r < P_real have label 1 (loss w_real softplus(-l), gradient
// gscale w_real (sigmoid(l) - 1)), the rest label 0 (w_fake softplus(l),
// gscale w_fake sigmoid(l)).  grad rows hold ld floats (channel 0 the
// gradient, the others 0); part[block] = the block's loss sum.
__device__ __forceinline__ float softplus_f(float a) { return fmaxf(a, 0.f) + log1pf(expf(-fabsf(a))); }

__global__ __launch_bounds__(256) void k_bce_logits(const float* logits, int ld, int64_t P_real, int64_t P_total,
                                                    float w_real, float w_fake, float gscale, float* grad,
                                                    int64_t per_block, float* part)
{
    __shared__ float red[256];
    const int64_t r0 = (int64_t)blockIdx.x * per_block;
    const int64_t r1 = min(P_total, r0 + per_block);
    float acc = 0.f;
    for (int64_t r = r0 + threadIdx.x; r < r1; r += blockDim.x) {
        const float l = logits[r * ld];
        const float e = expf(-fabsf(l));
        const float sig = l >= 0.f ? 1.f / (1.f + e) : e / (1.f + e);
        const bool real = r < P_real;
        const float w = real ? w_real : w_fake;
        acc += w * softplus_f(real ? -l : l);
        grad[r * ld] = gscale * w * (real ? sig - 1.f : sig);
        for (int c = 1; c < ld; ++c) grad[r * ld + c] = 0.f;
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// gy[p] += dz[p * ld + c]
__global__ void k_add_channel(float* gy, const float* dz, int ld, int c, int64_t P)
{
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < P; p += (int64_t)gridDim.x * blockDim.x)
        gy[p] += dz[p * ld + c];
}

// L1 loss: per-block partial sums of |yhat - y| * scale (scale = 1 / n);
// grad = sign(yhat - y) * scale
__global__ void k_l1(const float* yhat, const float* y, int64_t n, float scale, float* grad, int64_t per_block,
                     float* part)
{
    __shared__ float red[256];
    const int64_t i0 = (int64_t)blockIdx.x * per_block;
    const int64_t i1 = min(n, i0 + per_block);
    float s = 0.f;
    for (int64_t i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
        const float d = yhat[i] - y[i];
        s += fabsf(d);
        grad[i] = d > 0.f ? scale : (d < 0.f ? -scale : 0.f);
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0] * scale;   // mean over all n
}

// Adam on FP32 masters; writes the bf16 weights [Co][K] and their transpose
// WT [Ci][taps][Co] (data gradient operand)
// Adam's per-step scalars on the device, so a captured step reads them at
// replay: steps[0] (and steps[1], the discriminator's, when disc) count the
// updates; coef = {lr, 1 - b1^t, 1 - b2^t, 1 - b1^td, 1 - b2^td}
__global__ void k_adam_coef(int64_t* steps, float* coef, float lr, float b1, float b2, int disc)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    const int64_t t = steps[0] + 1;
    steps[0] = t;
    coef[0] = lr;
    coef[1] = 1.f - powf(b1, (float)t);
    coef[2] = 1.f - powf(b2, (float)t);
    if (disc) {
        const int64_t td = steps[1] + 1;
        steps[1] = td;
        coef[3] = 1.f - powf(b1, (float)td);
        coef[4] = 1.f - powf(b2, (float)td);
    }
}

// Adam over a parameter vector made of segments (one launch for all of a
// network's tensors): block b works on kAdamChunk elements of the segment
// whose block0 <= b; a weight segment also refreshes its bf16 copy.  One with
// a transpose (the [Ci][taps][Co] copy of the data gradient) is dealt out in
// tiles of 32 output x 32 input channels of one tap, so that the transpose is
// written in runs of 64 bytes: written element by element, each in a line of
// its own that blocks on several XCDs share, 1.8 million parameters took 47 us,
// now 15.
constexpr int kAdamChunk = 2048, kAdamTile = 32;
__global__ __launch_bounds__(256) void k_adam_multi(const AdamSeg* __restrict__ segs, int nseg, float* w, float* m,
                                                    float* v, const float* __restrict__ g, uint16_t* wb, uint16_t* wt,
                                                    const float* __restrict__ coef, int ci, float b1, float b2,
                                                    float eps)
{
    __shared__ int s_seg;
    __shared__ uint16_t tile[kAdamTile][kAdamTile + 1];
    for (int k = threadIdx.x; k < nseg; k += 256)   // (one thread walking the table waited for each entry)
        if (segs[k].block0 <= (int)blockIdx.x && (k + 1 == nseg || segs[k + 1].block0 > (int)blockIdx.x)) s_seg = k;
    __syncthreads();
    const AdamSeg sg = segs[s_seg];
    const float lr = coef[0], c1 = coef[ci], c2 = coef[ci + 1];
    auto update = [&](int64_t i) __attribute__((always_inline)) -> float {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.f - b1) * gi;
        const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        const float wi = w[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
        w[i] = wi;
        return wi;
    };
    const uint32_t b = (uint32_t)blockIdx.x - (uint32_t)sg.block0;
    if (!sg.transpose) {
        const int64_t base = (int64_t)b * kAdamChunk;
        const int64_t end = min(base + (int64_t)kAdamChunk, sg.n);
        for (int64_t j = base + threadIdx.x; j < end; j += 256) {
            const float wi = update(sg.off + j);
            if (sg.bf16) wb[sg.off + j] = f2bf(wi);
        }
        return;
    }
    // element (co, t, ci) at (co * taps + t) * Ci + ci, transposed at (ci * taps + t) * Co + co
    const uint32_t nci = ((uint32_t)sg.Ci + kAdamTile - 1) / kAdamTile, q = b / nci, tc = q / (uint32_t)sg.taps;
    const int ci0 = (int)(b - q * nci) * kAdamTile, t = (int)(q - tc * (uint32_t)sg.taps), co0 = (int)tc * kAdamTile;
    for (int e = threadIdx.x; e < kAdamTile * kAdamTile; e += 256) {
        const int r = e / kAdamTile, c = e % kAdamTile;
        if (co0 + r >= sg.Co || ci0 + c >= sg.Ci) continue;
        const int64_t i = sg.off + ((int64_t)(co0 + r) * sg.taps + t) * sg.Ci + ci0 + c;
        const uint16_t bb = f2bf(update(i));
        wb[i] = bb;
        tile[r][c] = bb;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < kAdamTile * kAdamTile; e += 256) {
        const int c = e / kAdamTile, r = e % kAdamTile;
        if (co0 + r >= sg.Co || ci0 + c >= sg.Ci) continue;
        wt[sg.off + ((int64_t)(ci0 + c) * sg.taps + t) * sg.Co + co0 + r] = tile[r][c];
    }
}

// the step's losses into a ring of R steps: hist[(t - 1) mod R] = loss[0..2], t = steps[0]
__global__ void k_loss_log(const float* loss, const int64_t* steps, float* hist, int R)
{
    if (threadIdx.x < 3 && blockIdx.x == 0) {
        const int64_t slot = (steps[0] - 1) % R;
        hist[slot * 3 + threadIdx.x] = loss[threadIdx.x];
    }
}

// bf16 copies of FP32 weights and the transpose (initialisation / load)
__global__ void k_weights_to_bf16(const float* w, int64_t n, uint16_t* wb, uint16_t* wt, int Co, int taps, int Ci)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const uint16_t b = f2bf(w[i]);
        wb[i] = b;
        if (wt) {
            const int ci = (int)(i % Ci);
            const int64_t q = i / Ci;
            const int t = (int)(q % taps);
            const int co = (int)(q / taps);
            wt[((int64_t)ci * taps + t) * Co + co] = b;
        }
    }
}

// wt[ci][t][co] = w[co][t][ci] (bf16)
__global__ void k_transpose_w(const uint16_t* w, uint16_t* wt, int Co, int taps, int Ci)
{
    const int64_t n = (int64_t)Co * taps * Ci;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int ci = (int)(i % Ci);
        const int64_t q = i / Ci;
        const int t = (int)(q % taps);
        const int co = (int)(q / taps);
        wt[((int64_t)ci * taps + t) * Co + co] = w[i];
    }
}

// PSNR of clamp(yhat frame idx[b], 0, 1) against target frame b (peak 1).  One block per frame, few of them: bound
// by the latency of its loads, so 1024 threads with four pixels each in flight (8 frames of 32768 pixels: with 256
// threads and one 54 us, now 9)
__global__ __launch_bounds__(1024) void k_psnr_idx(const float* __restrict__ yhat, const float* __restrict__ y,
                                                   const int32_t* __restrict__ idx, int64_t frame,
                                                   float* __restrict__ psnr)
{
    constexpr int NT = 1024, U = 4;
    __shared__ float red[NT];
    const float* a = yhat + (int64_t)idx[blockIdx.x] * frame;
    const float* b = y + (int64_t)blockIdx.x * frame;
    float s = 0.f;
    for (int64_t i0 = threadIdx.x; i0 < frame; i0 += U * NT) {
        float av[U], bv[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int64_t i = min(i0 + k * NT, frame - 1);
            av[k] = a[i];
            bv[k] = b[i];
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const float d = fminf(fmaxf(av[k], 0.f), 1.f) - bv[k];
            if (i0 + k * NT < frame) s += d * d;
        }
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int st = NT / 2; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const float mse = red[0] / (float)frame;
        psnr[blockIdx.x] = mse > 0.f ? -10.f * log10f(mse) : 200.f;
    }
}

int64_t grid_for(int64_t n, int64_t per = 256)
{
    int64_t b = (n + per - 1) / per;
    if (b > 8192) b = 8192;
    return b < 1 ? 1 : b;
}

// sum of `splits` rows of n partial results into out, in a fixed order
hipError_t reduce_parts(const float* part, int64_t n, int splits, float* out, hipStream_t s)
{
    if (splits <= 16 || n >= 65536) {
        hipLaunchKernelGGL(k_sum_parts, dim3((unsigned)grid_for(n)), dim3(256), 0, s, part, n, splits, out);
        return hipGetLastError();
    }
    int ob = 64;   // outputs per block; fewer when that leaves under 256 blocks
    while (ob > 1 && (n + ob - 1) / ob < 256) ob >>= 1;
    hipLaunchKernelGGL(k_sum_parts_grouped, dim3((unsigned)((n + ob - 1) / ob)), dim3(256), 0, s, part, n, splits,
                       out, ob);
    return hipGetLastError();
}

template <int MODE, int BM, int BN, int WM, int WN>
hipError_t launch_gemm(const ConvGeom& g, const ConvArgs& a, int splits, hipStream_t s)
{
    const int64_t gm = (g.M + BM - 1) / BM;
    const int gn = (g.N + BN - 1) / BN;
    hipLaunchKernelGGL((k_conv_gemm<MODE, BM, BN, WM, WN>), dim3((unsigned)gm, gn, splits), dim3(kThreads), 0, s,
                       g, a);
    return hipGetLastError();
}

}  // namespace

// ---------------------------------------------------------------------------

bool conv_tile_supported(const ConvGeom& g)
{
    const bool shape = g.kh == 3 && g.kw == 3 && g.stride == 1 && g.pad == 1 && (g.Co == 16 || g.Co == 32) &&
                       g.Ho == (g.up ? 2 * g.H : g.H) && g.Wo == (g.up ? 2 * g.W : g.W);
    // 64 input channels only upsampled, where the staged tile is the 10 x 18 stored one
    return shape && (g.C == 8 || g.C == 16 || g.C == 24 || g.C == 32 || (g.C == 64 && g.up && g.Co == 32));
}

template <int C, int CO, bool UP, bool DIL = false>
hipError_t launch_tile(const ConvGeom& g, const ConvArgs& a, hipStream_t s)
{
    constexpr int TH = kTileH;
    const int64_t blocks = conv_tile_blocks(g.Kw / ((int64_t)g.Ho * g.Wo), g.Ho, g.Wo);   // Kw = N * Ho * Wo
    if (blocks > 0x7FFFFFFFll) return hipErrorInvalidValue;
    if (a.out_f32 && a.add) {   // data gradients added to something (never upsampled)
        if constexpr (UP) return hipErrorInvalidValue;
        else hipLaunchKernelGGL((k_conv3x3_tile<C, CO, false, DIL, true, TH>), dim3((unsigned)blocks), dim3(32 * TH), 0, s,
                                g, a);
    } else {
        hipLaunchKernelGGL((k_conv3x3_tile<C, CO, UP, DIL, false, TH>), dim3((unsigned)blocks), dim3(32 * TH), 0, s, g, a);
    }
    return hipGetLastError();
}

template <int CO>
hipError_t launch_tile_co(const ConvGeom& g, const ConvArgs& a, hipStream_t s)
{
    if (g.up) {
        switch (g.C) {
        case 8: return launch_tile<8, CO, true>(g, a, s);
        case 16: return launch_tile<16, CO, true>(g, a, s);
        case 24: return launch_tile<24, CO, true>(g, a, s);
        case 32: return launch_tile<32, CO, true>(g, a, s);
        default:
            if constexpr (CO == 32) return launch_tile<64, 32, true>(g, a, s);
            return hipErrorInvalidValue;
        }
    }
    switch (g.C) {
    case 8: return launch_tile<8, CO, false>(g, a, s);
    case 16: return launch_tile<16, CO, false>(g, a, s);
    case 24: return launch_tile<24, CO, false>(g, a, s);
    default: return launch_tile<32, CO, false>(g, a, s);
    }
}

hipError_t conv_pair(int C, int up, int CM, int EX, int CO, const PairArgs& a, hipStream_t s)
{
    const int64_t blocks = (int64_t)a.N * ((a.H + 15) / 16) * ((a.W + 31) / 32);
    if (blocks < 1 || blocks > 0x7FFFFFFFll || !a.out == !a.head_out || (up && (a.H % 2 || a.W % 2)))
        return hipErrorInvalidValue;
    const dim3 gr((unsigned)blocks), bl(512);
    if (C == 8 && !up && CM == 16 && EX == 0 && CO == 16)
        hipLaunchKernelGGL((k_conv3x3_pair<8, false, 16, 0, 16>), gr, bl, 0, s, a);
    else if (C == 32 && up && CM == 16 && EX == 8 && CO == 16)
        hipLaunchKernelGGL((k_conv3x3_pair<32, true, 16, 8, 16>), gr, bl, 0, s, a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

bool dgrad_tile_supported(const ConvGeom& g)
{
    const int Hin = g.up ? 2 * g.H : g.H, Win = g.up ? 2 * g.W : g.W;
    const bool geom = g.kh == 3 && g.kw == 3 && g.pad == 1 &&
                      ((g.stride == 1 && g.Ho == Hin && g.Wo == Win) ||
                       (g.stride == 2 && !g.up && Hin == 2 * g.Ho && Win == 2 * g.Wo));
    // the forward tile conv's channels: dy's Co in, the layer's C out
    return geom && (g.Co == 8 || g.Co == 16 || g.Co == 24 || g.Co == 32) && (g.C == 16 || g.C == 32);
}

namespace {
template <int CO, bool DIL>
hipError_t launch_dgrad_tile(const ConvGeom& f, const ConvArgs& a, hipStream_t s)
{
    switch (f.C) {
    case 8: return launch_tile<8, CO, false, DIL>(f, a, s);
    case 16: return launch_tile<16, CO, false, DIL>(f, a, s);
    case 24: return launch_tile<24, CO, false, DIL>(f, a, s);
    default: return launch_tile<32, CO, false, DIL>(f, a, s);
    }
}
}  // namespace

int64_t conv_tile_blocks(int64_t N, int H, int W)
{
    return N * ((H + kTileH - 1) / kTileH) * ((W + kTileW - 1) / kTileW);
}

hipError_t dgrad_tile(const ConvGeom& g, const uint16_t* dy, const uint16_t* wt, float* dx, const float* add,
                      const DpreArgs& m, hipStream_t s)
{
    if (!dgrad_tile_supported(g)) return hipErrorInvalidValue;
    const int Hin = g.up ? 2 * g.H : g.H, Win = g.up ? 2 * g.W : g.W;
    ConvGeom f = g;   // forward conv: dy (Ho x Wo, Co channels) -> dx (Hin x Win, C channels)
    f.C = g.Co;
    f.Co = g.C;
    f.H = g.Ho;
    f.W = g.Wo;
    f.Ho = Hin;
    f.Wo = Win;
    f.stride = 1;
    f.up = 0;
    f.Kw = (g.Kw / ((int64_t)g.Ho * g.Wo)) * Hin * Win;   // N * Hin * Win
    ConvArgs a;
    std::memset(&a, 0, sizeof(a));
    a.a = dy;
    a.b = wt;
    a.flip = 1;
    a.out_f32 = dx;
    a.add = add;
    a.mask = m.mask;
    a.dpre = m.dpre;
    a.colsum = m.colsum;
    a.pool2 = g.up;   // an upsampled layer's gradient at its stored input resolution
    const bool dil = g.stride == 2;
    if (f.Co == 16) return dil ? launch_dgrad_tile<16, true>(f, a, s) : launch_dgrad_tile<16, false>(f, a, s);
    return dil ? launch_dgrad_tile<32, true>(f, a, s) : launch_dgrad_tile<32, false>(f, a, s);
}

bool dgrad_parity_supported(const ConvGeom& g)
{
    return g.kh == 3 && g.kw == 3 && g.stride == 2 && g.pad == 1 && !g.up && g.Co % 8 == 0 && g.C % 8 == 0 &&
           g.H >= 2 && g.W >= 2;
}

hipError_t dgrad_parity(const ConvGeom& g, const uint16_t* dy, const uint16_t* wt, float* dx, const float* add,
                        hipStream_t s)
{
    if (!dgrad_parity_supported(g)) return hipErrorInvalidValue;
    if (g.H < 2 || g.W < 2) return hipErrorInvalidValue;   // every class has pixels
    // one launch: class blockIdx.z; the grid covers class 0's rows, the largest class
    const int64_t N = g.Kw / ((int64_t)g.Ho * g.Wo);
    ConvGeom c = g;
    c.par = 4;
    for (int par = 0; par < 4; ++par) {
        c.hc4[par] = (g.H - (par >> 1) + 1) / 2;
        c.wc4[par] = (g.W - (par & 1) + 1) / 2;
        c.f_hw4[par] = make_fastdiv((uint32_t)(c.hc4[par] * c.wc4[par]));
        c.f_w4[par] = make_fastdiv((uint32_t)c.wc4[par]);
    }
    c.M = N * c.hc4[0] * c.wc4[0];
    c.K = 4 * g.Co;   // the largest class's (for the launch shape only)
    c.kb = 9 * g.Co;
    ConvArgs a;
    std::memset(&a, 0, sizeof(a));
    a.a = dy;
    a.b = wt;
    a.out_f32 = dx;
    a.add = add;
    return conv_gemm(kDgrad, c, a, 1, s);
}

namespace {
// the halo kernel's layers: g is the forward conv (of dy as data gradient)
bool halo_supported(const ConvGeom& g, bool dgrad)
{
    const bool shape = g.kh == 3 && g.kw == 3 && g.stride == 1 && g.pad == 1 && g.Co % kHaloN == 0 &&
                       g.Ho == (g.up ? 2 * g.H : g.H) && g.Wo == (g.up ? 2 * g.W : g.W);
    if (!shape || g.Wo < kHaloT || g.Ho < kHaloT || !(g.C == 64 || g.C == 128 || (g.C == 256 && g.up))) return false;
    if (dgrad && (g.Ho % kHaloT || g.Wo % kHaloT)) return false;
    return halo_pays(dgrad, g.C, g.Co, g.up != 0, g.Kw / ((int64_t)g.Ho * g.Wo), g.Ho, g.Wo);   // Kw = N * Ho * Wo
}

template <int MODE, bool UP>
hipError_t launch_halo(const ConvGeom& g, const ConvArgs& a, hipStream_t s)
{
    const int64_t blocks = halo_blocks(g.Co, g.Kw / ((int64_t)g.Ho * g.Wo), g.Ho, g.Wo);
    if (blocks > 0x7FFFFFFFll) return hipErrorInvalidValue;
    const dim3 gr((unsigned)blocks), bl(kHaloThreads);
    if (g.C == 64) hipLaunchKernelGGL((k_conv3x3_halo<MODE, 64, UP>), gr, bl, 0, s, g, a);
    else if (g.C == 128) hipLaunchKernelGGL((k_conv3x3_halo<MODE, 128, UP>), gr, bl, 0, s, g, a);
    else {
        if constexpr (UP) hipLaunchKernelGGL((k_conv3x3_halo<MODE, 256, UP>), gr, bl, 0, s, g, a);
        else return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
}  // namespace

hipError_t conv_gemm(int mode, const ConvGeom& g, const ConvArgs& a, int splits, hipStream_t s)
{
    if (a.head_out && (mode != kFwd || !conv_tile_supported(g) || g.Co != 16 || !a.head_w || !a.head_b))
        return hipErrorInvalidValue;
    if (a.extra && (mode != kFwd || !conv_tile_supported(g) || !a.out2_bf16 || a.extra_c < 8 || a.extra_c % 8 ||
                    g.Co + a.extra_c > a.ld_out2))
        return hipErrorInvalidValue;
    if (a.dpre) return hipErrorInvalidValue;   // (the tiled data gradient's only)
    if (mode == kFwd && conv_tile_supported(g))
        return g.Co == 16 ? launch_tile_co<16>(g, a, s) : launch_tile_co<32>(g, a, s);
    if (mode == kFwd && halo_supported(g, false))
        return g.up ? launch_halo<kFwd, true>(g, a, s) : launch_halo<kFwd, false>(g, a, s);
    if (mode == kDgrad && g.stride == 1 && g.kh == 3 && g.kw == 3 && g.pad == 1) {
        ConvGeom f = g;   // the forward conv of dy
        f.C = g.Co;
        f.Co = g.C;
        f.H = g.Ho;
        f.W = g.Wo;
        f.Ho = g.up ? 2 * g.H : g.H;
        f.Wo = g.up ? 2 * g.W : g.W;
        f.up = 0;
        f.Kw = (g.Kw / ((int64_t)g.Ho * g.Wo)) * f.Ho * f.Wo;
        if (halo_supported(f, true)) {
            ConvArgs d = a;
            d.pool2 = g.up;
            return launch_halo<kDgrad, false>(f, d, s);
        }
    }
    if (mode == kWgrad) {
        if (g.M <= 16) return launch_gemm<kWgrad, 16, 128, 1, 4>(g, a, splits, s);
        if (g.M <= 32) return launch_gemm<kWgrad, 32, 128, 1, 4>(g, a, splits, s);
        return launch_gemm<kWgrad, 64, 128, 2, 2>(g, a, splits, s);
    }
    // data gradient: four parity classes (g.par == 4), one per grid z
    const int nz = mode == kDgrad && g.par == 4 ? 4 : 1;
    const GemmTile t = gemm_tile(g.M, g.N, nz);
    if (mode == kFwd) {
        if (t.bn == 16)
            return t.bm == 256 ? launch_gemm<kFwd, 256, 16, 4, 1>(g, a, 1, s) : launch_gemm<kFwd, 64, 16, 4, 1>(g, a, 1, s);
        if (t.bn == 32)
            return t.bm == 128 ? launch_gemm<kFwd, 128, 32, 4, 1>(g, a, 1, s) : launch_gemm<kFwd, 64, 32, 4, 1>(g, a, 1, s);
        if (t.bn == 128) return launch_gemm<kFwd, 128, 128, 2, 2>(g, a, 1, s);
        if (t.bm == 128) return launch_gemm<kFwd, 128, 64, 2, 2>(g, a, 1, s);
        if (t.bm == 64) return launch_gemm<kFwd, 64, 64, 1, 4>(g, a, 1, s);
        return launch_gemm<kFwd, 32, 64, 1, 4>(g, a, 1, s);
    }
    if (t.bn == 16)
        return t.bm == 256 ? launch_gemm<kDgrad, 256, 16, 4, 1>(g, a, nz, s) : launch_gemm<kDgrad, 64, 16, 4, 1>(g, a, nz, s);
    if (t.bn == 32)
        return t.bm == 128 ? launch_gemm<kDgrad, 128, 32, 4, 1>(g, a, nz, s) : launch_gemm<kDgrad, 64, 32, 4, 1>(g, a, nz, s);
    if (t.bn == 128) return launch_gemm<kDgrad, 128, 128, 2, 2>(g, a, nz, s);
    if (t.bm == 128) return launch_gemm<kDgrad, 128, 64, 2, 2>(g, a, nz, s);
    if (t.bm == 64) return launch_gemm<kDgrad, 64, 64, 2, 2>(g, a, nz, s);
    return launch_gemm<kDgrad, 32, 64, 1, 4>(g, a, nz, s);
}

bool wgrad_tile_plan(const ConvGeom& g, WgradTilePlan* plan)
{
    const bool s1 = g.stride == 1 && g.Ho == (g.up ? 2 * g.H : g.H) && g.Wo == (g.up ? 2 * g.W : g.W);
    const bool s2 = g.stride == 2 && !g.up && g.Ho == (g.H - 1) / 2 + 1 && g.Wo == (g.W - 1) / 2 + 1;
    if (!(g.kh == 3 && g.kw == 3 && g.pad == 1 && (s1 || s2))) return false;
    int ci_g = 0, co_g = 0;
    if (s2 && (g.C == 24 || g.C == 32 || (g.C % 32 == 0 && g.Wo >= 16)))
        ci_g = g.C == 24 ? 8 : 16;   // (the staged halo of 32 channels needs more registers than there are)
    else if (g.C == 8 || g.C == 16 || g.C == 24 || g.C == 32)
        ci_g = g.C;
    else if (g.C % 32 == 0 && g.Wo >= 16)   // wider layers in groups of 32 (tiles at least half full)
        ci_g = 32;
    if (g.Co == 16 || g.Co == 32)
        co_g = g.Co;
    else if (g.Co % 32 == 0 && g.Wo >= 16)
        co_g = 32;
    if (!ci_g || !co_g) return false;
    if (plan) {
        const int gy = g.C / ci_g, gz = g.Co / co_g;
        const int th = g.stride == 2 ? kWgH2 : kWgH;
        const int64_t tiles = (g.Kw / ((int64_t)g.Ho * g.Wo)) * (int64_t)((g.Ho + th - 1) / th) *
                              ((g.Wo + kWgW - 1) / kWgW);
        const int64_t fill = 256 * wgrad_blocks_per_cu(ci_g, co_g, g.stride == 1 && !g.up);   // every block resident at once
        const int64_t want = std::max<int64_t>(1, (fill + gy * gz - 1) / (gy * gz));
        plan->gx = (int)std::min<int64_t>(std::max<int64_t>(tiles, 1), want);
        plan->gy = gy;
        plan->gz = gz;
        plan->ci_g = ci_g;
        plan->co_g = co_g;
    }
    return true;
}

int64_t wgrad_tile_part_floats(const WgradTilePlan& p)
{
    return (int64_t)p.gx * p.gy * p.gz * p.co_g * 9 * p.ci_g;   // gx partials of the whole dW
}

namespace {
template <int CI, int CO>
hipError_t launch_wgrad_tile(const ConvGeom& g, const uint16_t* x, const uint16_t* dy, float* part,
                             const WgradTilePlan& p, hipStream_t s)
{
    const dim3 grid(p.gx, p.gy, p.gz);
    if (g.stride == 2) {
        if constexpr (CI > 16) return hipErrorInvalidValue;
        else hipLaunchKernelGGL((k_wgrad3x3_tile<CI, CO, false, true>), grid, dim3(256), 0, s, g, x, dy, part);
    } else if (g.up) {
        hipLaunchKernelGGL((k_wgrad3x3_tile<CI, CO, true, false>), grid, dim3(256), 0, s, g, x, dy, part);
    } else {
        hipLaunchKernelGGL((k_wgrad3x3_tile<CI, CO, false, false>), grid, dim3(256), 0, s, g, x, dy, part);
    }
    return hipGetLastError();
}

template <int CO>
hipError_t launch_wgrad_tile_co(const ConvGeom& g, const uint16_t* x, const uint16_t* dy, float* part,
                                const WgradTilePlan& p, hipStream_t s)
{
    switch (p.ci_g) {
    case 8: return launch_wgrad_tile<8, CO>(g, x, dy, part, p, s);
    case 16: return launch_wgrad_tile<16, CO>(g, x, dy, part, p, s);
    case 24: return launch_wgrad_tile<24, CO>(g, x, dy, part, p, s);
    case 32: return launch_wgrad_tile<32, CO>(g, x, dy, part, p, s);
    default: return hipErrorInvalidValue;
    }
}
}  // namespace

hipError_t wgrad_tile(const ConvGeom& g, const uint16_t* x, const uint16_t* dy, float* part, const WgradTilePlan& p,
                      float* dw, hipStream_t s)
{
    WgradTilePlan q;
    if (!wgrad_tile_plan(g, &q) || q.gx != p.gx || q.gy != p.gy || q.gz != p.gz || q.ci_g != p.ci_g ||
        q.co_g != p.co_g)
        return hipErrorInvalidValue;
    const hipError_t e = p.co_g == 16 ? launch_wgrad_tile_co<16>(g, x, dy, part, p, s)
                                      : launch_wgrad_tile_co<32>(g, x, dy, part, p, s);
    if (e != hipSuccess) return e;
    return reduce_parts(part, (int64_t)g.Co * 9 * g.C, p.gx, dw, s);
}

int wgrad_tile_m(int M) { return M <= 16 ? 16 : (M <= 32 ? 32 : 64); }

hipError_t mask_colsum(const float* g, int ldg, const uint16_t* y, uint16_t* out, int64_t rows, int C, float* part,
                       int blocks, float* bias_grad, hipStream_t s, float slope)
{
    if (C > 256 || C % 8 || (ldg != 0 && (ldg < C || ldg % 4))) return hipErrorInvalidValue;
    const int64_t per = (rows + blocks - 1) / blocks;
    hipLaunchKernelGGL(k_mask_colsum, dim3(blocks), dim3(256), 0, s, g, ldg ? ldg : C, nullptr, y, out, rows, C, per,
                       part, slope);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !bias_grad) return e;
    return reduce_parts(part, C, blocks, bias_grad, s);
}

hipError_t reduce_segments(const float* part, float* out, const ReduceSegs& t, hipStream_t s)
{
    if (t.count < 1 || t.count > kMaxReduceSegs) return hipErrorInvalidValue;
    const ReduceSeg& last = t.s[t.count - 1];
    hipLaunchKernelGGL(k_reduce_segments, dim3((unsigned)(last.first + last.n)), dim3(256), 0, s, part, out, t);
    return hipGetLastError();
}

int depth_scan_blocks(int N, int W)
{
    return (int)(((int64_t)N * W + kScanCols - 1) / kScanCols);
}

hipError_t depth_map_scan_fwd(const uint16_t* e, const uint16_t* w, const float* b, uint16_t* out, int N, int H,
                              int W, float scale, int ld, int c_off, hipStream_t s)
{
    if (ld % 8 || c_off % 8 || c_off + kScanC > ld) return hipErrorInvalidValue;
    if (H <= kScan1Seg * kScan1Rows) {   // one read of e
        const int64_t blocks = ((int64_t)N * W + kScan1Cols - 1) / kScan1Cols;
        hipLaunchKernelGGL(k_depth_map_scan_fwd1, dim3((unsigned)blocks), dim3(256), 0, s, e, w, b, out, N, H, W, scale,
                           ld, c_off);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_depth_map_scan_fwd, dim3((unsigned)depth_scan_blocks(N, W)), dim3(256), 0, s, e, w, b, out, N,
                       H, W, scale, ld, c_off);
    return hipGetLastError();
}

hipError_t depth_scan_bwd(const float* g, int ld, int c_off, uint16_t* dp, float* part, float* bias_grad, int N,
                          int H, int W, float scale, hipStream_t s)
{
    if (ld % 4 || c_off % 4 || c_off + kScanC > ld) return hipErrorInvalidValue;
    const int blocks = depth_scan_blocks(N, W);
    hipLaunchKernelGGL(k_depth_scan_bwd, dim3((unsigned)blocks), dim3(256), 0, s, g, ld, c_off, dp, part, N, H, W,
                       scale);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return reduce_parts(part, kScanC, blocks, bias_grad, s);
}

hipError_t proj_bwd(const uint16_t* dp, const uint16_t* x, const uint16_t* w, const float* gs, int ld,
                    const uint16_t* u, float* g, uint16_t* dpre, int64_t P, int KC, int C, float* part,
                    float* bias_part, float* dw, hipStream_t s)
{
    if (KC != 8 || C != 16 || P < 1 || ld < C || ld % 4) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_proj_bwd<8, 16>), dim3(kProjBlocks), dim3(256), 0, s, dp, x, w, gs, ld, u, g, dpre, P, part,
                       bias_part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return reduce_parts(part, KC * C, kProjBlocks, dw, s);
}

int proj_bwd_blocks() { return kProjBlocks; }

hipError_t to_bf16(const float* x, uint16_t* out, int64_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_to_bf16, dim3((unsigned)grid_for(n)), dim3(256), 0, s, x, out, n);
    return hipGetLastError();
}

hipError_t replace_frames(const float* src, const int2* pairs, int n, int64_t frame, float* out, uint16_t* out_bf16,
                          hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const int64_t by = std::min<int64_t>(64, (frame + 1023) / 1024);   // about four pixels a thread
    hipLaunchKernelGGL(k_replace_frames, dim3((unsigned)n, (unsigned)by), dim3(256), 0, s, src, pairs, frame, out,
                       out_bf16);
    return hipGetLastError();
}

hipError_t colsum_bf16(const uint16_t* x, int64_t rows, int cols, float* part, int blocks, float* out,
                       hipStream_t s)
{
    if (cols > 256 || cols % 8) return hipErrorInvalidValue;
    const int64_t per = (rows + blocks - 1) / blocks;
    hipLaunchKernelGGL(k_mask_colsum, dim3(blocks), dim3(256), 0, s, nullptr, cols, x, nullptr, nullptr, rows, cols,
                       per, part, 0.f);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return reduce_parts(part, cols, blocks, out, s);
}

hipError_t sum_parts(const float* part, int64_t n, int splits, float* out, hipStream_t s)
{
    return reduce_parts(part, n, splits, out, s);
}

hipError_t head_bwd(const uint16_t* x, const uint16_t* w, const float* g, float* dx, uint16_t* dpre, int64_t P,
                    float* part, float* bias_part, int blocks, float* dwb, hipStream_t s)
{
    const int64_t per = (P + blocks - 1) / blocks;
    hipLaunchKernelGGL(k_head_bwd, dim3(blocks), dim3(256), 0, s, x, w, g, dx, dpre, P, per, part, bias_part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return reduce_parts(part, 17, blocks, dwb, s);
}

hipError_t l1_loss(const float* yhat, const float* y, int64_t n, float* grad, float* part, int blocks, float* loss,
                   hipStream_t s)
{
    const int64_t per = (n + blocks - 1) / blocks;
    hipLaunchKernelGGL(k_l1, dim3(blocks), dim3(256), 0, s, yhat, y, n, 1.f / (float)n, grad, per, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return reduce_parts(part, 1, blocks, loss, s);
}

hipError_t disc_input(const uint16_t* x, const float* y_real, const float* y_fake, uint16_t* z, int64_t P,
                      hipStream_t s)
{
    hipLaunchKernelGGL(k_disc_input, dim3((unsigned)grid_for(2 * P)), dim3(256), 0, s, x, y_real, y_fake, z, P);
    return hipGetLastError();
}

hipError_t bce_logits(const float* logits, int ld, int64_t P_real, int64_t P_total, float w_real, float w_fake,
                      float gscale, float* grad, float* part, int blocks, float* loss, hipStream_t s)
{
    const int64_t per = (P_total + blocks - 1) / blocks;
    hipLaunchKernelGGL(k_bce_logits, dim3(blocks), dim3(256), 0, s, logits, ld, P_real, P_total, w_real, w_fake,
                       gscale, grad, per, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return reduce_parts(part, 1, blocks, loss, s);
}

hipError_t add_channel(float* gy, const float* dz, int ld, int c, int64_t P, hipStream_t s)
{
    hipLaunchKernelGGL(k_add_channel, dim3((unsigned)grid_for(P)), dim3(256), 0, s, gy, dz, ld, c, P);
    return hipGetLastError();
}

int adam_blocks(const AdamSeg& a)
{
    if (!a.transpose) return (int)((a.n + kAdamChunk - 1) / kAdamChunk);
    return (a.Co + kAdamTile - 1) / kAdamTile * a.taps * ((a.Ci + kAdamTile - 1) / kAdamTile);
}

hipError_t adam_coef(int64_t* steps, float* coef, float lr, float b1, float b2, int disc, hipStream_t s)
{
    hipLaunchKernelGGL(k_adam_coef, dim3(1), dim3(64), 0, s, steps, coef, lr, b1, b2, disc);
    return hipGetLastError();
}

hipError_t adam_multi(const AdamSeg* segs, int nseg, int blocks, float* w, float* m, float* v, const float* g,
                      uint16_t* wb, uint16_t* wt, const float* coef, int ci, float b1, float b2, float eps,
                      hipStream_t s)
{
    if (nseg < 1 || blocks < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_adam_multi, dim3((unsigned)blocks), dim3(256), 0, s, segs, nseg, w, m, v, g, wb, wt, coef, ci,
                       b1, b2, eps);
    return hipGetLastError();
}

hipError_t loss_log(const float* loss, const int64_t* steps, float* hist, int R, hipStream_t s)
{
    hipLaunchKernelGGL(k_loss_log, dim3(1), dim3(64), 0, s, loss, steps, hist, R);
    return hipGetLastError();
}

hipError_t weights_to_bf16(const float* w, int64_t n, uint16_t* wb, uint16_t* wt, int Co, int taps, int Ci,
                           hipStream_t s)
{
    hipLaunchKernelGGL(k_weights_to_bf16, dim3((unsigned)grid_for(n)), dim3(256), 0, s, w, n, wb, wt, Co, taps, Ci);
    return hipGetLastError();
}

hipError_t transpose_w(const uint16_t* w, uint16_t* wt, int Co, int taps, int Ci, hipStream_t s)
{
    const int64_t n = (int64_t)Co * taps * Ci;
    hipLaunchKernelGGL(k_transpose_w, dim3((unsigned)grid_for(n)), dim3(256), 0, s, w, wt, Co, taps, Ci);
    return hipGetLastError();
}

hipError_t psnr_indexed(const float* yhat, const float* y, const int32_t* idx, int n_frames, int64_t frame,
                        float* psnr, hipStream_t s)
{
    if (n_frames <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_psnr_idx, dim3(n_frames), dim3(1024), 0, s, yhat, y, idx, frame, psnr);
    return hipGetLastError();
}

}  // namespace sg
