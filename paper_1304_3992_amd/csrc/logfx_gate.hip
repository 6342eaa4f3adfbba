// The smoothing gate: a small CNN that decides per image whether the hybrid
// median is applied.  The paper leaves that choice to the user, according
// to the noise in the extracted map (abstract; Sec. 4).
//
// Network: three 3x3 convolutions of stride 2 with zero padding
// (3 -> 16 -> 32 -> 32 channels, 128 -> 64 -> 32 -> 16), ReLU after each,
// global average pooling and a linear layer to one logit.  The convolutions
// run as implicit GEMMs on v_mfma_f32_16x16x16_bf16 with FP32 accumulation:
// forward, a workgroup stages its input rows and the weights in LDS;
// backward, a band of the layer's input and of its output gradient.  Stored activations and their
// gradients are bfloat16; biases, the head, the loss and AdamW are FP32.
// Every reduction has a fixed order (the workgroups' partial weight gradients are
// summed in a fixed order, no float atomics), so a training step is deterministic.
#include "logfx_gate.h"

namespace logfx {
namespace gate {
namespace {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short short8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ inline uint16_t to_bf16(float f) {
    // round to nearest, ties to even (finite values)
    const uint32_t u = __float_as_uint(f);
    return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}
__device__ inline float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// D += A B on one 16 x 16 x 16 block.  Operand layout of the instruction:
// lane l = 16 q + c holds A(c, 4q + i) and B(4q + i, c) for i = 0..3, and
// receives D(4q + i, c).
__device__ inline f32x4 mfma(const bf16x4 &a, const bf16x4 &b, const f32x4 &d) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, d, 0, 0, 0);
}

// The same on a 32-deep block: lane l = 16 q + c holds A(c, 8q + i) and
// B(8q + i, c) for i = 0..7.
__device__ inline f32x4 mfma32(const bf16x8 &a, const bf16x8 &b, const f32x4 &d) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, d, 0, 0, 0);
}

template <int CI, int CO, int HI>
struct Geo {
    static constexpr int HO = HI / 2, HWI = HI * HI, HWO = HO * HO;
    static constexpr int MB = CO / 16;
    static_assert(CO % 16 == 0 && HWO % 16 == 0, "layer shape");
};

// ---------------------------------------------------------------- forward
// out[b][co][p] = bf16(relu(bias[co] + sum_{ci,ky,kx} w[co][ci][ky][kx] in[b][ci][2oy+ky-1][2ox+kx-1]))
// for output pixel p = (oy, ox).  GEMM rows = co, columns = 16 pixels of one
// output row, reduction over k = (tap, ci), tap = 3 ky + kx, channels
// padded to a multiple of four (CI = 3 -> 4, with zero weights).
//
// A workgroup takes TH output rows of one image.  It first stages in LDS
// the 2 TH + 1 input rows they read, channel-innermost (one 8-byte slot per
// four channels of a pixel, column -1 and row -1 as the zero padding), and
// copies the layer's weights, kept in that [co][k] order beside the flat
// parameters, as they are; a lane's four reduction indices of a
// 16-deep block are then four consecutive channels at one tap, so each
// MFMA operand is one 8-byte LDS read.  Neighbouring lanes of an operand
// read pixels two apart (an odd number of slots per pixel) or weight rows
// 2 (mod 4) words apart, so the 32 lanes of a half-wave hit distinct banks.  Each of the four waves computes PW
// blocks of 16 pixels for all output channels.
template <int CI, int HI, int TH>
struct Stage {
    static constexpr int CIP = perm_cip(CI);            // padded channels
    static constexpr int G4 = CIP / 4;                  // four-channel groups per pixel
    static constexpr int P = G4 % 2 ? G4 : G4 + 1;      // 8-byte slots per pixel
    static constexpr int X = HI + 1;                    // columns -1 .. HI-1
    static constexpr int R = 2 * TH + 1;                // input rows of TH output rows
    static constexpr int KB = (9 * CIP + 15) / 16;      // 16-deep reduction blocks
    static constexpr int KROW = perm_row(CI);           // weight row: KB * 16 + 8
    static_assert(KROW == KB * 16 + 8, "weight row of the forward layout");
};

template <int CI, int CO, int HI, int TH>
__global__ __launch_bounds__(256) void conv_fwd(const uint16_t *__restrict__ in, const int *__restrict__ idx,
                                                const uint16_t *__restrict__ w, const float *__restrict__ bias,
                                                uint16_t *__restrict__ out, int B) {
    using G = Geo<CI, CO, HI>;
    using S = Stage<CI, HI, TH>;
    constexpr int HO = G::HO, BR = HO / 16, NB = TH * BR, PW = NB / 4, TILES = HO / TH;
    static_assert(HO % TH == 0 && NB % 4 == 0 && HI % 4 == 0, "tile shape");
    typedef uint32_t u32x2a2 __attribute__((ext_vector_type(2), aligned(2)));
    __shared__ uint2 xs[S::R * S::X * S::P];
    __shared__ __align__(16) uint16_t ws[CO * S::KROW];
    const int b = blockIdx.x / TILES, oy0 = (blockIdx.x % TILES) * TH;
    if (b >= B) return;   // uniform over the workgroup
    const int t = threadIdx.x;
    const uint16_t *ib = in + (long long)(idx ? idx[b] : b) * CI * G::HWI;

    // Input rows 2 oy0 - 1 .. 2 oy0 + 2 TH - 1: four pixels of four channels
    // per item, read as one 8-byte word per channel and written as four
    // slots; the weights in 16-byte chunks.  All reads are issued before
    // the first LDS write.
    constexpr int XQ = HI / 4, NI = S::R * S::G4 * XQ, UI = (NI + 255) / 256;
    constexpr int NW = CO * S::KROW / 8, UW = (NW + 255) / 256;
    static_assert((CO * S::KROW) % 8 == 0, "weights in 8-element chunks");
    uint32_t v[UI][4][2];
    uint4 wc[UW];
#pragma unroll
    for (int u = 0; u < UI; ++u) {
        const int it = t + 256 * u, xq = it % XQ, rg = it / XQ, g = rg % S::G4, r = rg / S::G4;
        const int iy = 2 * oy0 - 1 + r;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int ch = 4 * g + j;
            if (it < NI && ch < CI && iy >= 0) {
                const u32x2a2 x = *reinterpret_cast<const u32x2a2 *>(ib + ch * G::HWI + iy * HI + 4 * xq);
                v[u][j][0] = x.x;
                v[u][j][1] = x.y;
            } else {
                v[u][j][0] = v[u][j][1] = 0u;
            }
        }
    }
#pragma unroll
    for (int u = 0; u < UW; ++u) {
        const int it = t + 256 * u;
        wc[u] = it < NW ? reinterpret_cast<const uint4 *>(w)[it] : make_uint4(0u, 0u, 0u, 0u);
    }
#pragma unroll
    for (int u = 0; u < UI; ++u) {
        const int it = t + 256 * u, xq = it % XQ, rg = it / XQ, g = rg % S::G4, r = rg / S::G4;
        if (it >= NI) break;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int sh = 16 * (p & 1), wd = p >> 1;
            const uint32_t c0 = (v[u][0][wd] >> sh) & 0xFFFFu, c1 = (v[u][1][wd] >> sh) & 0xFFFFu;
            const uint32_t c2 = (v[u][2][wd] >> sh) & 0xFFFFu, c3 = (v[u][3][wd] >> sh) & 0xFFFFu;
            xs[(r * S::X + 4 * xq + p + 1) * S::P + g] = make_uint2(c0 | (c1 << 16), c2 | (c3 << 16));
        }
    }
    for (int it = t; it < S::R * S::G4; it += 256)
        xs[(it / S::G4) * S::X * S::P + it % S::G4] = make_uint2(0u, 0u);
#pragma unroll
    for (int u = 0; u < UW; ++u) {
        const int it = t + 256 * u;
        if (it < NW) reinterpret_cast<uint4 *>(ws)[it] = wc[u];
    }
    __syncthreads();

    const int wv = t >> 6, l = t & 63, q = l >> 4, c = l & 15;
    f32x4 acc[G::MB][PW];
#pragma unroll
    for (int mb = 0; mb < G::MB; ++mb)
#pragma unroll
        for (int j = 0; j < PW; ++j) acc[mb][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < S::KB; ++kb) {
        const int k0 = 16 * kb + 4 * q;   // the lane's four reduction indices: k0 .. k0 + 3
        const int tap = k0 / S::CIP, g = (k0 - tap * S::CIP) >> 2;
        const int tc = tap < 9 ? tap : 0, ky = tc / 3, kx = tc - 3 * ky;
        bf16x4 av[G::MB];
#pragma unroll
        for (int mb = 0; mb < G::MB; ++mb)
            av[mb] = *reinterpret_cast<const bf16x4 *>(ws + (mb * 16 + c) * S::KROW + k0);
#pragma unroll
        for (int j = 0; j < PW; ++j) {
            const int blk = wv * PW + j, row = blk / BR, ox = (blk % BR) * 16 + c;
            bf16x4 bv = *reinterpret_cast<const bf16x4 *>(xs + ((2 * row + ky) * S::X + 2 * ox + kx) * S::P + g);
            if (tap >= 9) bv = bf16x4{0, 0, 0, 0};
#pragma unroll
            for (int mb = 0; mb < G::MB; ++mb) acc[mb][j] = mfma(av[mb], bv, acc[mb][j]);
        }
    }
#pragma unroll
    for (int j = 0; j < PW; ++j) {
        const int blk = wv * PW + j;
        const int p = (oy0 + blk / BR) * HO + (blk % BR) * 16 + c;
#pragma unroll
        for (int mb = 0; mb < G::MB; ++mb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int co = mb * 16 + 4 * q + i;
                out[((long long)b * CO + co) * G::HWO + p] = to_bf16(fmaxf(acc[mb][j][i] + bias[co], 0.0f));
            }
    }
}

// gap[b][c] = mean of a3[b][c]; z[b] = sum_c gap[b][c] wf[c] + bf, and,
// where asked for, the decision z[b] > 0 as flags[b] / decisions[b].  Eight
// lanes per channel, 32 positions each; the lane sums are combined by a
// butterfly, so the order is fixed and every lane of the eight holds the
// same total.
__global__ __launch_bounds__(256) void head_fwd(const uint16_t *__restrict__ a3, const float *__restrict__ theta,
                                               float *__restrict__ gap, float *__restrict__ logits,
                                               int *__restrict__ flags, uint8_t *__restrict__ decisions) {
    constexpr int HW = kH3 * kH3;
    static_assert(kC3 * 8 == 256 && HW == 8 * 32, "eight lanes of 32 positions per channel");
    typedef uint32_t u32x4a2 __attribute__((ext_vector_type(4), aligned(2)));
    __shared__ float part[kC3];
    const int b = blockIdx.x, t = threadIdx.x, ch = t >> 3;
    const uint16_t *p = a3 + ((long long)b * kC3 + ch) * HW + (t & 7) * 32;
    float s = 0.0f;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const u32x4a2 u = *reinterpret_cast<const u32x4a2 *>(p + 8 * v);
#pragma unroll
        for (int e = 0; e < 4; ++e) s += __uint_as_float(u[e] << 16) + __uint_as_float(u[e] & 0xFFFF0000u);
    }
    s += __shfl_xor(s, 1);
    s += __shfl_xor(s, 2);
    s += __shfl_xor(s, 4);
    const float g = s / (float)HW;
    if ((t & 7) == 0) {
        gap[b * kC3 + ch] = g;
        part[ch] = g * theta[kOffWf + ch];
    }
    __syncthreads();
    if (t < 64) {
        float z = t < kC3 ? part[t] : 0.0f;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) z += __shfl_xor(z, off);
        if (t == 0) {
            z += theta[kOffBf];
            logits[b] = z;
            if (flags) flags[b] = z > 0.0f;
            if (decisions) decisions[b] = (uint8_t)(z > 0.0f);
        }
    }
}

// ---------------------------------------------------------------- backward
// d loss / d logit of batch row b: (sigmoid(z) - y) / B.
__device__ inline float dlogit(const NetBuffers &n, int b) {
    return (1.0f / (1.0f + expf(-n.logits[b])) - n.labels[n.idx ? n.idx[b] : b]) / (float)n.B;
}

// A band of the input of a stride-2 convolution in LDS, one plane per kernel
// column kx: plane (kx, ci) holds in[ci][2 oy0 - 1 + r][2 u + kx - 1] at
// r HO + u, r = 0 .. 2 TH.  The pixels that consecutive output columns u
// read through one tap are then consecutive, so eight of them are one
// 16-byte LDS read.  A plane takes an odd number of 16-byte units: lanes on
// neighbouring channels (or taps) read different banks.
template <int CI, int HI, int TH>
struct Planes {
    static constexpr int HO = HI / 2, R = 2 * TH + 1;
    static constexpr int STR = (R * HO / 8 + 1 - (R * HO / 8) % 2) * 8;   // elements per plane
    static constexpr int ELEMS = 3 * CI * STR;
    static_assert(HO % 8 == 0 && HI % 8 == 0, "whole 16-byte units");
    // Fills the planes from the image at `ib`: eight input pixels and the
    // one to their left per item, U items' loads in flight.
    static __device__ void fill(uint16_t *pl, const uint16_t *__restrict__ ib, int oy0, int t) {
        typedef uint32_t u32x4a2 __attribute__((ext_vector_type(4), aligned(2)));
        constexpr int XC = HI / 8, N = CI * R * XC, U = (N + 255) / 256 < 9 ? (N + 255) / 256 : 9;
        for (int i0 = t; i0 < N; i0 += 256 * U) {
            u32x4a2 v[U];
            uint32_t lf[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int it = i0 + 256 * k, xc = it % XC, rc = it / XC, r = rc % R, ci = rc / R;
                const int iy = 2 * oy0 - 1 + r;
                v[k] = u32x4a2{0u, 0u, 0u, 0u};
                lf[k] = 0u;
                if (it < N && iy >= 0) {
                    const uint16_t *p = ib + (long long)ci * HI * HI + iy * HI + 8 * xc;
                    v[k] = *reinterpret_cast<const u32x4a2 *>(p);
                    if (xc > 0) lf[k] = p[-1];
                }
            }
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int it = i0 + 256 * k, xc = it % XC, rc = it / XC, r = rc % R, ci = rc / R;
                if (it >= N) break;
                const uint32_t e0 = (v[k].x & 0xFFFFu) | (v[k].y << 16), e1 = (v[k].z & 0xFFFFu) | (v[k].w << 16);
                const uint32_t o0 = (v[k].x >> 16) | (v[k].y & 0xFFFF0000u), o1 = (v[k].z >> 16) | (v[k].w & 0xFFFF0000u);
                uint16_t *q = pl + ci * STR + r * HO + 4 * xc;
                *reinterpret_cast<uint2 *>(q) = make_uint2(lf[k] | (o0 << 16), (o0 >> 16) | (o1 << 16));
                *reinterpret_cast<uint2 *>(q + CI * STR) = make_uint2(e0, e1);
                *reinterpret_cast<uint2 *>(q + 2 * CI * STR) = make_uint2(o0, o1);
            }
        }
    }
};

// Partial sums of a layer's weight gradient, one set per workgroup:
// [co][tap][ci], then the biases [co].
template <int CI, int CO> constexpr int kGradSet = CO * (9 * CI + 1);

// Workgroups of a backward kernel: each walks items g, g + groups, ... and
// keeps its weight-gradient sums in registers, so that the partial sums the
// reduction reads stay at 29 MB however large the batch is.  512 workgroups
// are two per CU; at batch 256 they take 1 item each (layer 3) and 4 (layers
// 2 and 1).  Layer 2 took 32 us with 512, 38 with 768 (a last round of
// items on a third of them); bands of 8 rows there, one workgroup per CU, 52.
constexpr int kBwdGroups = 512;
constexpr int kBand3 = 8, kBand2 = 4, kBand1 = 8;   // output rows per item
constexpr int bwd_groups(int B, int ho, int th) { return B * (ho / th) < kBwdGroups ? B * (ho / th) : kBwdGroups; }

// Backward of one layer with 32 output channels: the weight and bias
// gradient, and the data gradient gin[b][ci][y][x] = bf16(sum_{co,ky,kx}
// w[co][ci][ky][kx] g[b][co][oy][ox]) where act[b][ci][y][x] > 0, over
// (oy, ox) with y = 2 oy + ky - 1, x = 2 ox + kx - 1.
//
// An item is a band of TH output rows of one sample.  Its gradient rows
// (and the row below, which the band's odd input rows read) and the band of
// the layer's input are staged in LDS once and serve both products:
//  * weight gradient: rows = co, columns = 16 input channels at one tap,
//    reduction over the band's output pixels, 32 per MFMA; both operands
//    are eight consecutive pixels, one 16-byte LDS read.  The tiles of
//    (tap, 16 channels) are dealt to the four waves.
//  * data gradient: the input pixels of one parity class (y mod 2, x mod 2)
//    read the same taps -- 1, 2, 2 and 4 of the nine -- so each class is a
//    dense product of 16 pixels x 32 output channels per tap: nine MFMAs
//    give 64 input pixels, and no product with a zero is formed.
// The gather form this replaces (2-byte global loads per operand element,
// the nine taps over all pixels) took 89 + 41 us (layer 3) and 209 + 105 us
// (layer 2) on 256 samples, this one 28 and 32 us; the bytes alone take 5
// and 13 us.  More loads in flight change nothing: the LDS traffic of the
// staging and the operands, two or three workgroups per CU, bounds it.
// HEAD: g is the last layer's gradient, bf16(dz wf[c] / 256) where a3 > 0,
// formed from the activations `g` while they are staged.
template <int CI, int HI, int TH, bool HEAD>
__global__ __launch_bounds__(256) void conv_bwd(NetBuffers n, const uint16_t *__restrict__ g,
                                                const uint16_t *__restrict__ act, const uint16_t *__restrict__ wd,
                                                uint16_t *__restrict__ gin, float *__restrict__ partial) {
    constexpr int CO = 32, HO = HI / 2, BANDS = HO / TH, PX = TH * HO;
    constexpr int MB = CI / 16, NT = 9 * MB, TPW = (NT + 1 + 3) / 4;   // column tiles (and the bias) per wave
    using PL = Planes<CI, HI, TH>;
    constexpr int GPS = PX + 8;        // pixel-innermost gradient rows: an odd number of 16-byte units
    constexpr int GCS = CO + 8;        // channel-innermost pixels: 5 units
    static_assert(PX % 32 == 0 && (PX / 8) % 2 == 0 && HO % 16 == 0 && (TH * HO / 16) % 4 == 0, "band shape");
    __shared__ __align__(16) uint16_t pl[PL::ELEMS];
    __shared__ __align__(16) uint16_t gp[CO * GPS];
    __shared__ __align__(16) uint16_t gc[(TH + 1) * (HO + 1) * GCS];
    const int t = threadIdx.x, l = t & 63, q = l >> 4, c = l & 15;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    f32x4 acc[TPW][2];
#pragma unroll
    for (int j = 0; j < TPW; ++j) acc[j][0] = acc[j][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 wa[9][MB];                  // the data gradient's weights: rows = ci, reduction over co
#pragma unroll
    for (int tap = 0; tap < 9; ++tap)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
            wa[tap][mb] = *reinterpret_cast<const bf16x8 *>(wd + (tap * CI + 16 * mb + c) * CO + 8 * q);

    for (int item = blockIdx.x; item < n.B * BANDS; item += gridDim.x) {
        const int b = item / BANDS, oy0 = (item % BANDS) * TH;
        PL::fill(pl, act + (long long)b * CI * HI * HI, oy0, t);
        // gradient rows oy0 .. oy0 + TH, four pixels of four channels per item
        constexpr int XQ = HO / 4, NG = (CO / 4) * (TH + 1) * XQ;
        const float dz = HEAD ? dlogit(n, b) : 0.0f;
        for (int it = t; it < NG; it += 256) {
            const int xq = it % XQ, rg = it / XQ, r = rg % (TH + 1), c4 = rg / (TH + 1);
            uint2 v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[j] = make_uint2(0u, 0u);
                if (oy0 + r < HO) {
                    v[j] = *reinterpret_cast<const uint2 *>(g + ((long long)b * CO + 4 * c4 + j) * HO * HO +
                                                            (oy0 + r) * HO + 4 * xq);
                    if constexpr (HEAD) {
                        const uint32_t d = to_bf16(dz * n.theta[kOffWf + 4 * c4 + j] / (float)(kH3 * kH3));
                        v[j].x = ((v[j].x & 0xFFFFu) ? d : 0u) | ((v[j].x >> 16) ? d << 16 : 0u);
                        v[j].y = ((v[j].y & 0xFFFFu) ? d : 0u) | ((v[j].y >> 16) ? d << 16 : 0u);
                    }
                }
                if (r < TH) *reinterpret_cast<uint2 *>(gp + (4 * c4 + j) * GPS + r * HO + 4 * xq) = v[j];
            }
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const int sh = 16 * (p & 1);
                uint32_t w[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) w[j] = ((p < 2 ? v[j].x : v[j].y) >> sh) & 0xFFFFu;
                *reinterpret_cast<uint2 *>(gc + (r * (HO + 1) + 4 * xq + p) * GCS + 4 * c4) =
                    make_uint2(w[0] | (w[1] << 16), w[2] | (w[3] << 16));
            }
        }
        // column HO of the gradient: zero
        for (int it = t; it < (TH + 1) * (CO / 4); it += 256)
            *reinterpret_cast<uint2 *>(gc + ((it / (CO / 4)) * (HO + 1) + HO) * GCS + 4 * (it % (CO / 4))) =
                make_uint2(0u, 0u);
        __syncthreads();

        // weight gradient
#pragma unroll
        for (int kb = 0; kb < PX / 32; ++kb) {
            const int p = 32 * kb + 8 * q, oy = p / HO, ox = p % HO;   // the lane's eight pixels
            bf16x8 av[2];
#pragma unroll
            for (int m = 0; m < 2; ++m) av[m] = *reinterpret_cast<const bf16x8 *>(gp + (16 * m + c) * GPS + p);
#pragma unroll
            for (int j = 0; j < TPW; ++j) {
                const int tile = wv + 4 * j;   // wave-uniform
                bf16x8 bv;
                if (tile < NT) {
                    const int tap = tile / MB, h = tile - tap * MB, ky = tap / 3, kx = tap - 3 * ky;
                    bv = *reinterpret_cast<const bf16x8 *>(pl + (kx * CI + 16 * h + c) * PL::STR + (2 * oy + ky) * HO + ox);
                } else {
                    const short one = tile == NT && c == 0 ? 0x3F80 : 0;   // 1.0: the bias
                    const short8 o = {one, one, one, one, one, one, one, one};
                    bv = __builtin_bit_cast(bf16x8, o);
                }
#pragma unroll
                for (int m = 0; m < 2; ++m) acc[j][m] = mfma32(av[m], bv, acc[j][m]);
            }
        }
        // data gradient: jobs of 16 columns u of one row v
        constexpr int UB = HO / 16, JOBS = TH * UB;
        for (int job = wv; job < JOBS; job += 4) {
            const int v = job / UB, u = (job % UB) * 16 + c;   // v relative to oy0
            f32x4 d[2][2][MB];
#pragma unroll
            for (int k = 0; k < 4 * MB; ++k) d[k >> 1 & 1][k & 1][k >> 2] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int tap = 0; tap < 9; ++tap) {
                const int ky = tap / 3, kx = tap - 3 * ky;
                const bf16x8 bv = *reinterpret_cast<const bf16x8 *>(
                    gc + ((v + (ky == 0)) * (HO + 1) + u + (kx == 0)) * GCS + 8 * q);
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) d[ky != 1][kx != 1][mb] = mfma32(wa[tap][mb], bv, d[ky != 1][kx != 1][mb]);
            }
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int py = 0; py < 2; ++py)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int ci = 16 * mb + 4 * q + i;
                        const uint16_t *a = pl + (CI + ci) * PL::STR + (2 * v + py + 1) * HO + u;
                        const uint32_t e = a[0] != 0 ? to_bf16(d[py][0][mb][i]) : 0u;
                        const uint32_t o = a[CI * PL::STR] != 0 ? to_bf16(d[py][1][mb][i]) : 0u;
                        *reinterpret_cast<uint32_t *>(gin + (((long long)b * CI + ci) * HI + 2 * (oy0 + v) + py) * HI + 2 * u) =
                            e | (o << 16);
                    }
        }
        __syncthreads();   // the staged band is replaced by the next item's
    }
    float *set = partial + (long long)blockIdx.x * kGradSet<CI, CO>;
#pragma unroll
    for (int j = 0; j < TPW; ++j) {
        const int tile = wv + 4 * j;
        const int tap = tile / MB, h = tile - tap * MB;
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int co = 16 * m + 4 * q + i;
                if (tile < NT) set[(co * 9 + tap) * CI + 16 * h + c] = acc[j][m][i];
                else if (tile == NT && c == 0) set[CO * 9 * CI + co] = acc[j][m][i];
            }
    }
}

// Weight and bias gradient of the first layer (3 input channels, no data
// gradient): rows = the 16 output channels, columns = the 27 (ci, tap)
// pairs and the bias, reduction over the pixels of a band of TH output
// rows, each wave a quarter of them.  The gradient operand is eight
// consecutive pixels of a channel straight from memory.  256 samples: 13 us
// (the 59 MB it reads take 11), 128 us with gathered operands before.
template <int TH>
__global__ __launch_bounds__(256) void conv1_bwd(NetBuffers n, float *__restrict__ partial) {
    constexpr int CI = kC0, CO = kC1, HI = kH0, HO = kH1, BANDS = HO / TH, KB = TH * HO / 32 / 4;
    using PL = Planes<CI, HI, TH>;
    static_assert(CO == 16 && 9 * CI + 1 <= 32 && TH * HO % 128 == 0 && HO % 32 == 0, "layer shape");
    __shared__ __align__(16) uint16_t pl[PL::ELEMS];
    __shared__ float red[3][64][8];
    const int t = threadIdx.x, l = t & 63, q = l >> 4, c = l & 15;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    // the lane's two columns: n = ci 9 + tap, 27 = the bias, above: nothing
    int at[2];
    short pad[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int col = 16 * j + c, ci = col / 9, tap = col - 9 * ci, ky = tap / 3, kx = tap - 3 * ky;
        at[j] = col < 9 * CI ? (kx * CI + ci) * PL::STR + ky * HO : -1;
        pad[j] = col == 9 * CI ? 0x3F80 : 0;
    }
    for (int item = blockIdx.x; item < n.B * BANDS; item += gridDim.x) {
        const int b = item / BANDS, oy0 = (item % BANDS) * TH;
        const uint16_t *gb = n.g1 + ((long long)b * CO + c) * HO * HO + oy0 * HO;
        bf16x8 av[KB];
#pragma unroll
        for (int k = 0; k < KB; ++k) av[k] = *reinterpret_cast<const bf16x8 *>(gb + 32 * (wv * KB + k) + 8 * q);
        PL::fill(pl, n.x0 + (long long)(n.idx ? n.idx[b] : b) * CI * HI * HI, oy0, t);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < KB; ++k) {
            const int p = 32 * (wv * KB + k) + 8 * q, oy = p / HO, ox = p % HO;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const short8 o = {pad[j], pad[j], pad[j], pad[j], pad[j], pad[j], pad[j], pad[j]};
                bf16x8 bv = __builtin_bit_cast(bf16x8, o);
                if (at[j] >= 0) bv = *reinterpret_cast<const bf16x8 *>(pl + at[j] + 2 * oy * HO + ox);
                acc[j] = mfma32(av[k], bv, acc[j]);
            }
        }
        __syncthreads();
    }
    // the four waves' sums, in wave order
    if (wv > 0) {
#pragma unroll
        for (int k = 0; k < 8; ++k) red[wv - 1][l][k] = acc[k >> 2][k & 3];
    }
    __syncthreads();
    if (wv > 0) return;
    float *set = partial + (long long)blockIdx.x * kGradSet<CI, CO>;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        float s = acc[k >> 2][k & 3];
#pragma unroll
        for (int w = 0; w < 3; ++w) s += red[w][l][k];
        const int col = 16 * (k >> 2) + c, co = 4 * q + (k & 3), ci = col / 9;
        if (col < 9 * CI) set[(co * 9 + col - 9 * ci) * CI + ci] = s;
        else if (col == 9 * CI) set[CO * 9 * CI + co] = s;
    }
}

// The gradient from the partial sums, and the head's gradient and the mean
// loss from the logits.  32 parameters per workgroup: 32 threads each
// add every 32nd set in order, and their sums are added in order, so the
// result does not depend on timing.  15 us at batch 256, with all of a
// thread's loads in flight; one thread per parameter walking all sets, and
// one wave walking the samples for the head, took 60 us a layer and 79 us
// (8 threads per parameter: 26 us in all).
constexpr int kRedCols = 32, kRedWays = 32;
template <int CI, int CO>
__device__ void reduce_layer(const float *__restrict__ partial, float *__restrict__ grad, int offw, int offb, int sets,
                             int block, float (*sum)[kRedCols]) {
    constexpr int SET = kGradSet<CI, CO>;
    const int k = threadIdx.x % kRedCols, way = threadIdx.x / kRedCols, i = block * kRedCols + k;
    float s = 0.0f;
    if (i < SET) {
#pragma unroll 16
        for (int w = way; w < sets; w += kRedWays) s += partial[(long long)w * SET + i];
    }
    sum[way][k] = s;
    __syncthreads();
    if (way != 0 || i >= SET) return;
#pragma unroll
    for (int w = 1; w < kRedWays; ++w) s += sum[w][k];
    const int co = i / (9 * CI), tap = (i - co * 9 * CI) / CI, ci = i % CI;
    if (i < CO * 9 * CI) grad[offw + (co * CI + ci) * 9 + tap] = s;
    else grad[offb + i - CO * 9 * CI] = s;
}
__device__ void reduce_head(const NetBuffers &n, float (*sum)[kRedCols]) {
    __shared__ float sdz[kRedWays], sl[kRedWays];
    const int c = threadIdx.x % kRedCols, way = threadIdx.x / kRedCols;
    float s = 0.0f, d = 0.0f, lo = 0.0f;
    for (int b = way; b < n.B; b += kRedWays) {
        const float dz = dlogit(n, b), z = n.logits[b], y = n.labels[n.idx ? n.idx[b] : b];
        s += n.gap[b * kC3 + c] * dz;
        d += dz;
        lo += fmaxf(z, 0.0f) - z * y + log1pf(expf(-fabsf(z)));
    }
    sum[way][c] = s;
    if (c == 0) {
        sdz[way] = d;
        sl[way] = lo;
    }
    __syncthreads();
    if (way != 0) return;
#pragma unroll
    for (int w = 1; w < kRedWays; ++w) s += sum[w][c];
    n.grad[kOffWf + c] = s;
    if (c == 0) {
#pragma unroll
        for (int w = 1; w < kRedWays; ++w) {
            d += sdz[w];
            lo += sl[w];
        }
        n.grad[kOffBf] = d;
        if (n.loss) n.loss[0] = lo / (float)n.B;
    }
}
constexpr int red_blocks(int set) { return (set + kRedCols - 1) / kRedCols; }
constexpr int kRed3 = red_blocks(kGradSet<kC2, kC3>), kRed2 = red_blocks(kGradSet<kC1, kC2>),
              kRed1 = red_blocks(kGradSet<kC0, kC1>);
static_assert(kC3 == kRedCols, "one column per head weight");
__global__ __launch_bounds__(kRedCols * kRedWays) void reduce_grad(NetBuffers n, const float *p3, const float *p2, const float *p1,
                                                   int s3, int s2, int s1) {
    __shared__ float sum[kRedWays][kRedCols];
    const int b = blockIdx.x;   // uniform over the workgroup
    if (b < kRed3) reduce_layer<kC2, kC3>(p3, n.grad, kOffW3, kOffB3, s3, b, sum);
    else if (b < kRed3 + kRed2) reduce_layer<kC1, kC2>(p2, n.grad, kOffW2, kOffB2, s2, b - kRed3, sum);
    else if (b < kRed3 + kRed2 + kRed1) reduce_layer<kC0, kC1>(p1, n.grad, kOffW1, kOffB1, s1, b - kRed3 - kRed2, sum);
    else reduce_head(n, sum);
}

// ---------------------------------------------------------------- AdamW
// Index in the bfloat16 copy of parameter i's second place, in the forward
// layout of its convolution's weights, or -1 for biases and the head; and of
// its third, in the data gradient's layout ([tap][ci][co], layers 2 and 3),
// or -1.
template <int CI>
__device__ inline int forward_at_layer(int n, int perm) {
    const int co = n / (CI * 9), k = n - co * CI * 9, ci = k / 9, tap = k - 9 * ci;
    return perm + co * perm_row(CI) + tap * perm_cip(CI) + ci;
}
__device__ inline int forward_at(int i) {
    if (i >= kOffW1 && i < kOffB1) return forward_at_layer<kC0>(i - kOffW1, kPermW1);
    if (i >= kOffW2 && i < kOffB2) return forward_at_layer<kC1>(i - kOffW2, kPermW2);
    if (i >= kOffW3 && i < kOffB3) return forward_at_layer<kC2>(i - kOffW3, kPermW3);
    return -1;
}

template <int CI, int CO>
__device__ inline int backward_at_layer(int n, int perm) {
    const int co = n / (CI * 9), k = n - co * CI * 9, ci = k / 9, tap = k - 9 * ci;
    return perm + (tap * CI + ci) * CO + co;
}
__device__ inline int backward_at(int i) {
    if (i >= kOffW2 && i < kOffB2) return backward_at_layer<kC1, kC2>(i - kOffW2, kBackW2);
    if (i >= kOffW3 && i < kOffB3) return backward_at_layer<kC2, kC3>(i - kOffW3, kBackW3);
    return -1;
}
__device__ inline void store_bf16(uint16_t *wbf, int i, float v) {
    const uint16_t h = to_bf16(v);
    wbf[i] = h;
    const int f = forward_at(i), b = backward_at(i);
    if (f >= 0) wbf[f] = h;
    if (b >= 0) wbf[b] = h;
}

// Decoupled weight decay on every parameter; refreshes the bfloat16 copy.
__global__ __launch_bounds__(256) void adamw(AdamArgs a) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.n) return;
    const float g = a.grad[i];
    const float m = a.beta1 * a.m[i] + (1.0f - a.beta1) * g;
    const float v = a.beta2 * a.v[i] + (1.0f - a.beta2) * g * g;
    a.m[i] = m;
    a.v[i] = v;
    const float p = a.theta[i];
    const float np = p - a.lr * ((m / a.bc1) / (sqrtf(v / a.bc2) + a.eps) + a.wd * p);
    a.theta[i] = np;
    store_bf16(a.wbf, i, np);
}

__global__ __launch_bounds__(256) void params_to_bf16(const float *theta, uint16_t *wbf) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kNParam) return;
    store_bf16(wbf, i, theta[i]);
}

// ---------------------------------------------------------------- features
// Number of positions i in [0, n) with floor(i * cells / n) == c.
__device__ inline long long cell_span(long long c, long long n, long long cells) {
    return ((c + 1) * n + cells - 1) / cells - (c * n + cells - 1) / cells;
}

// Cell sums to bfloat16 features: (mean value) / maxval, (pixels with
// Z_1 != 0) / area, (Z_2 != 0) / area.  Feature set blockIdx.y covers
// image blockIdx.y / (gx gy) and, within it, region blockIdx.y % (gx gy)
// (row-major, gx regions per row) of kCells x kCells cells; the image's
// cell grid is gy kCells rows by gx kCells columns (gx = gy = 1: the whole
// image).  A workgroup takes kFinRows cell rows of one set; the cell
// spans of its rows and columns (64-bit divisions) are computed once into
// LDS.
constexpr int kFinRows = 16;
__global__ __launch_bounds__(256) void finish_features(Launch L, const unsigned long long *__restrict__ cells,
                                                       double maxval, uint16_t *__restrict__ feats, int gx,
                                                       int gy) {
    static_assert(kCells + kFinRows <= 256 && kCells % kFinRows == 0, "spans of one workgroup");
    __shared__ long long span_x[kCells], span_y[kFinRows];
    const int set = blockIdx.y, nreg = gx * gy;
    const int img = set / nreg, reg = set - img * nreg;
    const ImageJob &J = L.nimg == 1 ? L.one : L.jobs[img];
    const long long CX = (long long)gx * kCells, CY = (long long)gy * kCells;
    const int r0 = blockIdx.x * kFinRows;
    const long long cy0 = (long long)(reg / gx) * kCells + r0, cx0 = (long long)(reg % gx) * kCells;
    const int t = threadIdx.x;
    const unsigned long long *cs0 = cells + (long long)img * 2 * CX * CY + cy0 * CX + cx0;
    uint16_t *f = feats + (long long)set * kFeatC * kCellCount + r0 * kCells;
    // every cell's two sums are loaded before the spans and the first use
    constexpr int U = kFinRows * kCells / 256;
    static_assert(U * 256 == kFinRows * kCells, "whole cells per thread");
    unsigned long long sv[U], zz[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int j = t + 256 * u, r = j / kCells, x = j - r * kCells;
        sv[u] = cs0[r * CX + x];
        zz[u] = cs0[CX * CY + r * CX + x];
    }
    if (t < kCells) span_x[t] = cell_span(cx0 + t, J.img.W, CX);
    else if (t < kCells + kFinRows) span_y[t - kCells] = cell_span(cy0 + (t - kCells), J.img.H, CY);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int j = t + 256 * u, r = j / kCells, x = j - r * kCells;
        const long long area = span_y[r] * span_x[x];
        uint16_t f0 = 0, f1 = 0, f2 = 0;
        if (area > 0) {
            const double ar = (double)area;
            f0 = to_bf16((float)(((double)sv[u] / ar) / maxval));
            f1 = to_bf16((float)((double)(zz[u] & 0xFFFFFFFFull) / ar));
            f2 = to_bf16((float)((double)(zz[u] >> 32) / ar));
        }
        f[j] = f0;
        f[kCellCount + j] = f1;
        f[2 * kCellCount + j] = f2;
    }
}

// Clears n2 16-byte words (the cell sums: two per pair of cells).
__global__ __launch_bounds__(256) void zero_cells(ulonglong2 *p, long long n2) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n2) p[i] = make_ulonglong2(0ull, 0ull);
}

inline unsigned blocks(long long n, int t) { return (unsigned)((n + t - 1) / t); }

template <int CI, int CO, int HI, int TH>
hipError_t fwd(const uint16_t *in, const int *idx, const uint16_t *w, const float *bias, uint16_t *out, int B,
               hipStream_t s) {
    hipLaunchKernelGGL((conv_fwd<CI, CO, HI, TH>), dim3((unsigned)B * (HI / 2 / TH)), dim3(256), 0, s, in, idx, w,
                       bias, out, B);
    return hipGetLastError();
}

}  // namespace

long long partial_elems(int B) {
    return (long long)bwd_groups(B, kH3, kBand3) * kGradSet<kC2, kC3> +
           (long long)bwd_groups(B, kH2, kBand2) * kGradSet<kC1, kC2> +
           (long long)bwd_groups(B, kH1, kBand1) * kGradSet<kC0, kC1>;
}

hipError_t launch_zero_cells(unsigned long long *cells, long long nsets, hipStream_t s) {
    const long long n = nsets * 2 * kCellCount;
    static_assert(kCellCount % 2 == 0, "cell sums in 16-byte words");
    hipLaunchKernelGGL(zero_cells, dim3(blocks(n / 2, 256)), dim3(256), 0, s, reinterpret_cast<ulonglong2 *>(cells),
                       n / 2);
    return hipGetLastError();
}

hipError_t launch_finish_features(const Launch &L, const unsigned long long *cells, double maxval, uint16_t *feats,
                                  int gx, int gy, hipStream_t s) {
    hipLaunchKernelGGL(finish_features, dim3(kCells / kFinRows, L.nimg * gx * gy), dim3(256), 0, s, L, cells, maxval,
                       feats, gx, gy);
    return hipGetLastError();
}

hipError_t launch_forward(const NetBuffers &n, hipStream_t s, int *flags, uint8_t *decisions) {
    // conv_fwd copies each layer's weights in 16-byte chunks
    static_assert(kPermW1 % 8 == 0 && kPermW2 % 8 == 0 && kPermW3 % 8 == 0, "weight offsets");
    hipError_t e;
    // output rows per workgroup: 4, 4, 8 (measured against 8, 8 and 4, 16)
    if ((e = fwd<kC0, kC1, kH0, 4>(n.x0, n.idx, n.w + kPermW1, n.theta + kOffB1, n.a1, n.B, s)) != hipSuccess) return e;
    if ((e = fwd<kC1, kC2, kH1, 4>(n.a1, nullptr, n.w + kPermW2, n.theta + kOffB2, n.a2, n.B, s)) != hipSuccess) return e;
    if ((e = fwd<kC2, kC3, kH2, 8>(n.a2, nullptr, n.w + kPermW3, n.theta + kOffB3, n.a3, n.B, s)) != hipSuccess) return e;
    hipLaunchKernelGGL(head_fwd, dim3(n.B), dim3(256), 0, s, n.a3, n.theta, n.gap, n.logits, flags, decisions);
    return hipGetLastError();
}

hipError_t launch_backward(const NetBuffers &n, hipStream_t s) {
    static_assert(kC2 == 32 && kC3 == 32 && kBackW2 % 8 == 0 && kBackW3 % 8 == 0, "conv_bwd's layers");
    const int s3 = bwd_groups(n.B, kH3, kBand3), s2 = bwd_groups(n.B, kH2, kBand2), s1 = bwd_groups(n.B, kH1, kBand1);
    float *p3 = n.partial, *p2 = p3 + (long long)s3 * kGradSet<kC2, kC3>, *p1 = p2 + (long long)s2 * kGradSet<kC1, kC2>;
    hipError_t e;
    hipLaunchKernelGGL((conv_bwd<kC2, kH2, kBand3, true>), dim3(s3), dim3(256), 0, s, n, n.a3, n.a2, n.w + kBackW3,
                       n.g2, p3);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL((conv_bwd<kC1, kH1, kBand2, false>), dim3(s2), dim3(256), 0, s, n, n.g2, n.a1, n.w + kBackW2,
                       n.g1, p2);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL((conv1_bwd<kBand1>), dim3(s1), dim3(256), 0, s, n, p1);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(reduce_grad, dim3(kRed3 + kRed2 + kRed1 + 1), dim3(kRedCols * kRedWays), 0, s, n, p3, p2, p1, s3, s2, s1);
    return hipGetLastError();
}

hipError_t launch_adamw(const AdamArgs &a, hipStream_t s) {
    hipLaunchKernelGGL(adamw, dim3(blocks(a.n, 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_params_to_bf16(const float *theta, uint16_t *wbf, hipStream_t s) {
    hipLaunchKernelGGL(params_to_bf16, dim3(blocks(kNParam, 256)), dim3(256), 0, s, theta, wbf);
    return hipGetLastError();
}

}  // namespace gate
}  // namespace logfx
