// Pass 1 with the LoG on the matrix cores.
//
// The LoG is a contraction of 81 (25) pixels with 16-bit taps.  On the FP64
// path, which 16-bit images take (their sums need 35 bits), the vector unit
// spends most of pass 1 on it: a conversion and an FP64 multiply-add per
// orbit.  The bytes' products need no more than int32, so here it costs the
// vector unit the issue of the matrix instructions: 6001 x 3501, pass 1 169
// -> 129 us.  (The integer path keeps its packed form, two taps per vector
// instruction: 8192^2, 196 us against 256 for this one with int32 responses,
// whose vector and matrix instructions ran one after the other at three waves
// per SIMD.)
//
// Here pixels and taps are split into signed bytes, p = 256 (ph + 128) +
// (pl + 128) and k = 256 kh + kl, and the products run as
// v_mfma_i32_16x16x64_i8, whose sums are exact:
//   L = 65536 sum kh ph + 256 sum (kh pl + kl ph) + sum kl pl + K0,
// K0 = 128 * 257 sum k (0 for the zero-sum masks).
//
// GEMM rows are 16 output columns x, GEMM columns are 8 output rows of two
// neighbouring blocks of 16 x, and the reduction runs over 2 image rows x 32
// image columns per MFMA.  The taps' operand is a band matrix: lane
// (row x, 16 columns) holds 16 consecutive bytes of a zero-padded tap row, so
// it is one 16-byte load from a table of padded rows, 1152 bytes that come as a
// kernel argument: nothing is allocated or launched for a pair of masks (6001 x
// 3501, all of the call: 171 us with a table in device memory, 171 so).
// The pixels' operand is 16 consecutive bytes of a byte plane in LDS.  An odd
// number of mask rows leaves one row slot of the last pair free: it reads the
// centre row again, with what its taps exceed 16 bits by (the centre tap of
// the default masks does).
//
// A wave owns 64 columns (62 of them output columns) of a strip and walks
// down it 8 rows at a time, on its own: it stages the 8 image rows that enter
// the window into its ring of 16 rows in LDS (their loads are issued a block
// ahead), takes both LoGs of 8 rows and writes them to LDS, and then reads
// them back with one lane per column for the crossings, whose vertical
// neighbours are the rows before and after in registers.  No barrier until
// the strip ends.
#pragma once
#include "logfx_kernels.h"

namespace logfx {
namespace kern {

typedef int i32x4 __attribute__((ext_vector_type(4)));

// Sign bits in place of compares and selects: adds, xors and ands issue at
// nearly twice their rate.  Decision (all ones or zero) of a crossing of
// centre a stronger than thr, and its strength c.  For a < 0, a + lo < 0, and
// a + hi >= 0 iff some neighbour reaches -a; for a > 0, a + hi > 0, and
// a + lo < 0 likewise: a crossing iff the two sums differ in sign.  ZERO: the
// rule for a zero centre as well (opposite signs left / right or up / down).
__device__ inline double max_f64(double a, double b) {   // finite operands
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ inline double min_f64(double a, double b) {
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
template <bool ZERO>
__device__ inline int crossing(double a, double up, double dn, double lf, double rt, double thr, double &c) {
    const double hi = max_f64(max_f64(max_f64(up, dn), max_f64(lf, rt)), a);
    const double lo = min_f64(min_f64(min_f64(up, dn), min_f64(lf, rt)), a);
    c = hi - lo;   // exact, like the sums below: integers below 2^52
    const int strong = __double2hiint(thr - c);
    int m = (__double2hiint(a + hi) ^ __double2hiint(a + lo)) & strong;   // a difference of equals is +0
    if constexpr (ZERO) m = a == 0.0 ? ((opposite(lf, rt) | opposite(up, dn)) ? strong : 0) : m;
    return m >> 31;
}
__device__ inline double masked(double c, int m) {
    return __hiloint2double(__double2hiint(c) & m, __double2loint(c) & m);
}

// LDS of a workgroup: the waves' pixel rings in two regions of 8 rows each,
// a power of two apart (the block's parity toggles one address bit), each
// wave's planes of 8 rows x 80 bytes (5 units of 16 bytes: 8 rows of an
// operand read lie in different banks); then the waves' responses, 8 rows of
// 64 pairs with 16 bytes of padding.
struct MatLds {
    static constexpr int PLANE = 8 * 80, WAVE = 2 * PLANE;
    static constexpr int REGION = 8192;
    static_assert(kTileWaves * WAVE <= REGION, "ring region");
    static constexpr int RESP = REGION + kTileWaves * WAVE;
    static constexpr int LROW = 64 * 2 * (int)sizeof(double) + 16, LWAVE = 8 * LROW;
    static constexpr int BYTES = RESP + kTileWaves * LWAVE;
    static_assert(RESP % 16 == 0, "aligned responses");
    static_assert(BYTES + (kTileSums + 2) * kTileWaves * 8 == kMatLdsBytes, "LDS that the host counts on");
};

// Waves per SIMD the registers have to allow (the taps' operands alone take
// 40, the sums of a block 24).  With masks of 5 and 9 the form that stores the
// strengths takes 159 and runs at 3, with the gate's cells 169 and 2.
constexpr int kPass1mWaves = 2;

template <int RA, int RB, int MODE, bool LOOP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kPass1mWaves)))
void pass1m_kernel(Pass1Args<OrbitTapsD> a, MatTable table) {
    using M = MatLds;
    using Acc = double;
    constexpr int HL = kHalo1, OW = kWave - 2 * HL, TW = tile_out_width(HL);
    constexpr int GA = (RA + 1) / 2, GB = (RB + 1) / 2;   // pairs of distances of the two masks
    constexpr int NP = 1 + 2 * GB;                        // row pairs: the centre, then g above, g below
    static_assert(HL == 1, "a strip's responses start one row above it");
    __shared__ __align__(16) unsigned char sm[M::BYTES];
    __shared__ unsigned long long red[kTileSums][kTileWaves];
    __shared__ long long redc[2][kTileWaves];
    extern __shared__ unsigned cellv[];       // cell sums (kP1Cells)
    unsigned *const cellc = cellv + a.cell_rows * a.cell_slots;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int q = lane >> 4, n = lane & 15;   // MFMA lane coordinates

    // the taps' operands: [pair of distances][high, low byte]
    i32x4 ta[GA + 1][2], tb[GB + 1][2];
    {
        typedef i32x4 V __attribute__((aligned(1)));
        const unsigned char *row = table.b + 16 * (q & 1) - n + 15;   // column 16 (q & 1) - 8 - x, at 23 + column
#pragma unroll
        for (int g = 0; g <= GB; ++g)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int e = 2 * g + (q >> 1);
                if (g <= GA) ta[g <= GA ? g : 0][h] = *reinterpret_cast<const V *>(row + (e * 2 + h) * kMatRow);
                tb[g][h] = *reinterpret_cast<const V *>(row + ((kMatEntries + e) * 2 + h) * kMatRow);
            }
    }
    // LDS offsets of the pixels' operands for an even block: the lane's row
    // and 16 columns of each pair (an odd radius leaves a row with zero taps
    // in its last pairs, which may wrap around the ring)
    int at[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        const int d = j == 0 ? 0 : 2 * ((j + 1) / 2) - 1 + (q >> 1);   // distance
        const int s = ((n & 7) + RB + (j % 2 ? -d : d)) & 15;          // ring row
        at[j] = (s >> 3) * M::REGION + wave * M::WAVE + (s & 7) * 80 + 16 * ((n >> 3) + (q & 1));
    }
    unsigned char *const resp = sm + M::RESP + wave * M::LWAVE;
    unsigned char *const rput = resp + (n & 7) * M::LROW + ((n >> 3) * 16 + 4 * q) * 2 * (int)sizeof(Acc);
    const unsigned char *const rget = resp + lane * 2 * (int)sizeof(Acc);
    // staging: chunks of 8 pixels, 10 per ring row, the lane's at rows fr[], columns 8 fc[]
    int fr[2], fx[2], fa[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int id = lane + 64 * k;
        fr[k] = id / 10;
        fx[k] = 8 * (id - 10 * fr[k]);
        fa[k] = wave * M::WAVE + fr[k] * 80 + fx[k];
    }

    for_each_tile<LOOP>(a.L.total1, [&](const int item) __attribute__((always_inline)) {
    const int image = a.L.nimg == 1 ? 0 : a.L.owner1[item];
    const ImageJob J = job_of(a.L, image);
    const int H = (int)J.img.H, W = (int)J.img.W;
    const int tile = item - J.base1, tx = tile % J.tiles_x1, ty = tile / J.tiles_x1;
    const int x0 = tx * TW, y0 = ty * a.rows;
    const int Rv = __builtin_amdgcn_readfirstlane(min(a.rows, H - y0));
    const int base = x0 + wave * OW - HL, xc = base + lane;
    const bool outc = lane >= HL && lane < HL + OW && xc < W;
    const long long zoff = (long long)__builtin_amdgcn_readfirstlane((int)(J.zoff >> 32)) << 32 |
                           (unsigned)__builtin_amdgcn_readfirstlane((int)J.zoff);
    const bool clampL = xc <= 0, clampR = xc >= W - 1;
    const int t0 = y0 - HL, nrows = Rv + 2 * HL;   // responses of rows t0 .. t0 + nrows - 1
    const bool u16 = J.img.dtype == 1;
    const long long pitch = J.img.pitch;
    const int c0 = base - 8;                       // image column of ring column 0

    if constexpr ((MODE & kP1Cells) != 0) {
        for (int i = threadIdx.x; i < a.cell_rows * a.cell_slots; i += blockDim.x) cellv[i] = cellc[i] = 0;
        __syncthreads();
    }
    LaneSums<Acc> sums;
    int cnt[2] = {0, 0};
    // the gate's cells: see pass1_kernel (the same sums and slots)
    auto cell_of = [](long long v, int cells, long long d) { return (int)floor((double)v * cells / (double)d); };
    unsigned fv = 0, fc[2] = {0, 0};
    int fcy = 0, fat = 0, fslot = 0, fend = 0;
    const int flast = y0 + Rv - 1;
    auto cell_end = [&](const long long cy) __attribute__((always_inline)) {
        return (int)((((cy + 1) * H + (1ll << a.cells_ly) - 1) >> a.cells_ly) - 1);
    };
    if constexpr ((MODE & kP1Cells) != 0) {
        const int CX = 1 << a.cells_lx, CY = 1 << a.cells_ly;
        fslot = outc ? cell_of(xc, CX, W) - cell_of(x0, CX, W) : 0;
        fcy = cell_of(y0, CY, H);
        fend = min(__builtin_amdgcn_readfirstlane(cell_end(fcy)), flast);
    }
    auto flush = [&](const int r) __attribute__((always_inline)) {
        if (outc && (fv | fc[0] | fc[1])) {
            atomicAdd(&cellv[fat + fslot], fv);
            atomicAdd(&cellc[fat + fslot], fc[0] | fc[1] << 16);
        }
        cnt[0] += (int)fc[0];
        cnt[1] += (int)fc[1];
        fv = fc[0] = fc[1] = 0;
        int cy = fcy + 1;   // the first cell row past fcy that reaches past r
        while (cell_end(cy) < r + 1) ++cy;
        fat += (cy - fcy) * a.cell_slots;
        fcy = cy;
        fend = min(__builtin_amdgcn_readfirstlane(cell_end(cy)), flast);
    };

    if (base + HL < W) {   // wave-uniform: a wave right of the image has nothing to do
        const bool inner_x = c0 >= 0 && c0 + 80 <= W;
        // the lane's two chunks of 8 image rows from row y, clamped to the image
        uint4 px[2];
        auto fetch = [&](const int y) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                if (k == 1 && lane >= 16) break;   // 80 chunks
                const long long row = (long long)min(max(y + fr[k], 0), H - 1) * pitch;
                const int c = c0 + fx[k];
                if (inner_x || (c >= 0 && c + 8 <= W)) {
                    px[k] = load8(J.img.data, row + c, u16);
                } else {
                    typedef __attribute__((address_space(1))) const uint16_t GU16;
                    typedef __attribute__((address_space(1))) const uint8_t GU8;
                    // pixel by pixel with clamped columns; rolled, for its
                    // registers are live beside the taps'
                    auto pixel = [&](const int x) __attribute__((always_inline)) {
                        const long long o = row + min(max(x, 0), W - 1);
                        return u16 ? (unsigned)((GU16 *)J.img.data)[o] : (unsigned)((GU8 *)J.img.data)[o];
                    };
                    uint4 v = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll 1
                    for (int i = 0; i < 8; i += 2) {
                        const unsigned w = pixel(c + i) | pixel(c + i + 1) << 16;
                        v = make_uint4(v.y, v.z, v.w, w);
                    }
                    px[k] = v;
                }
            }
        };
        // the fetched rows into ring region g, as planes of bytes less 128
        auto stage = [&](const int g) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                if (k == 1 && lane >= 16) break;
                unsigned char *d = sm + g * M::REGION + fa[k];
                const uint4 v = px[k];
                *reinterpret_cast<uint2 *>(d) =
                    make_uint2(__builtin_amdgcn_perm(v.y, v.x, 0x06040200u) ^ 0x80808080u,
                               __builtin_amdgcn_perm(v.w, v.z, 0x06040200u) ^ 0x80808080u);
                *reinterpret_cast<uint2 *>(d + M::PLANE) =
                    make_uint2(__builtin_amdgcn_perm(v.y, v.x, 0x07050301u) ^ 0x80808080u,
                               __builtin_amdgcn_perm(v.w, v.z, 0x07050301u) ^ 0x80808080u);
            }
        };
        // both responses of the 8 rows of block b to LDS; whether one is zero
        auto responses = [&](const int b) __attribute__((always_inline)) {
            const int flip = (b & 1) * M::REGION;
            uint64_t zeros = 0;
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                i32x4 hh[2] = {}, mid[2] = {}, ll[2] = {};
                // each pair's pixels are read while the pair before is multiplied
                i32x4 bl, bh = {};
                auto read = [&](const int j, i32x4 &l, i32x4 &h) __attribute__((always_inline)) {
                    const unsigned char *src = sm + (at[j] ^ flip) + 32 * p;
                    l = *reinterpret_cast<const i32x4 *>(src);
                    h = *reinterpret_cast<const i32x4 *>(src + M::PLANE);
                };
                read(0, bl, bh);
#pragma unroll
                for (int j = 0; j < NP; ++j) {
                    const int g = (j + 1) / 2, gc = g <= GA ? g : 0;
                    i32x4 nl = {}, nh = {};
                    if (j + 1 < NP) read(j + 1, nl, nh);
                    ll[1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(tb[g][1], bl, ll[1], 0, 0, 0);
                    mid[1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(tb[g][0], bl, mid[1], 0, 0, 0);
                    if (g <= GA) {
                        ll[0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ta[gc][1], bl, ll[0], 0, 0, 0);
                        mid[0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ta[gc][0], bl, mid[0], 0, 0, 0);
                    }
                    hh[1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(tb[g][0], bh, hh[1], 0, 0, 0);
                    if (g <= GA) hh[0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ta[gc][0], bh, hh[0], 0, 0, 0);
                    mid[1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(tb[g][1], bh, mid[1], 0, 0, 0);
                    if (g <= GA) mid[0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ta[gc][1], bh, mid[0], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);   // keeps the reads one pair ahead, not all at once
                    bl = nl;
                    bh = nh;
                }
                Acc r[2][4];
#pragma unroll
                for (int m = 0; m < 2; ++m)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        int t = (mid[m][i] << 8) + ll[m][i];
                        asm("" : "+v"(t));   // two shift-adds (left to itself the compiler takes three instructions)
                        r[m][i] = __fma_rn((double)hh[m][i], 65536.0, (double)t);
                    }
                if (a.mat.sum) {   // masks that do not sum to zero
#pragma unroll
                    for (int m = 0; m < 2; ++m)
#pragma unroll
                        for (int i = 0; i < 4; ++i) r[m][i] += a.mat.kd[m];
                }
#pragma unroll
                for (int m = 0; m < 2; ++m)
#pragma unroll
                    for (int i = 0; i < 4; ++i) zeros |= __ballot(r[m][i] == Acc(0));
                unsigned char *d = rput + p * 32 * 2 * (int)sizeof(Acc);
#pragma unroll
                for (int i = 0; i < 4; ++i) *reinterpret_cast<double2 *>(d + 16 * i) = make_double2(r[0][i], r[1][i]);
                __builtin_amdgcn_sched_barrier(0);
            }
            return zeros != 0;
        };
        Acc L1[2] = {0, 0}, L2[2] = {0, 0};   // the responses of the two rows before
        struct Pair {
            Acc v[2];
        };
        auto get = [&](const int i, Acc (&v)[2]) __attribute__((always_inline)) {
            const Pair p = *reinterpret_cast<const Pair *>(rget + i * M::LROW);
            v[0] = p.v[0];
            v[1] = p.v[1];
        };
        // response row t, v; with it the crossings of row t - 1 (unless t is
        // the strip's first or second response row)
        auto step = [&](const int t, Acc (&v)[2], auto clamp, auto zero, const bool skip, const unsigned pixel)
                        __attribute__((always_inline)) {
            constexpr bool C = decltype(clamp)::value;
            const int r = t - 1;
            Acc z[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                if (C && t > H - 1) v[j] = L1[j];   // below the image the last row repeats
                if (C && t == 0) L1[j] = v[j];      // above it the first
            }
            if (!skip) {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    Acc lf, rt, c;
                    neighbours<C>(L1[j], clampL, clampR, lf, rt);
                    int m = crossing<decltype(zero)::value>(L1[j], L2[j], v[j], lf, rt, AccOps<Acc>::thr(a, j), c);
                    asm("" : "+v"(m));   // one mask, not also its sign bit on its own
                    z[j] = masked(c, m);
                    sums.add(j, z[j]);   // every lane; what the lanes outside the output hold is dropped after the strip
                    fc[j] -= (unsigned)m;
                }
                if constexpr ((MODE & kP1StoreZ) != 0) {
                    if (outc) store_strengths(a.z, zoff + (long long)r * W + base, lane, z);
                }
                if constexpr ((MODE & kP1Cells) != 0) {
                    fv += pixel;
                    if (r == fend) flush(r);
                }
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                L2[j] = L1[j];
                L1[j] = v[j];
            }
            __builtin_amdgcn_sched_barrier(0);   // row by row: interleaved rows cost registers
        };
        // the gate: pixel values of the 8 rows whose crossings block b takes
        // (ring row of response row i - 1, column 8 + lane), kept from before
        // their ring rows are replaced
        unsigned pv[(MODE & kP1Cells) != 0 ? 8 : 1] = {};
        auto pixels = [&](const int b) __attribute__((always_inline)) {
            if constexpr ((MODE & kP1Cells) != 0) {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int sr = i - 1 + RB;
                    const unsigned char *p = sm + (((sr >> 3) ^ (b & 1)) * M::REGION) + wave * M::WAVE + (sr & 7) * 80 + 8 + lane;
                    pv[i] = (p[0] ^ 0x80u) | (p[M::PLANE] ^ 0x80u) << 8;
                }
            }
        };
        // a block of 8 response rows from row t, none of them and of the row
        // before with a zero; each row is read a row ahead
        auto block = [&](const int t, auto clamp) __attribute__((always_inline)) {
            Acc v[2][2];
            get(0, v[0]);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                if (i < 7) get(i + 1, v[(i + 1) & 1]);
                step(t + i, v[i & 1], clamp, bool_c<false>{}, false, (MODE & kP1Cells) != 0 ? pv[i] : 0u);
            }
        };
        // the same with the zero rule, for `count` rows (rolled: the strip's
        // first and last blocks and those with zeros); rows i < 2 of the first
        // block only fill the registers
        auto part = [&](const int t, const int count, const bool first) __attribute__((always_inline)) {
            Acc v[2], w[2];
            get(0, v);
#pragma unroll 1
            for (int i = 0; i < count; ++i) {
                get(min(i + 1, 7), w);
                unsigned pixel = 0;
                if constexpr ((MODE & kP1Cells) != 0) {   // pv[i], rotated
                    pixel = pv[0];
#pragma unroll
                    for (int k = 0; k < 7; ++k) pv[k] = pv[k + 1];
                }
                step(t + i, v, bool_c<true>{}, bool_c<true>{}, first && i < 2, pixel);
                v[0] = w[0];
                v[1] = w[1];
            }
            // nothing in flight here: the wait for the next block's pixels
            // then counts the other path's stores only
            __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
        };
        auto order = [] {   // LDS is written and read by different lanes of the wave, which executes in order
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        };
        const bool inner = c0 + 8 >= 1 && base + kWave <= W - 1 && t0 >= 1 && t0 + nrows - 1 <= H - 1;
        const int y_ring = t0 - RB;   // image row of ring row 0
        bool carried = false;
        // per block: both LoGs, then the ring takes the 8 rows fetched during
        // the block before and the next 8 are fetched, then the crossings; so
        // the wait for the rows is no wait for the strengths stored after them
        fetch(y_ring);
        order();   // (a persistent launch: the previous tile's reads)
        stage(0);
        fetch(y_ring + 8);
        stage(1);
        fetch(y_ring + 16);
        for (int b = 0; 8 * b < nrows; ++b) {
            const int t = t0 + 8 * b, left = nrows - 8 * b;
            order();
            const bool zeros = responses(b);
            pixels(b);
            order();
            if (left > 8) stage(b & 1);
            if (left > 16) fetch(y_ring + 8 * b + 24);
            if (b == 0 || left < 8 || zeros || carried) part(t, min(8, left), b == 0);
            else if (inner) block(t, bool_c<false>{});
            else block(t, bool_c<true>{});
            carried = zeros;   // its last row is the next block's first centre
        }
    }
    cnt[0] += (int)fc[0];
    cnt[1] += (int)fc[1];

    if constexpr ((MODE & kP1Cells) != 0) {
        // the tile's cell slots into the image's counters, one thread per slot
        __syncthreads();
        unsigned long long *fcells = a.cells + ((long long)image << (a.cells_lx + a.cells_ly + 1));
        const int CX = 1 << a.cells_lx, CY = 1 << a.cells_ly;
        const int fkey0 = cell_of(x0, CX, W);
        const int fslots = cell_of(min(x0 + TW, W) - 1, CX, W) - fkey0 + 1;
        const int fcy0 = cell_of(y0, CY, H);
        const int fspan = cell_of(flast, CY, H) - fcy0 + 1;
        for (int i = threadIdx.x; i < fspan * fslots; i += blockDim.x) {
            const int cr = i / fslots, cc = i - cr * fslots;
            const unsigned v = cellv[cr * a.cell_slots + cc];
            const unsigned c = cellc[cr * a.cell_slots + cc];
            if (v | c) {
                unsigned long long *cell = fcells + ((long long)(fcy0 + cr) << a.cells_lx) + fkey0 + cc;
                atomicAdd(cell, (unsigned long long)v);
                atomicAdd(cell + (1ll << (a.cells_lx + a.cells_ly)),
                          (unsigned long long)(c & 0xFFFFu) | ((unsigned long long)(c >> 16) << 32));
            }
        }
    }

    // Deterministic per-tile reduction: fixed butterfly per wave, then the
    // waves in order.
#pragma unroll
    for (int k = 0; k < LaneSums<Acc>::words; ++k) {
        const unsigned long long v = sums.word(k, outc);
        if (lane == 0) red[k][wave] = v;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) cnt[j] = wave_sum(outc ? cnt[j] : 0);
    if (lane == 0) {
        redc[0][wave] = cnt[0];
        redc[1][wave] = cnt[1];
    }
    __syncthreads();
    if (threadIdx.x < LaneSums<Acc>::words) {
        unsigned long long v = red[threadIdx.x][0];
        for (int w = 1; w < kTileWaves; ++w) v = LaneSums<Acc>::plus(v, red[threadIdx.x][w]);
        a.partials[(long long)item * kTileSums + threadIdx.x] = v;
    } else if (threadIdx.x >= kWave && threadIdx.x < kWave + 2) {
        const int j = threadIdx.x - kWave;
        a.counts[(long long)item * 2 + j] = (redc[j][0] + redc[j][1]) + (redc[j][2] + redc[j][3]);
    }
    __syncthreads();   // the reduction buffers are reused by the next tile
    });
}

template <int RA, int RB, int MODE>
hipError_t p1m(const Pass1Args<OrbitTapsD> &a, const MatTable &t, int grid, hipStream_t s, int *max_grid) {
    const size_t shm = (MODE & kP1Cells) != 0 ? 2 * sizeof(unsigned) * a.cell_rows * a.cell_slots : 0;
    const dim3 block(kTileWaves * kWave);
    constexpr bool CAN_LOOP = (MODE & kP1Cells) == 0;   // the cell-summing form runs one tile per workgroup
    if (max_grid) return occupancy(pass1m_kernel<RA, RB, MODE, CAN_LOOP>, shm, max_grid);
    if (!CAN_LOOP || grid >= a.L.total1)
        hipLaunchKernelGGL((pass1m_kernel<RA, RB, MODE, false>), dim3(a.L.total1), block, shm, s, a, t);
    else
        hipLaunchKernelGGL((pass1m_kernel<RA, RB, MODE, CAN_LOOP>), dim3(grid), block, shm, s, a, t);
    return hipGetLastError();
}

}  // namespace kern
}  // namespace logfx
