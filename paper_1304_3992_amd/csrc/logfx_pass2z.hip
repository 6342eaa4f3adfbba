// Pass 2 on stored crossing strengths: E_j = [3x3 deviation of Z_j > T_j]
// (eq. (2), Sec. 4.1), E = E_1 OR E_2, F = hybrid median of E (Sec. 3.4).
//
// Pass 1 has written the strengths (Z_1, Z_2) of every pixel to HBM, so this
// pass computes no LoG: each lane of a wave reads its column's strengths,
// eight rows at a time, with clamp-to-edge coordinates (the columns and rows
// outside the image read the edge pixel's, which are the clamped operands of
// the deviation), and takes the neighbours' column sums from the adjacent
// lanes.  No LDS; halo 3 columns (median 2 + deviation 1), 58 output columns
// per wave.
//
// Read in full, the strengths' way through memory bounds this pass (8192^2:
// 154 to 159 us with FP64 tests, 150 to 159 with FP32 ones, 154 with no
// arithmetic at all).  So the strengths are
// stored split (ZMap), and the deviation test is decided from the top 16
// bits of each, 4 bytes per pixel, wherever they can decide it: what the low
// bits may add and the rounding error of the FP32 evaluation are bounded,
// and rows in which some lane's distance to the threshold is within that
// bound (one in two to five hundred on the package's scenes) are tested
// again on the exact strengths in FP64, with the operations and in the order
// of the pass that recomputes the strengths.  The extracted bits are
// therefore those of the FP64 test, everywhere.  Where the threshold is
// small against the code step (kCoarse), the low bits are read for every row
// and only the rounding is left to bound.  8192^2: 103 us, 295 MB read, 42
// vector instructions per output pixel (halo lanes and rows included), which
// take 0.82 of the issue slots; pass 1 pays 8 us for the split.  6001 x 3501, 16 bits (12 bytes a
// pixel stored, 16 before, of which 4 are read): 89 -> 39 us.
//
// Each lane collects the E bits of its own column in a 64-bit shift register
// (two words, the newest row at bit 0).  Once 36 rows past a word's start are
// known, the hybrid median of its 32 output rows is taken on whole words: a
// row offset is a funnel shift of the two words, a column offset a lane
// shift, and each logic operation treats 32 pixels.
//
// With the 5x5 first stage (Sec. 4.1, std5_max >= 0) a pixel is extracted
// only if its 5x5 deviation also exceeds std5_max: five-row column sums
// beside the three-row ones, halo 4 (56 output columns).
#include "logfx_kernels.h"

namespace logfx {
namespace kern {

typedef __attribute__((address_space(1))) uint8_t GlobalU8;
// Bits s .. s + 31 of the 64-bit word hi:lo.
__device__ inline unsigned funnel(unsigned hi, unsigned lo, int s) { return __builtin_amdgcn_alignbit(hi, lo, s); }

// Hybrid median (window M = 3 or 5) of the 32 pixels of a column word:
// bit k of w1:w0 >> 2 is the centre of output pixel k, bits k .. k + 4 its
// column window (in either row order: the median is symmetric); the other
// columns come from the neighbouring lanes.
template <int M>
__device__ inline unsigned median_word(unsigned w0, unsigned w1) {
    const unsigned c = funnel(w1, w0, 2);
    const unsigned l0 = from_left(w0), l1 = from_left(w1);     // column x - 1
    const unsigned r0 = from_right(w0), r1 = from_right(w1);   // column x + 1
    if constexpr (M == 3) {
        const unsigned p[4] = {funnel(l1, l0, 2), funnel(r1, r0, 2), funnel(w1, w0, 1), funnel(w1, w0, 3)};
        const unsigned x[4] = {funnel(l1, l0, 1), funnel(r1, r0, 1), funnel(l1, l0, 3), funnel(r1, r0, 3)};
        return hybrid_median_bits<3>(c, p, x);
    } else {
        const unsigned ll0 = from_left(l0), ll1 = from_left(l1);     // column x - 2
        const unsigned rr0 = from_right(r0), rr1 = from_right(r1);   // column x + 2
        const unsigned p[8] = {funnel(ll1, ll0, 2), funnel(l1, l0, 2), funnel(r1, r0, 2), funnel(rr1, rr0, 2),
                               w0, funnel(w1, w0, 1), funnel(w1, w0, 3), funnel(w1, w0, 4)};
        const unsigned x[8] = {ll0, rr0, funnel(l1, l0, 1), funnel(r1, r0, 1),
                               funnel(l1, l0, 3), funnel(r1, r0, 3), funnel(ll1, ll0, 4), funnel(rr1, rr0, 4)};
        return hybrid_median_bits<5>(c, p, x);
    }
}

// Row sums of the 5x5 deviation (the 5x5 first stage, Sec. 4.1): the 3x3
// row sums (s, q) of the pixel plus its neighbours two columns away.
__device__ inline void dev_row5(double zl2, double zr2, double s, double q, double &s5, double &q5) {
    s5 = s + (zl2 + zr2);
    q5 = __fma_rn(zr2, zr2, __fma_rn(zl2, zl2, q));
}
// Sums over the columns x - 1 .. x + 1 of four values, the neighbours' taken
// by the adds themselves (DPP).  Written out because the compiler folds a
// lane move into an add only within 20 instructions of it, and left six in
// seven of them as moves; a VALU result needs two wait states before a DPP
// read, which the one s_nop gives to all four.
__device__ inline void row_sums(const float (&v)[2], const float (&w)[2], float (&s)[2], float (&q)[2]) {
    asm("s_nop 1\n\t"
        "v_add_f32_dpp %0, %4, %4 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %1, %5, %5 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %2, %6, %6 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %3, %7, %7 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %0, %4, %0 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %1, %5, %1 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %2, %6, %2 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %3, %7, %3 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1"
        : "=&v"(s[0]), "=&v"(q[0]), "=&v"(s[1]), "=&v"(q[1])
        : "v"(v[0]), "v"(w[0]), "v"(v[1]), "v"(w[1]));
}
// The same over x - 2 .. x + 2: with p = v(x - 1) + v(x) and r = v(x) + v(x + 1),
// v(x) + p(x - 1) + r(x + 1).
__device__ inline void row_sums5(const float (&v)[2], const float (&w)[2], float (&s)[2], float (&q)[2]) {
    float r0, r1, r2, r3, t0, t1, t2, t3;
    asm("s_nop 1\n\t"
        "v_add_f32_dpp %4, %12, %12 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %5, %13, %13 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %6, %14, %14 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %7, %15, %15 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %8, %12, %12 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %9, %13, %13 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %10, %14, %14 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %11, %15, %15 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %0, %4, %12 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %1, %5, %13 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %2, %6, %14 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %3, %7, %15 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %0, %8, %0 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %1, %9, %1 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %2, %10, %2 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %3, %11, %3 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1"
        : "=&v"(s[0]), "=&v"(q[0]), "=&v"(s[1]), "=&v"(q[1]), "=&v"(t0), "=&v"(t1), "=&v"(t2), "=&v"(t3),
          "=&v"(r0), "=&v"(r1), "=&v"(r2), "=&v"(r3)
        : "v"(v[0]), "v"(w[0]), "v"(v[1]), "v"(w[1]));
}
// The low / high 16 bits of v as FP32.
__device__ inline float cvt_lo16(unsigned v) {
    float r;
    asm("v_cvt_f32_u32_sdwa %0, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_0" : "=v"(r) : "v"(v));
    return r;
}
__device__ inline float cvt_hi16(unsigned v) {
    float r;
    asm("v_cvt_f32_u32_sdwa %0, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1" : "=v"(r) : "v"(v));
    return r;
}

// FP32 form of the deviation test.  With e = 2^-24: a strength converted to
// FP32 errs by e relative; a 3x3 (5x5) sum of them by at most 5 e (9 e) on
// top, whatever the order, since all terms are >= 0; the sum S squared by
// 13 e (21 e), the sum Q of squares by 8 e (12 e).  thr - D = S^2 - N Q + thr
// (N = 9 or 25, D = N Q - S^2, S^2 <= N Q) then errs by at most
// (13 + 8 + 2) e N Q + 3 e thr in the two fused multiply-adds that form it
// ((21 + 12 + 2) e for 5x5; second-order terms are far below the slack).
// Where |thr - D| >= kFilter (N Q + thr), kFilter = 48 e, its sign is that of
// the exact difference, and of the FP64 evaluation, whose own error is
// 2^-29 of this bound.
//
// Codes in place of strengths: in units of the code step each strength lies
// in [code, code + 1).  sqrt(D) is N^(1/2) times the norm of the window's
// deviations from their mean, a seminorm, so the fractions move it by at most
// N^(1/2) times their own largest such norm, N^(1/2) / 2: by r = 4.5 (3x3)
// or 12.5 (5x5).  D of the codes outside [(t - r)^2, (t + r)^2], t^2 the
// threshold, decides: with centre t^2 + r^2 and half width 2 r t, that is one
// more term in the bound (t < r cannot decide from below: kCoarse keeps such
// thresholds off this form).
//
// (The strengths are integers below 2^52 here, so that nothing over- or
// underflows.  Sums that round, LOGFX_ALLOW_INEXACT, may exceed any bound or
// be tiny against it: the FP32 copies of pairs are scaled by the power of two
// zscale, which brings the largest to 2^52, and zfloor = 2^-120 is added to
// the bound for what may then underflow.  Both are neutral, 1 and 0, in
// exact calls.)
constexpr float kFilter = 48.0f / 16777216.0f;
// Below this threshold (T's square root form t above, in code steps) codes
// leave too many rows open: the half width is 9 / t of the threshold (3x3),
// 1.6 % at the line.
constexpr double kCoarse = 576.0;
struct Filter {
    float c[2], n[2];   // centre, and the bound's constant part, per mask
};
// A test of D against thr (in squared FP32 units), whose codes (r > 0) or
// strengths (r = 0) it sees.
__device__ inline void make_filter(Filter &f, int j, double thr, double r, float floor) {
    // D stays below 25^2 2^104 < 1e36: thresholds past 1e37 (infinite ones
    // too) decide as 1e37 does
    const double t2 = fmin(thr, 1e37), t = sqrt(t2);
    f.c[j] = (float)(t2 + r * r);
    f.n[j] = (float)(2.0 * r * t) + __fmaf_rn(kFilter, f.c[j], floor);
}

// How a group of rows is read: the codes alone, codes and low bits, or
// double pairs.
template <class LO> struct ZFull {
    unsigned hi;
    LO lo;
};
template <class Acc> using LowBits = typename std::conditional<std::is_same<Acc, int>::value, unsigned, uint2>::type;

// The finalize of a single image of few pass-1 tiles, by every workgroup for
// itself, with the finalize kernel's bits: integer sums on the integer path,
// and on the FP64 path its order (thread t of 256 adds tiles t and t + 256,
// threads 128 and then 64 apart are added, then a butterfly).  A launch of
// its own for it took 4.7 us of 20 at 512^2.
template <class Acc>
__device__ inline void fused_finalize(const FinalizeArgs &a, double (&thr72)[2]) {
    constexpr int NW = LaneSums<Acc>::words;
    __shared__ unsigned long long sd[NW][256];
    const ImageJob &J = a.L.one;
    const int t = threadIdx.x, l = t % kWave;
    unsigned long long v[NW];
#pragma unroll
    for (int k = 0; k < NW; ++k) v[k] = 0;   // also the double 0
    long long c[2] = {0, 0};
#pragma unroll
    for (int u = 0; u < kFuseTiles / 256; ++u) {
        const int i = t + 256 * u;
        if (i < J.ntiles1) {
#pragma unroll
            for (int k = 0; k < NW; ++k) v[k] = LaneSums<Acc>::plus(v[k], a.partials[(long long)i * kTileSums + k]);
            if (blockIdx.x == 0) {
                c[0] += a.counts[(long long)i * 2];
                c[1] += a.counts[(long long)i * 2 + 1];
            }
        }
    }
#pragma unroll
    for (int k = 0; k < NW; ++k) sd[k][t] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        v[k] = LaneSums<Acc>::plus(LaneSums<Acc>::plus(sd[k][l], sd[k][l + 128]),
                                   LaneSums<Acc>::plus(sd[k][l + 64], sd[k][l + 192]));
        if constexpr (std::is_same<Acc, int>::value) {
            v[k] = wave_total(v[k]);   // 512^2: 17.8 us with the LDS permutes below, 17.0 so
        } else {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) v[k] = LaneSums<Acc>::plus(v[k], __shfl_xor(v[k], off));
        }
    }
    long long z[2] = {0, 0};
    if (blockIdx.x == 0) {
        __shared__ long long sc[2][kTileWaves];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            c[k] = (long long)wave_sum((unsigned long long)c[k]);
            if (l == 0) sc[k][t / kWave] = c[k];
        }
        __syncthreads();
        for (int w = 0; w < kTileWaves; ++w) {
            z[0] += sc[0][w];
            z[1] += sc[1][w];
        }
    }
    double s[4];
    if constexpr (std::is_same<Acc, int>::value) {
        exact_sums(v, s);
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) s[k] = __longlong_as_double((long long)v[k]);
    }
    DevStats st;
    image_stats(a, J.img.H * J.img.W, s, z, st);
    if (blockIdx.x == 0 && t == 0) a.stats[0] = st;
    thr72[0] = st.thr72[0];
    thr72[1] = st.thr72[1];
}

// S5: with the 5x5 first stage, E_j(p) also needs the 5x5 deviation of Z_j
// above std5_max; the halo grows to 4 columns (56 output columns per wave).
// SPLIT: the form of the strengths (the integer path has only this one).
template <class Acc, int MED, bool LOOP, bool S5, bool SPLIT>
__global__ __launch_bounds__(256) void pass2z_kernel(Pass2Args<typename AccOps<Acc>::Taps> a) {
    using LO = LowBits<Acc>;
    using Full = typename std::conditional<SPLIT, ZFull<LO>, double2>::type;
    __shared__ int redc[2][8];
    constexpr int HL = S5 ? kHalo2Z5 : kHalo2Z, OW = kWave - 2 * HL, TW = tile_out_width(HL);
    constexpr int WR = S5 ? 2 : 1;        // half-height of the widest deviation window
    constexpr int NP = 2 * WR;            // rows kept from before a group

    // mixed: (gated per region) the tile's output pixels span regions, so
    // each pixel takes F or E by its own region's flag
    auto tile = [&](const int item, auto medc, const bool mixed) __attribute__((always_inline)) {
        constexpr int M = decltype(medc)::value;
        const int image = a.L.nimg == 1 ? 0 : a.L.owner2[item];
        const ImageJob J = job_of(a.L, image);
        const int H = (int)J.img.H, W = (int)J.img.W;
        const int tile = item - J.base2, tx = tile % J.tiles_x2, ty = tile / J.tiles_x2;
        const int x0 = tx * TW, y0 = ty * a.rows;
        const int Rv = __builtin_amdgcn_readfirstlane(min(a.rows, H - y0));
        const int lane = threadIdx.x & (kWave - 1);
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
        const int base = x0 + wave * OW - HL, xc = base + lane;
        const bool outc = lane >= HL && lane < HL + OW && xc < W;
        const unsigned zx = (unsigned)min(max(xc, 0), W - 1);   // the lane's column in the map

        const int lo_lane = base < 0 ? -base : 0;
        const int hi_lane = min(max(W - 1 - base, 0), kWave - 1);
        const unsigned outm = outc ? ~0u : 0u;
        // the output map: the caller's, or the scratch map of a median cascade
        uint8_t *const obase = a.out_map ? a.out_map + J.zoff : J.out;
        const long long opitch = a.out_map ? (long long)W : J.out_pitch;

        // gated per region: the region column of the lane's (clamped) column
        int rx = 0;
        if constexpr (MED < 0) {
            if (mixed) rx = min(max(xc, 0), W - 1) / a.region;
        }
        double thr72[2];
        if (MED >= 0 && !LOOP && a.fused) {
            fused_finalize<Acc>(a.fin, thr72);
        } else {
            thr72[0] = a.stats[image].thr72[0];
            thr72[1] = a.stats[image].thr72[1];
        }
        // FP32 strengths are in code steps (split) or scaled by zscale (pairs)
        const double unit[2] = {SPLIT ? __longlong_as_double((long long)(1023 - a.z.shift[0]) << 52) : a.zscale[0],
                                SPLIT ? __longlong_as_double((long long)(1023 - a.z.shift[1]) << 52) : a.zscale[1]};
        float pz[2][NP], pq[2][NP];       // the last NP rows read, z and z^2
        // E bits of the lane's column, the newest row at bit 0
        unsigned elo = 0, ehi = 0;
        int wb = 0;                       // first output row, relative to y0, of the next word to emit
        unsigned ecnt = 0, fcnt = 0;      // per lane, output pixels only

        // F of output rows y0 + wb .. y0 + wb + n - 1 (n <= 32); bit 0 of elo
        // is E row y0 + wb + n + 1 + skip
        auto emit = [&](const int n, const int skip) __attribute__((always_inline)) {
            unsigned w0 = funnel(ehi, elo, skip), w1 = ehi >> skip;
            if (lo_lane > 0) {   // columns left of the image repeat column 0
                const unsigned s0 = __builtin_amdgcn_readlane(w0, lo_lane);
                const unsigned s1 = __builtin_amdgcn_readlane(w1, lo_lane);
                w0 = lane < lo_lane ? s0 : w0;
                w1 = lane < lo_lane ? s1 : w1;
            }
            if (hi_lane < kWave - 1) {   // columns right of the image repeat column W - 1
                const unsigned s0 = __builtin_amdgcn_readlane(w0, hi_lane);
                const unsigned s1 = __builtin_amdgcn_readlane(w1, hi_lane);
                w0 = lane > hi_lane ? s0 : w0;
                w1 = lane > hi_lane ? s1 : w1;
            }
            // bit n - 1 - k of c and f: output row y0 + wb + k
            const unsigned c = funnel(w1, w0, 2);
            unsigned f;
            if constexpr (M == 0) f = c;
            else f = median_word<M>(w0, w1);
            if constexpr (MED < 0 && M != 0) {
                if (mixed) {
                    // each pixel takes F or E as its region's flag says; the
                    // word's rows cross at most one region boundary, after d
                    // of its n rows
                    const int R = a.region, yr = y0 + wb, ry = yr / R;
                    const int d = (ry + 1) * R - yr;
                    const unsigned nxt = d >= n ? 0u : (1u << (n - d)) - 1u;
                    const int *fl = a.med_flags + (long long)ry * a.reg_gx + rx;
                    const unsigned s0 = fl[0] ? ~0u : 0u;
                    const unsigned s1 = (nxt != 0u && (ry + 1) * R < H) ? (fl[a.reg_gx] ? ~0u : 0u) : 0u;
                    const unsigned sel = (s0 & ~nxt) | (s1 & nxt);
                    f = (f & sel) | (c & ~sel);
                }
            }
            const unsigned rm = (n >= 32 ? ~0u : (1u << n) - 1u) & outm;
            ecnt += __popc(c & rm);
            fcnt += __popc(f & rm);
            // a wave-uniform row address plus the lane's column
            GlobalU8 *orow = (GlobalU8 *)(obase + (long long)(y0 + wb) * opitch);
            if (outc) {
#pragma unroll 8
                for (int k = 0; k < n; ++k) {
                    orow[(unsigned)xc] = (uint8_t)__builtin_amdgcn_ubfe(f, n - 1 - k, 1);
                    orow += opitch;
                }
            }
            wb += 32;
        };
        // a wave-uniform row address plus the lane's 32-bit column
        auto load = [&](const int row, auto &v) __attribute__((always_inline)) {
            const long long at = J.zoff + (long long)min(max(row, 0), H - 1) * W;
            using V = typename std::remove_reference<decltype(v)>::type;
            if constexpr (std::is_same<V, double2>::value) {
                v = (static_cast<const double2 *>(a.z.hi) + at)[zx];
            } else if constexpr (std::is_same<V, unsigned>::value) {
                v = (static_cast<const unsigned *>(a.z.hi) + at)[zx];
            } else {
                v.hi = (static_cast<const unsigned *>(a.z.hi) + at)[zx];
                v.lo = (static_cast<const LO *>(a.z.lo) + at)[zx];
            }
        };
        auto to_f64 = [&](const Full &v, double (&z)[2]) __attribute__((always_inline)) {
            if constexpr (SPLIT) {
                restore_strengths(a.z, v.hi, v.lo, z);
            } else {
                z[0] = v.x;
                z[1] = v.y;
            }
        };
        auto to_f32 = [&](const auto &v, float (&z)[2]) __attribute__((always_inline)) {
            if constexpr (std::is_same<decltype(v), const unsigned &>::value) {
                z[0] = cvt_lo16(v);
                z[1] = cvt_hi16(v);
            } else {
                double d[2];
                to_f64(v, d);
                z[0] = (float)(d[0] * unit[0]);
                z[1] = (float)(d[1] * unit[1]);
            }
        };
        // The exact test of row y, with the operations of dev_row, dev_72var and
        // dev_row5 in their order (rolled over the masks: it is rare, and its
        // registers are the kernel's while it runs).
        auto exact = [&](const int y) __attribute__((always_inline)) {
            unsigned ej = 0;
            Full v[2 * WR + 1];   // all loads at once: one latency, not one per row
#pragma unroll
            for (int r = 0; r <= 2 * WR; ++r) load(y - WR + r, v[r]);
#pragma unroll 1
            for (int j = 0; j < 2; ++j) {
                double S3 = 0.0, Q3 = 0.0, S25 = 0.0, Q25 = 0.0;   // sums of terms >= 0: 0 + x is x
#pragma unroll
                for (int r = 0; r <= 2 * WR; ++r) {
                    double zn[2], hs, hq;
                    to_f64(v[r], zn);
                    const double z = j == 0 ? zn[0] : zn[1], zl = from_left(z), zr = from_right(z);
                    dev_row(zl, z, zr, hs, hq);
                    if (!S5 || (r >= 1 && r <= 3)) {
                        S3 += hs;
                        Q3 += hq;
                    }
                    if constexpr (S5) {
                        double ws, wq;
                        dev_row5(from_left(zl), from_right(zr), hs, hq, ws, wq);
                        S25 += ws;
                        Q25 += wq;
                    }
                }
                bool e = __fma_rn(-S3, S3, 9.0 * Q3) > thr72[j];
                if constexpr (S5) e = e && (__fma_rn(-S25, S25, 25.0 * Q25) > a.thr600[j]);
                ej |= e ? ~0u : 0u;
            }
            return ej;
        };
        // N further rows v (the first at image row y): the E bits of the N
        // rows ending WR rows above the last one
        auto group = [&](const auto &v, const int y, const Filter &f3, const Filter &f5, auto clamp)
                         __attribute__((always_inline)) {
            constexpr bool C = decltype(clamp)::value;
            constexpr int N = sizeof(v) / sizeof(v[0]);
            float z[2][NP + N], q[2][NP + N];
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int k = 0; k < NP; ++k) {
                    z[j][k] = pz[j][k];
                    q[j][k] = pq[j][k];
                }
            unsigned e[N];
            uint64_t near[N], open = 0;   // lanes whose test FP32 leaves open
#pragma unroll
            for (int k = 0; k < N; ++k) {
                if (k % 2 == 0) {
                    // two rows at a time, in this order: left to itself the
                    // compiler interleaves all of them and takes half as many
                    // registers again
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        float zn[2];
                        to_f32(v[k + i], zn);
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            z[j][NP + k + i] = zn[j];
                            q[j][NP + k + i] = zn[j] * zn[j];
                        }
                    }
                }
                float vz[2], vq[2], S[2], Q[2], d[2];
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    // column sums of three rows; rows k and k + 1 share their
                    // middle pair
                    const int m = k + WR, o = k & ~1;
                    const float pzs = z[j][o + WR] + z[j][o + WR + 1], pqs = q[j][o + WR] + q[j][o + WR + 1];
                    vz[j] = (k & 1) ? pzs + z[j][m + 1] : z[j][m - 1] + pzs;
                    vq[j] = (k & 1) ? pqs + q[j][m + 1] : q[j][m - 1] + pqs;
                }
                row_sums(vz, vq, S, Q);
                near[k] = 0;
                uint64_t n3[2], r3[2];   // S5: the lanes open, and those not rejected, by the 3x3 test
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    d[j] = __fmaf_rn(S[j], S[j], __fmaf_rn(-9.0f, Q[j], f3.c[j]));   // < 0: extracted
                    const float bound = __fmaf_rn(9.0f * kFilter, Q[j], f3.n[j]);
                    n3[j] = __ballot(fabsf(d[j]) < bound);
                    if constexpr (S5) r3[j] = __ballot(d[j] < bound);
                    else near[k] |= n3[j];
                }
                if constexpr (S5) {
                    float uz[2], uq[2];
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        uz[j] = vz[j] + (z[j][k] + z[j][k + 4]);
                        uq[j] = vq[j] + (q[j][k] + q[j][k + 4]);
                    }
                    row_sums5(uz, uq, S, Q);
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const float d5 = __fmaf_rn(S[j], S[j], __fmaf_rn(-25.0f, Q[j], f5.c[j]));
                        // open only where neither test rejects for certain
                        const float bound = __fmaf_rn(25.0f * kFilter, Q[j], f5.n[j]);
                        near[k] |= r3[j] & __ballot(d5 < bound) & (n3[j] | __ballot(fabsf(d5) < bound));
                        d[j] = fmaxf(d[j], d5);
                    }
                }
                e[k] = __float_as_uint(fminf(d[0], d[1]));   // its sign bit: E
                open |= near[k];
            }
            if (__builtin_expect(open != 0, 0)) {
                unsigned rows = 0;
#pragma unroll
                for (int k = 0; k < N; ++k) rows |= near[k] ? 1u << k : 0u;
                while (rows) {   // wave-uniform
                    const int k = __builtin_ctz(rows);
                    rows &= rows - 1;
                    const unsigned x = exact(y - WR + k);
#pragma unroll
                    for (int i = 0; i < N; ++i) e[i] = i == k ? x : e[i];
                }
            }
            ehi = funnel(ehi, elo, 32 - N);
#pragma unroll
            for (int k = 0; k < N; ++k) {
                if constexpr (C) {
                    const int ey = y - WR + k;   // the E row: below the image the last row's bit repeats
                    const unsigned b = ey > H - 1 ? elo << 31 : e[k];
                    elo = funnel(elo, b, 31);
                    if (ey == 0) elo = (elo & 1u) ? 7u : 0u;   // y0 = 0: the two rows above repeat row 0
                } else {
                    elo = funnel(elo, e[k], 31);
                }
            }
#pragma unroll
            for (int k = 0; k < NP; ++k)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    pz[j][k] = z[j][N + k];
                    pq[j][k] = q[j][N + k];
                }
        };
        // V: how the rows are read (codes, or the exact strengths)
        auto run = [&](auto vtype, const Filter &f3, const Filter &f5, auto clamp) __attribute__((always_inline)) {
            using V = decltype(vtype);
            constexpr int G = std::is_same<V, unsigned>::value ? 8 : 4;   // rows read at a time
            // rows y0 - HL .. : NP rows that only fill the windows, four that
            // give the first E bits (rows y0 - 2 .. y0 + 1), then groups of G
            V v0[NP], v4[4];
#pragma unroll
            for (int k = 0; k < NP; ++k) load(y0 - HL + k, v0[k]);
#pragma unroll
            for (int k = 0; k < 4; ++k) load(y0 - HL + NP + k, v4[k]);
#pragma unroll
            for (int k = 0; k < NP; ++k) {
                float zn[2];
                to_f32(v0[k], zn);
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    pz[j][k] = zn[j];
                    pq[j][k] = zn[j] * zn[j];
                }
            }
            group(v4, y0 - HL + NP, f3, f5, clamp);
            int r = 0;
            for (; r < Rv; r += G) {
                V v[G];
#pragma unroll
                for (int k = 0; k < G; ++k) load(y0 - HL + NP + 4 + r + k, v[k]);
                group(v, y0 - HL + NP + 4 + r, f3, f5, clamp);
                if (r + G - wb == 32 && wb + 32 <= Rv) emit(32, 0);
            }
            if (wb < Rv) emit(Rv - wb, r - Rv);
        };
        // the E rows y0-2 .. y0+Rv+1 the output uses lie inside the image:
        // no row clamping of the extracted bits
        const bool inner = y0 - 2 >= 0 && y0 + Rv + 1 <= H - 1;
        double t3[2], t5[2];
        bool coarse = !SPLIT;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            t3[j] = thr72[j] * (unit[j] * unit[j]);
            t5[j] = a.thr600[j] * (unit[j] * unit[j]);
            coarse |= t3[j] < kCoarse * kCoarse;
            if constexpr (S5) coarse |= t5[j] < kCoarse * kCoarse * 7.7;   // its half width is 25 / t
        }
        auto with = [&](auto vtype, const double r3, const double r5, const float floor) __attribute__((always_inline)) {
            Filter f3, f5;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                make_filter(f3, j, t3[j], r3, floor);
                make_filter(f5, j, t5[j], r5, floor);
            }
            if (inner) run(vtype, f3, f5, bool_c<false>{});
            else run(vtype, f3, f5, bool_c<true>{});
        };
        if constexpr (SPLIT) {
            if (coarse) with(Full{}, 0.0, 0.0, 0.0f);
            else with(0u, 4.5, 12.5, 0.0f);
        } else {
            with(Full{}, 0.0, 0.0, a.zfloor);
        }

        const int w = threadIdx.x / kWave;
        const int es = wave_sum((int)ecnt), fs = wave_sum((int)fcnt);
        if (lane == 0) {
            redc[0][w] = es;
            redc[1][w] = fs;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            int s0 = 0, s1 = 0;
            for (int k = 0; k < (int)(blockDim.x / kWave); ++k) {
                s0 += redc[0][k];
                s1 += redc[1][k];
            }
            a.counts[(long long)item * 2] = s0;
            a.counts[(long long)item * 2 + 1] = s1;
        }
        __syncthreads();   // the reduction buffer is reused by the next tile
    };
    for_each_tile<LOOP>(a.L.total2, [&](const int item) __attribute__((always_inline)) {
        if constexpr (MED >= 0) {
            tile(item, int_c<MED>{}, false);
        } else {   // gated: the median of each image (or region) as its flag says
            const int image = a.L.nimg == 1 ? 0 : a.L.owner2[item];
            int flag;
            bool mixed = false;
            if (a.region > 0) {
                // a tile inside one region takes that region's flag as a whole
                const ImageJob J = job_of(a.L, image);
                const int t = item - J.base2, tx = t % J.tiles_x2, ty = t / J.tiles_x2;
                const int x0 = tx * TW, y0 = ty * a.rows;
                const int x1 = min(x0 + TW, (int)J.img.W) - 1, y1 = min(y0 + a.rows, (int)J.img.H) - 1;
                const int R = a.region;
                mixed = x0 / R != x1 / R || y0 / R != y1 / R;
                flag = a.med_flags[(y0 / R) * a.reg_gx + x0 / R];
            } else {
                flag = a.med_flags[image];
            }
            if (mixed || flag) tile(item, int_c<-MED>{}, mixed);
            else tile(item, int_c<0>{}, false);
        }
    });
}

// One further level of the median cascade: reads a 0/1 map (clamp-to-edge
// rows and columns, which is how every level reads its input), collects
// each lane's column in words as pass 2 does, and writes the hybrid median
// (or, for an image the gate leaves unsmoothed, the map itself).
template <int HL, int M>
__global__ __launch_bounds__(256) void median_level_kernel(LevelArgs a) {
    __shared__ int redc[8];
    constexpr int OW = kWave - 2 * HL, TW = tile_out_width(HL);
    constexpr int G = 6;
    const int item = blockIdx.x;
    const int image = a.L.nimg == 1 ? 0 : a.L.owner2[item];
    const ImageJob J = job_of(a.L, image);
    const int H = (int)J.img.H, W = (int)J.img.W;
    const int tile = item - J.base2, tx = tile % J.tiles_x2, ty = tile / J.tiles_x2;
    const int x0 = tx * TW, y0 = ty * a.rows, Rv = min(a.rows, H - y0);
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int xc = x0 + wave * OW - HL + lane;
    const bool outc = lane >= HL && lane < HL + OW && xc < W;
    const unsigned outm = outc ? ~0u : 0u;
    const bool copy = a.med_flags && !a.med_flags[image];
    uint8_t *const scr = a.scratch + J.zoff;
    const uint8_t *const src = a.from_scratch ? scr : J.out;
    uint8_t *const dst = a.from_scratch ? J.out : scr;
    const long long spitch = a.from_scratch ? (long long)W : J.out_pitch;
    const long long dpitch = a.from_scratch ? J.out_pitch : (long long)W;
    const uint8_t *const scol = src + min(max(xc, 0), W - 1);

    // bit k of elo (of ehi): input row y0 - 2 + wb + k (+ 32)
    unsigned elo = 0, ehi = 0, fcnt = 0;
    int wb = 0;
    const int nrows = Rv + 4;   // input rows y0 - 2 .. y0 + Rv + 1
    auto emit = [&](const int n) __attribute__((always_inline)) {
        unsigned f = funnel(ehi, elo, 2);
        if (!copy) f = M == 3 ? median_word<3>(elo, ehi) : median_word<5>(elo, ehi);
        fcnt += __popc(f & (n >= 32 ? ~0u : (1u << n) - 1u) & outm);
        GlobalU8 *orow = (GlobalU8 *)(dst + (long long)(y0 + wb) * dpitch);
        if (outc) {
#pragma unroll 8
            for (int k = 0; k < n; ++k) {
                orow[(unsigned)xc] = (uint8_t)__builtin_amdgcn_ubfe(f, k, 1);
                orow += dpitch;
            }
        }
        elo = ehi;
        ehi = 0;
        wb += 32;
    };
    auto put = [&](const int b, const uint8_t v) __attribute__((always_inline)) {
        const int p = b - wb;
        const unsigned m = v != 0 ? ~0u : 0u;
        elo |= m & (p < 32 ? 1u << p : 0u);
        ehi |= m & (p >= 32 ? 1u << (p - 32) : 0u);
    };
    int b0 = 0;
    for (; b0 + G <= nrows; b0 += G) {
        uint8_t q[G];
#pragma unroll
        for (int k = 0; k < G; ++k) q[k] = scol[(long long)min(max(y0 - 2 + b0 + k, 0), H - 1) * spitch];
#pragma unroll
        for (int k = 0; k < G; ++k) put(b0 + k, q[k]);
        if (b0 + G - wb >= 36) emit(32);   // rows wb .. wb + 35 present
    }
    for (; b0 < nrows; ++b0) put(b0, scol[(long long)min(max(y0 - 2 + b0, 0), H - 1) * spitch]);
    while (wb < Rv) emit(min(32, Rv - wb));

    if (a.counts) {
        const int fs = wave_sum((int)fcnt);
        if (lane == 0) redc[threadIdx.x / kWave] = fs;
        __syncthreads();
        if (threadIdx.x == 0) {
            int t = 0;
            for (int k = 0; k < (int)(blockDim.x / kWave); ++k) t += redc[k];
            a.counts[(long long)item * 2 + 1] = t;
        }
    }
}

template <class Acc, int MED, bool S5, bool SPLIT>
hipError_t p2z5s(const Pass2Args<typename AccOps<Acc>::Taps> &a, int grid, hipStream_t s, int *max_grid) {
    constexpr bool CAN_LOOP = MED >= 0;   // gated variants run one tile per workgroup
    if (max_grid) return occupancy(pass2z_kernel<Acc, MED, CAN_LOOP, S5, SPLIT>, 0, max_grid);
    if (!CAN_LOOP || grid >= a.L.total2)
        hipLaunchKernelGGL((pass2z_kernel<Acc, MED, false, S5, SPLIT>), dim3(a.L.total2), dim3(kTileWaves * kWave), 0, s, a);
    else
        hipLaunchKernelGGL((pass2z_kernel<Acc, MED, CAN_LOOP, S5, SPLIT>), dim3(grid), dim3(kTileWaves * kWave), 0, s, a);
    return hipGetLastError();
}
template <class Acc, int MED, bool S5>
hipError_t p2z5(const Pass2Args<typename AccOps<Acc>::Taps> &a, int grid, hipStream_t s, int *max_grid) {
    if constexpr (!std::is_same<Acc, int>::value) {
        if (!a.z.split) return p2z5s<Acc, MED, S5, false>(a, grid, s, max_grid);
    }
    return p2z5s<Acc, MED, S5, true>(a, grid, s, max_grid);
}
template <class Acc, int MED>
hipError_t p2z(const Pass2Args<typename AccOps<Acc>::Taps> &a, int grid, hipStream_t s, int *max_grid) {
    return a.std5 ? p2z5<Acc, MED, true>(a, grid, s, max_grid) : p2z5<Acc, MED, false>(a, grid, s, max_grid);
}

template <class Acc>
hipError_t p2z_any(const Pass2Args<typename AccOps<Acc>::Taps> &a, int grid, hipStream_t s, int *max_grid) {
    if (a.med_flags) return a.median_size == 3 ? p2z<Acc, -3>(a, grid, s, max_grid) : p2z<Acc, -5>(a, grid, s, max_grid);
    if (!a.smooth) return p2z<Acc, 0>(a, grid, s, max_grid);
    return a.median_size == 3 ? p2z<Acc, 3>(a, grid, s, max_grid) : p2z<Acc, 5>(a, grid, s, max_grid);
}

}  // namespace kern

hipError_t launch_pass2z_i(const Pass2Args<OrbitTapsI> &a, int grid, hipStream_t s, int *max_grid) {
    return kern::p2z_any<int>(a, grid, s, max_grid);
}
hipError_t launch_pass2z_d(const Pass2Args<OrbitTapsD> &a, int grid, hipStream_t s, int *max_grid) {
    return kern::p2z_any<double>(a, grid, s, max_grid);
}
hipError_t launch_median_level(const LevelArgs &a, int halo, hipStream_t s) {
    const dim3 grid(a.L.total2), block(kTileWaves * kWave);
    if (halo == kHalo2Z5) {
        if (a.median_size == 3) hipLaunchKernelGGL((kern::median_level_kernel<kHalo2Z5, 3>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((kern::median_level_kernel<kHalo2Z5, 5>), grid, block, 0, s, a);
    } else {
        if (a.median_size == 3) hipLaunchKernelGGL((kern::median_level_kernel<kHalo2Z, 3>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((kern::median_level_kernel<kHalo2Z, 5>), grid, block, 0, s, a);
    }
    return hipGetLastError();
}

}  // namespace logfx
