// Box-stencil sweep on the matrix cores (MFMA) with split BF16 / FP16 operands.
//
// The paper maps a one-dimensional stencil onto an outer-product matrix unit by
// multiplying the input rows with a zero-padded coefficient column (Sec. IV-A);
// written as a matrix product this is  out = T * in_window  with T a banded
// Toeplitz matrix.  Here the Toeplitz block of one dz is two-dimensional: its 16
// rows are the outputs of a 4 x 4 tile of (y, x), its columns the tile's window of
// (4 + 2r) x 12 input cells,
//     T_dz[(my, mx)][(y', x')] = c[dz][y' - r - my][x' - 4 - mx]   (zero outside the box),
// and the 16 columns of the other operand are 16 such tiles side by side along x:
//     D(4 x 4 cells, 16 x-blocks) += T_dz * In_{z+dz}(window of each block).
// A fraction (2r+1)^2 / (12 (4 + 2r)) of the products is useful (56 % at radius 4), where
// a one-dimensional block of 16 x-outputs per dy leaves (2r+1) / 24 (37 %): 126 against
// 189 MFMAs of 16 x 16 x 32 per 256 outputs at radius 4, 84 against 126 at radius 3, which
// took the 512^3 sweep from 1090 to 742 us and from 711 to 524.
//
// FP32 accuracy from 16-bit multipliers: every operand x is split as x = hi + lo
// (BF16: hi = RN(x), lo = RN(x - hi); FP16: the same after scaling by a power of
// two that keeps the largest |x| of the planes in hand below 2^14), and each product is
// formed as hi*hi + hi*lo + lo*hi with FP32 accumulation (lo*lo is dropped, except
// where a step has slots to spare).  The BF16X1 variant keeps hi*hi only.
//
// Work split.  A block of 8 waves owns a 64 x (32 NT) output tile of the (x, y) plane and
// streams a chunk of z, PZ input planes per step.  All Toeplitz fragments (hi and lo, every
// dz) are built once per block into LDS.  The planes of a step sit in LDS as 16-bit hi and
// lo parts, the 4-cell words of two neighbouring rows side by side ("pair words"), so that
// a lane's eight K values are one 16-byte read and the 16 lanes of a group read 256
// consecutive bytes.  Each wave owns NT tiles of 64 x 4 outputs; per K step it loads the
// input fragments once and reuses them for every dz and product (input plane z' feeds
// output z' - dz), and each Toeplitz fragment it loads feeds NT * PZ tiles.  A wave keeps
// 2r + PZ output planes of accumulators in flight; after each step the PZ oldest are
// complete, are written, and the window shifts.  The next step's planes are requested a
// whole step ahead and split halfway through it.  (step, dz) units that feed no output of
// the chunk are skipped, which matters where chunks are short.
//
// Cells that are not finite.  A block's window holds cells that an output's box does not, with
// zero weights, and 0 * NaN or 0 * Inf spoils that output.  So an output that is not finite is
// formed again from the cells of its box alone, in FP32: the check is one FMA an output (512^3:
// 0 to 1 %), and only what such a cell spoilt pays more.  (A bit map of such cells in LDS, with
// zeros in their place in the products, cost 3 % of every sweep and 10 % of short ones.)
//
// The kernel is bound by the matrix cores: at 512^3, radius 4, it issues 1.46 PFLOP/s of
// MFMA work (a large BF16 matrix product reaches 1.2 PFLOP/s on the same card).
#include <hip/hip_runtime.h>

#include "mms_internal.h"

namespace mms {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

// Launch shape per radius: 8 waves per block (two per SIMD, so that one wave's loads,
// splits and stores run beside the other's MFMAs), NT tiles of 64 x 4 outputs per wave
// along y, PZ input planes per step.  Every Toeplitz fragment read from LDS feeds
// NT * PZ tiles, and these reads are what LDS has to carry: at NT * PZ = 2 they take 84 %
// of its cycles at radius 4, at 4 less than half.  The product 4 as one row of tiles and
// four planes keeps the block's tile at 64 x 32 (more blocks for small grids, longer z
// chunks for large ones).  Measured, BF16X3, 512^3 / 300 x 301 x 290, us (NT, PZ): radius 4
// 742 / 158 (1, 4), 791 / 176 (2, 2), 768 / 172 (2, 1); radius 3 524 (1, 4), 529 (2, 2),
// 561 (2, 1).  Up to radius 2 the fragments are few enough that the compiler keeps them in
// registers and spills at (1, 4) (1188 at radius 2); (2, 2) runs at 343.
template <int R>
struct MCfg {
    static constexpr int NW = 8;
    static constexpr int NT = R >= 3 ? 1 : 2;
    static constexpr int PZ = R >= 3 ? 4 : 2;
};

struct MfmaArgs {
    Geom g;
    float c[729];      // [dz][dy][dx]
    int cexp;          // FP16 path: the weights are scaled by 2^cexp
};

// FP32 -> BF16 with round to nearest even (one v_cvt_pk_bf16_f32 on gfx950).
__device__ __forceinline__ uint16_t bf16_rn(float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); }
__device__ __forceinline__ float bf16_f(uint16_t h) {
    return __builtin_bit_cast(float, (uint32_t)h << 16);
}

template <int PREC>
__device__ __forceinline__ void split(float x, float scale, uint16_t &hi, uint16_t &lo) {
    if constexpr (PREC == MMS_FP16X3S) {
        const float xs = x * scale;
        const _Float16 h = (_Float16)xs;
        const _Float16 l = (_Float16)(xs - (float)h);
        hi = __builtin_bit_cast(uint16_t, h);
        lo = __builtin_bit_cast(uint16_t, l);
    } else {
        hi = bf16_rn(x);
        lo = bf16_rn(x - bf16_f(hi));
    }
}

template <int PREC>
__device__ __forceinline__ floatx4 mfma(const uint4 &a, const uint4 &b, floatx4 c) {
    if constexpr (PREC == MMS_FP16X3S) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a),
                                                      __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    } else {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
}

// K layout of one dz: 16-byte words of LDS, each holding 4 x-cells of two neighbouring
// rows ("pair words").  The window of a 4 x 4 output tile is 4 + 2r rows by 12 cells, so
// NP = 3 (2 + r) pair words; one MFMA step takes four of them (one per lane group).
template <int R>
struct Shape {
    static constexpr int NW = MCfg<R>::NW, NT = MCfg<R>::NT, PZ = MCfg<R>::PZ;
    static constexpr int BXT = 64;                  // 16 x-blocks of 4 cells (N)
    static constexpr int BYT = 4 * NT * NW;         // 4 rows per tile (M = 4 x 4 cells)
    static constexpr int Q = 2 * R + 1;             // output planes in flight, dz values
    static constexpr int NP = 3 * (2 + R);          // pair words of a tile's window
    // whole steps of four words; three left-over words take a whole step too
    static constexpr int NCH = NP % 4 == 3 ? NP / 4 + 1 : NP / 4;
    static constexpr int REM = NP % 4 == 3 ? 0 : NP % 4;   // 0, 1 or 2 words left over
    // A fragments per dz: hi and lo of each step, and those of the left-over words
    // (one word: its three products share one step; two words: two steps)
    static constexpr int NA = 2 * NCH + REM;
    static constexpr int NPR = (BYT + 2 * R) / 2;   // LDS row pairs of a plane
    static constexpr int C4 = BXT / 4 + 2;          // words per row pair
    static constexpr int NS = NPR * C4;             // pair words per plane
    static constexpr int NSK = (PZ * NS + 64 * NW - 1) / (64 * NW);
};

template <int R>
struct Smem {
    using S = Shape<R>;
    static constexpr int PZ = S::PZ;
    uint4 afrag[S::Q][S::NA][64];   // [dz][fragment][lane]
    uint4 d[2][PZ][S::NPR][S::C4];  // hi and lo parts of the planes
    float smax[S::NW];
};

template <int R, int PREC>
__global__ void __launch_bounds__(64 * MCfg<R>::NW) box_mfma_kernel(MfmaArgs a) {
    using S = Shape<R>;
    constexpr int BXT = S::BXT, BYT = S::BYT;
    constexpr int Q = S::Q, NCH = S::NCH, C4 = S::C4, NS = S::NS, NSK = S::NSK;
    constexpr int REM = S::REM, NP = S::NP, NW = S::NW, NT = S::NT, PZ = S::PZ;
    constexpr int NTH = 64 * NW;
    constexpr bool SPLIT3 = PREC != MMS_BF16X1;
    __shared__ Smem<R> sm;

    const Geom &g = a.g;
    int b = mms_xcd_remap(blockIdx.x, gridDim.x);
    const int txi = b % g.ntx;
    b /= g.ntx;
    const int tyi = b % g.nty;
    const int zci = b / g.nty;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int xt = txi * BXT, yt = tyi * BYT;
    const int zb = zci * g.zchunk;
    const int ze = min(zb + g.zchunk, g.nz);
    const int nx4 = (g.nx + 3) & ~3;
    const int ylim = g.ny + R;   // rows beyond the stencil's reach stay out of the products
    const int64_t sy = g.sy, sz = g.sz;

    // staging items: the two float4 of a pair word
    int s_z[NSK];
    int64_t s_off[NSK];
    bool s_ok[NSK][2];
#pragma unroll
    for (int k = 0; k < NSK; ++k) {
        const int i = tid + k * NTH;
        const int rp = i % NS / C4, col = i % NS % C4;
        const int yy = yt - R + 2 * rp, xx = xt - 4 + 4 * col;
        s_z[k] = i / NS;
        s_ok[k][0] = (i < PZ * NS) && (yy < ylim) && (xx <= nx4);
        s_ok[k][1] = (i < PZ * NS) && (yy + 1 < ylim) && (xx <= nx4);
        s_off[k] = (int64_t)yy * sy + xx;
    }
    const int z_first = zb - R, z_last = ze + R;

    const float cscale = (PREC == MMS_FP16X3S) ? ldexpf(1.0f, a.cexp) : 1.0f;

    // Toeplitz fragments of every dz into LDS (A operand), from a copy of the weights that
    // borrows the plane buffer
    float *cl = reinterpret_cast<float *>(&sm.d[0][0][0][0]);
    static_assert(sizeof(sm.d) >= Q * Q * Q * sizeof(float));
    for (int i = tid; i < Q * Q * Q; i += NTH) cl[i] = a.c[i];
    __syncthreads();
    for (int item = tid; item < Q * S::NA * 64; item += NTH) {
        const int l = item & 63, f = (item >> 6) % S::NA, dz = (item >> 6) / S::NA;
        const int m = l & 15, grp = l >> 4;
        const int my = m >> 2, mx = m & 3;
        // the word and part (hi or lo) of this lane group's slot
        int w, part;
        bool on = true;
        if (f < 2 * NCH) {
            w = 4 * (f >> 1) + grp;
            part = f & 1;
        } else if (REM == 1) {          // slots hi*hi, hi*lo, lo*hi
            w = 4 * NCH;
            part = grp == 2;
            on = SPLIT3 ? grp < 3 : grp == 0;
        } else {                        // slots hi, hi of the data, lo, lo of the data
            w = 4 * NCH + (grp & 1);
            part = f - 2 * NCH;
            on = SPLIT3 || grp < 2;
        }
        uint32_t o[4];
#pragma unroll
        for (int j2 = 0; j2 < 4; ++j2) {
            uint16_t p[2];
#pragma unroll
            for (int j1 = 0; j1 < 2; ++j1) {
                const int j = 2 * j2 + j1;
                const int dy = 2 * (w / 3) + (j >> 2) - R - my;
                const int dx = 4 * (w % 3) + (j & 3) - 4 - mx;
                float v = 0.f;
                if (on && w < NP && dy >= -R && dy <= R && dx >= -R && dx <= R)
                    v = cl[(dz * Q + dy + R) * Q + dx + R];
                uint16_t h, lo;
                split<PREC>(v, cscale, h, lo);
                p[j1] = part ? lo : h;
            }
            o[j2] = p[0] | (uint32_t)p[1] << 16;
        }
        sm.afrag[dz][f][l] = make_uint4(o[0], o[1], o[2], o[3]);
    }

    float4 stage[NSK][2];
    uint4 shi[NSK], slo[NSK];   // the staged plane split into packed 16-bit hi and lo parts
    auto load_plane = [&](int z) {
#pragma unroll
        for (int k = 0; k < NSK; ++k) {
            const float *p = g.in0 + (int64_t)min(z + s_z[k], z_last - 1) * sz + s_off[k];
#pragma unroll
            for (int j = 0; j < 2; ++j)
                stage[k][j] = guarded_load(p + j * sy, s_ok[k][j], g.in0);
        }
    };
    // FP16 path: one power-of-two scale per block and step, from the largest finite |x| of the
    // step's planes and of the earlier ones that still feed a sum (the last 2r), so that it falls
    // with the amplitudes as well as it rises.  Where it changes, the accumulators, which hold
    // sums in units of 2^-(dexp + cexp), are rescaled: exactly, and without overflow, since all
    // their terms lie within the window.  (A scale that only rises keeps few bits, or none, of
    // quiet planes after a loud one: amplitudes that fall by 0.66 a plane over a chunk of 64 had
    // errors of 0.3 of their own plane.)  A scan of the block's whole window before the first
    // product would cost a second read of the grid (0.15 of 0.9 ms at 512^3, radius 4).
    // The scales are held as exponents: an output leaves by one exact multiplication with
    // 2^-(data + weights), where the product of two factors could overflow or underflow on the way.
    constexpr int NPREV = (2 * R + PZ - 1) / PZ;   // earlier steps in the window
    int dexp = 0, dnext = 0;
    float mprev[NPREV];   // their maxima, the latest first
#pragma unroll
    for (int i = 0; i < NPREV; ++i) mprev[i] = 0.f;
    auto scale_step = [&]() {
        float m = 0.f;
#pragma unroll
        for (int k = 0; k < NSK; ++k)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const float4 v = stage[k][j];
                const float e[4] = {fabsf(v.x), fabsf(v.y), fabsf(v.z), fabsf(v.w)};
#pragma unroll
                for (int i = 0; i < 4; ++i) m = e[i] <= 3.402823466e38f ? fmaxf(m, e[i]) : m;
            }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
        if (lane == 0) sm.smax[wave] = m;
        __syncthreads();
        m = sm.smax[0];
#pragma unroll
        for (int w = 1; w < NW; ++w) m = fmaxf(m, sm.smax[w]);
        float wmax = m;
#pragma unroll
        for (int i = NPREV - 1; i >= 0; --i) {
            wmax = fmaxf(wmax, mprev[i]);
            mprev[i] = i > 0 ? mprev[i - 1] : m;
        }
        if (wmax > 0.f) {   // (zeros fit any scale)
            int e;
            frexpf(wmax, &e);  // wmax = f 2^e, 0.5 <= f < 1
            dnext = min(14 - e, 127);
        }
    };
    // the split runs while the previous step's MFMAs execute; only the LDS writes wait
    // for the barrier that frees the plane buffer
    auto split_plane = [&]() {
        const float sc = PREC == MMS_FP16X3S ? ldexpf(1.0f, dnext) : 1.0f;
#pragma unroll
        for (int k = 0; k < NSK; ++k) {
            uint32_t h[4], l[4];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                uint16_t h0, l0, h1, l1, h2, l2, h3, l3;
                split<PREC>(stage[k][j].x, sc, h0, l0);
                split<PREC>(stage[k][j].y, sc, h1, l1);
                split<PREC>(stage[k][j].z, sc, h2, l2);
                split<PREC>(stage[k][j].w, sc, h3, l3);
                h[2 * j] = h0 | (uint32_t)h1 << 16;
                h[2 * j + 1] = h2 | (uint32_t)h3 << 16;
                l[2 * j] = l0 | (uint32_t)l1 << 16;
                l[2 * j + 1] = l2 | (uint32_t)l3 << 16;
            }
            shi[k] = make_uint4(h[0], h[1], h[2], h[3]);
            slo[k] = make_uint4(l[0], l[1], l[2], l[3]);
        }
    };
    auto write_plane = [&]() {
#pragma unroll
        for (int k = 0; k < NSK; ++k) {
            const int i = tid + k * NTH;
            if (i < PZ * NS) {
                (&sm.d[0][0][0][0])[i] = shi[k];
                if (SPLIT3) (&sm.d[1][0][0][0])[i] = slo[k];
            }
        }
    };

    // The four outputs from (x, y, zo) on from their boxes alone.  A cell or weight whose hi part
    // is NaN or Inf makes an output NaN in the split forms (Inf - Inf in the lo part).
    auto box_sums = [&](int x, int y, int zo, float *s) {
        auto factor = [](float v) -> float {   // what a product of the variant takes v for
            const float h = PREC == MMS_FP16X3S ? v : bf16_f(bf16_rn(v));
            return !SPLIT3 ? h : fabsf(h) <= 3.402823466e38f ? v : __builtin_nanf("");
        };
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = 0.f;
#pragma unroll 1
        for (int dz = 0; dz < Q; ++dz) {
            if (s[0] != s[0] && s[1] != s[1] && s[2] != s[2] && s[3] != s[3]) break;
            const float *p = g.in0 + (int64_t)(zo + dz - R) * sz + (int64_t)(y - R) * sy + x;
#pragma unroll 3
            for (int dy = 0; dy < Q; ++dy, p += sy) {
                float w[12];
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const float4 v = *reinterpret_cast<const float4 *>(p - 4 + 4 * i);
                    w[4 * i] = factor(v.x);
                    w[4 * i + 1] = factor(v.y);
                    w[4 * i + 2] = factor(v.z);
                    w[4 * i + 3] = factor(v.w);
                }
#pragma unroll
                for (int dx = -R; dx <= R; ++dx) {
                    const float f = factor(a.c[(dz * Q + dy) * Q + dx + R]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) s[e] = fmaf(f, w[4 + e + dx], s[e]);
                }
            }
        }
    };

    // acc[k][t] holds the partial sum of output plane zi - R + k
    constexpr int NQ = Q + PZ - 1;
    floatx4 acc[NQ][NT];
#pragma unroll
    for (int s = 0; s < NQ; ++s)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[s][t] = floatx4{0.f, 0.f, 0.f, 0.f};

    const int n = lane & 15, grp = lane >> 4;   // B fragment: x-block n, word slot grp
    const int wrow = 4 * NT * wave;             // the wave's first row in the tile

    // word offsets of the lane's B fragments: step ch, and the left-over words
    const uint4 *bbase = &sm.d[0][0][wrow / 2][n];
    int boff[NCH], brem = 0;
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
        const int w = 4 * ch + grp < NP ? 4 * ch + grp : 0;   // a zero-weight slot reads word 0
        boff[ch] = (w / 3) * C4 + w % 3;
    }
    if constexpr (REM > 0) {
        const int w = 4 * NCH + (REM == 2 ? grp & 1 : 0);
        const bool lo = SPLIT3 && (REM == 2 ? grp >= 2 : grp == 1);
        brem = (w / 3) * C4 + w % 3 + (lo ? PZ * S::NS : 0);
    }

    load_plane(z_first);
    if constexpr (PREC == MMS_FP16X3S) scale_step();
    split_plane();
    dexp = dnext;
    __syncthreads();   // the weights' copy is read
    write_plane();
    if (z_first + PZ < z_last) load_plane(z_first + PZ);
    __syncthreads();

    uint4 bh[PZ][NT], bl[PZ][NT];
    auto load_b = [&](int ch) {
#pragma unroll
        for (int j = 0; j < PZ; ++j)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const uint4 *p = bbase + (ch < NCH ? boff[ch] : brem) + 2 * t * C4 + j * NS;
                bh[j][t] = *p;
                if (SPLIT3 && ch < NCH) bl[j][t] = p[PZ * NS];
            }
    };
    // units: (step, dz) pairs, then the left-over words of every dz
    constexpr int NU = Q * (NCH + (REM > 0));
    constexpr int PF = 2;   // A fragments one unit ahead
    uint4 ah[PF], al[PF];
    auto load_a = [&](int u, int slot) {
        const int ch = u / Q, dzi = u % Q;
        ah[slot] = sm.afrag[dzi][2 * ch][lane];
        if (ch < NCH ? SPLIT3 : REM == 2 && SPLIT3) al[slot] = sm.afrag[dzi][2 * ch + 1][lane];
    };

    for (int zi = z_first; zi < z_last; zi += PZ) {
        // keeps the fragment reads in the loop (hoisted out of it they spill)
        asm volatile("" ::: "memory");
        load_b(0);
#pragma unroll
        for (int u = 0; u < PF - 1; ++u) load_a(u, u);
        const int dlo = __builtin_amdgcn_readfirstlane(zi - ze + R + 1);
        const int dhi = __builtin_amdgcn_readfirstlane(zi - zb + R + PZ - 1);
        auto unit = [&](int u) {
            const int ch = u / Q, dzi = u % Q;
            if (dzi == 0 && u > 0) load_b(ch);
            if (u + PF - 1 < NU) load_a(u + PF - 1, (u + PF - 1) % PF);
            // keep the requests above this unit's MFMAs (the scheduler would sink them)
            __builtin_amdgcn_sched_barrier(0);
            const uint4 &ahi = ah[u % PF];
            const uint4 &alo = al[u % PF];
            // input plane zi + j feeds output zi + j - dz (dz = dzi - R), held in
            // acc[Q - 1 - dzi + j]; units that feed no output of the chunk are skipped
            if (dzi >= dlo && dzi <= dhi) {
#pragma unroll
                for (int j = 0; j < PZ; ++j)
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        acc[Q - 1 - dzi + j][t] = mfma<PREC>(ahi, bh[j][t], acc[Q - 1 - dzi + j][t]);
                if (SPLIT3 && ch < NCH) {
#pragma unroll
                    for (int j = 0; j < PZ; ++j)
#pragma unroll
                        for (int t = 0; t < NT; ++t)
                            acc[Q - 1 - dzi + j][t] = mfma<PREC>(ahi, bl[j][t], acc[Q - 1 - dzi + j][t]);
                }
                if (SPLIT3 && (ch < NCH || REM == 2)) {
#pragma unroll
                    for (int j = 0; j < PZ; ++j)
#pragma unroll
                        for (int t = 0; t < NT; ++t)
                            acc[Q - 1 - dzi + j][t] = mfma<PREC>(alo, bh[j][t], acc[Q - 1 - dzi + j][t]);
                }
            }
        };
#pragma unroll
        for (int u = 0; u < NU / 2; ++u) unit(u);
        if (zi + PZ < z_last) {   // the next step's planes
            if constexpr (PREC == MMS_FP16X3S) scale_step();
            split_plane();
        }
#pragma unroll
        for (int u = NU / 2; u < NU; ++u) unit(u);
        // output planes zi - R .. zi - R + PZ - 1 are complete (those outside [zb, ze) are dropped)
        const int oexp = -(dexp + a.cexp);
        const int x = xt + 4 * n;
        float spoilt = 0.f;   // NaN if one of the lane's sums is not finite
#pragma unroll
        for (int j = 0; j < PZ; ++j) {
            const int zo = zi - R + j;
            if (zo < zb || zo >= ze) continue;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int y = yt + wrow + 4 * t + grp;
                if (y < g.ny && x < g.nx) {
                    float *po = g.out0 + (int64_t)zo * sz + (int64_t)y * sy + x;
                    const floatx4 s = acc[j][t];
#pragma unroll
                    for (int e = 0; e < 4; ++e) spoilt = fmaf(s[e], 0.f, spoilt);
                    floatx4 o = s;
                    if constexpr (PREC == MMS_FP16X3S) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[e] = ldexpf(s[e], oexp);
                    }
                    if (x + 3 < g.nx) {
                        *reinterpret_cast<floatx4 *>(po) = o;
                    } else {
                        if (x + 0 < g.nx) po[0] = o[0];
                        if (x + 1 < g.nx) po[1] = o[1];
                        if (x + 2 < g.nx) po[2] = o[2];
                    }
                }
            }
        }
        if (__builtin_expect(spoilt != 0.f, 0)) {
#pragma unroll 1
            for (int i = 0; i < PZ * NT; ++i) {
                const int zo = zi - R + i / NT, y = yt + wrow + 4 * (i % NT) + grp;
                if (zo < zb || zo >= ze || y >= g.ny || x >= g.nx) continue;
                float *po = g.out0 + (int64_t)zo * sz + (int64_t)y * sy + x;
                bool on[4];   // the outputs to form again
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    on[e] = x + e < g.nx && !(fabsf(po[x + e < g.nx ? e : 0]) <= 3.402823466e38f);
                if (!(on[0] || on[1] || on[2] || on[3])) continue;
                float s[4];
                box_sums(x, y, zo, s);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (on[e]) po[e] = s[e];
            }
        }
#pragma unroll
        for (int s = 0; s < NQ; ++s)
#pragma unroll
            for (int t = 0; t < NT; ++t)
                acc[s][t] = s + PZ < NQ ? acc[s + PZ][t] : floatx4{0.f, 0.f, 0.f, 0.f};
        if (PREC == MMS_FP16X3S && dnext != dexp) {
#pragma unroll
            for (int s = 0; s < NQ; ++s)
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[s][t][e] = ldexpf(acc[s][t][e], dnext - dexp);
            dexp = dnext;
        }
        __syncthreads();   // every wave is done with plane zi
        if (zi + PZ < z_last) {
            write_plane();
            if (zi + 2 * PZ < z_last) load_plane(zi + 2 * PZ);   // requested a whole step ahead
        }
        __syncthreads();
    }
}

template <int R, int PREC>
int launch_rp(const float *in, float *out, const mms_grid *gd, const float *coeffs, hipStream_t s) {
    constexpr int Q = 2 * R + 1;
    using S = Shape<R>;
    MfmaArgs a{};
    Geom &g = a.g;
    g.H = gd->halo;
    g.in0 = in + (int64_t)g.H * (gd->sz + gd->sy + 1);
    g.out0 = out + (int64_t)g.H * (gd->sz + gd->sy + 1);
    g.nx = (int)gd->nx;
    g.ny = (int)gd->ny;
    g.nz = (int)gd->nz;
    g.sy = gd->sy;
    g.sz = gd->sz;
    g.ntx = (g.nx + S::BXT - 1) / S::BXT;
    g.nty = (g.ny + S::BYT - 1) / S::BYT;
    const int64_t cols = (int64_t)g.ntx * g.nty;
    // z chunks: one block per CU at a time, so for each number of rounds the most chunks that
    // fit it, and of those the choice with the fewest planes of work in a row.  A chunk reads
    // zc + 2r planes in steps of PZ; the constant stands for a block's start (fragments, first
    // loads), about four planes' time, and a quarter block for the uneven finish of a launch
    // of several rounds.  (With chunks of at least 32 planes a 100^3 grid ran on 16 of the 256
    // CUs: 297 us against 27.)
    int zc = g.nz;
    int64_t best = -1;
    const int64_t k0 = (cols + 255) / 256;
    for (int64_t k = k0; k < k0 + 16; ++k) {
        const int64_t fit = 256 * k / cols;
        const int nzc = (int)(fit < g.nz ? fit : g.nz), c = (g.nz + nzc - 1) / nzc;
        const int64_t planes = (c + 2 * R + S::PZ - 1) / S::PZ * S::PZ + 4;
        const int64_t cost = 4 * k * planes + (k > 1 ? planes : 0);
        if (best < 0 || cost < best) {
            best = cost;
            zc = c;
        }
    }
    g.zchunk = zc;
    g.nzc = (g.nz + zc - 1) / zc;
    float cmax = 0.f;
    for (int i = 0; i < Q * Q * Q; ++i) {
        a.c[i] = coeffs[i];
        const float v = coeffs[i] < 0 ? -coeffs[i] : coeffs[i];
        cmax = v > cmax ? v : cmax;
    }
    a.cexp = 0;
    if (PREC == MMS_FP16X3S && cmax > 0.f && cmax < 3.0e38f) {
        int e;
        frexpf(cmax, &e);
        a.cexp = 14 - e < 127 ? 14 - e : 127;
    }
    const int64_t nblk = (int64_t)g.ntx * g.nty * g.nzc;
    if (nblk > 0x7fffffff) return MMS_EINVAL;
    hipLaunchKernelGGL((box_mfma_kernel<R, PREC>), dim3((unsigned)nblk), dim3(64 * S::NW), 0,
                       s, a);
    return check_launch("box_mfma_kernel");
}

template <int R>
int launch_r(const float *in, float *out, const mms_grid *g, const float *coeffs, int prec,
             hipStream_t s) {
    switch (prec) {
        case MMS_BF16X3: return launch_rp<R, MMS_BF16X3>(in, out, g, coeffs, s);
        case MMS_FP16X3S: return launch_rp<R, MMS_FP16X3S>(in, out, g, coeffs, s);
        case MMS_BF16X1: return launch_rp<R, MMS_BF16X1>(in, out, g, coeffs, s);
        default: return MMS_EUNSUPPORTED;
    }
}

}  // namespace

int launch_box_mfma(const float *in, float *out, const mms_grid *g, int r, const float *coeffs,
                    int precision, hipStream_t s) {
    switch (r) {
        case 1: return launch_r<1>(in, out, g, coeffs, precision, s);
        case 2: return launch_r<2>(in, out, g, coeffs, precision, s);
        case 3: return launch_r<3>(in, out, g, coeffs, precision, s);
        case 4: return launch_r<4>(in, out, g, coeffs, precision, s);
        default: return MMS_EUNSUPPORTED;
    }
}

}  // namespace mms
