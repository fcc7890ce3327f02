// Pseudo-acoustic TTI step (gfx950): the two-field update of RTM in tilted
// transversely isotropic media (Sec. II-A, Sec. V-F), in units of
// C2 = (v_pz dt / h)^2:
//   p'' = C2 [ (1+2eps) H2 p + alpha H1 q + sigma H1 (p - alpha q) ]
//   q'' = C2 [ ((1+2delta)/alpha) H2 p + H1 q - sigma H2 (p/alpha - q) ]
//   H1 = (n . grad)^2 with n = (sin t cos f, sin t sin f, cos t),  H2 = Laplacian - H1,
// stepped as u^{n+1} = G (2u^n - G u^{n-1} + dt^2 u'') + dt^2 f^n delta_src.
//
// The six second derivatives follow the paper's decomposition into
// one-dimensional stencils (Sec. IV-G): Dxx, Dyy, Dzz with the per-axis
// second-derivative weights; the mixed ones as products of first-derivative
// stencils D (weights d_1..d_r, antisymmetric).  All of it runs in one pass over the
// fields, 44 bytes a point (a pass for the z derivatives through a workspace moved 84):
//  * a block of 512 threads owns a tile of up to 30 words x 32 rows (256 lanes in all) and
//    streams a chunk of z.  One half of the block carries p, the other q; per plane
//    they exchange H1 q and H2 p, the parts the other equation needs, through LDS;
//  * the tiles of planes z .. z+r, with 4 cells of x and r rows of y halo, sit in an LDS
//    ring, each plane requested a step ahead.  When a plane enters, Dx f and Dy f of a
//    lane's own cells are added to the running sums Dz(Dx f), Dz(Dy f) and, with f itself,
//    Dzz f of the 2r planes that wait for it, which are kept in registers (96 at radius
//    4): no z neighbour of a halo cell is ever needed.  Dy f also goes to an LDS ring,
//    halo words included, so that Dxy f = Dx(Dy f) is a row stencil r planes later;
//  * at the centre plane Dxx, Dyy and Dxy come from LDS, the direction cosines from theta and
//    phi; the update, with sponge, source and receivers, follows one step later, behind the
//    barrier that ends the step (the only one);
//  * the other operands are requested one plane ahead of their use; streaming stores.
// LDS holds one block per CU (157 KB at radius 4), 8 waves, two per SIMD.  What bounds it is
// latency: the vector ALUs issue half of the time (about 590 instructions a plane and wave at
// radius 4, 17 % of them beside the other wave's), radius 2 takes nearly as long with half of
// the FMAs, and HBM reads are near their least (2.49 GB against 2.30 at 400^3).  The rest are
// waits of waves in step; several of the loop's loads, and a store, sit behind branches, so the
// wait ahead of the LDS write covers every request in flight.
// Measured at 400^3: 1160 -> 756 us a step (radius 4), 1140 -> 724 (radius 2); 100^3 42 -> 24,
// 301 x 255 x 290 456 -> 287.  On the way: one thread for both fields 1082 (registers), two
// halves 962, Dxy through the Dy ring and z sums for Dzz 910, factored H1 848, one barrier a
// plane 796, angles a plane ahead 756.
#include "mms_internal.h"

namespace mms {
namespace {

typedef float f4v __attribute__((ext_vector_type(4)));

// sin and cos of an angle on the transcendental unit (v_sin_f32 / v_cos_f32 take the
// argument in revolutions and are valid below 256 revolutions in magnitude).  Measured
// on MI355X against FP64 over [-4 pi, 4 pi]: absolute error at most 9.2e-7, RMS 2.4e-7;
// one instruction each where a reduction plus polynomials took about 25, which made
// the eight evaluations per lane and plane 9 % of the kernel's time.
__device__ __forceinline__ void angle_sincos(float x, float *sn, float *cs) {
    const float t = x * 0.159154943091895336f;   // x / (2 pi)
    *sn = __builtin_amdgcn_sinf(t);
    *cs = __builtin_amdgcn_cosf(t);
}

struct TtiArgs {
    Geom g;
    int rows;                            // rows of a tile (txa * rows <= 256 lanes)
    float c2w[5], d1[4];
    const float *pc, *qc;                // stencil fields
    const float *pp, *qp, *c2, *eps, *delta, *theta, *phi;  // own words
    float c2s, sigma, alpha, inv_alpha;
    float *pn, *qn;
    float *traces;
    const float *src;
    int src_z, src_y, src_x;
    int sponge_w;
    float sponge_a;
    int faces;
};

// a b + c into a register of its own (left to itself the compiler accumulates in c's register
// and moves the sum afterwards, 82 moves a plane in the sums below)
__device__ __forceinline__ float fma_to(float a, float b, float c) {
    float d;
    asm("v_fma_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}

// LDS words of a plane's tile with its halo, (rows + 2r) (txa + 2), and of its rows alone,
// rows (txa + 2): what the launch may ask for
constexpr int tile_words(int r) { return (8 + 2 * r) * 32; }
constexpr int DW = 288;
constexpr int NL = 256;   // lanes of a tile, and threads per field

template <int R>
__global__ void __launch_bounds__(2 * NL) tti_kernel(TtiArgs a) {
    constexpr int RP = R + 2;                // ring planes: z .. z+R and the one being stored
    constexpr int TW = tile_words(R);
    constexpr int NLK = (TW + NL - 1) / NL;
    __shared__ float4 ring[2][RP][TW];
    __shared__ float4 dyr[2][R + 1][DW];     // Dy f of planes z .. z+R, rows of the tile
    __shared__ float4 swap[2][2][NL];        // H2 p and H1 q of planes z-1 and z

    const Geom &g = a.g;
    int b = mms_xcd_remap(blockIdx.x, gridDim.x);
    const int txi = b % g.ntx;
    b /= g.ntx;
    const int tyi = b % g.nty;
    const int zci = b / g.nty;
    const int f = __builtin_amdgcn_readfirstlane(threadIdx.x / NL);   // 0: p, 1: q
    const int tid = threadIdx.x % NL;
    // the lanes cover the tile's rows of txa words one after the other
    const int txa = g.txa, lw = txa + 2, rows = a.rows;
    const int ty = tid / txa, tx = tid - ty * txa;
    const bool lane_on = ty < rows;
    const int xt = 4 * txi * txa, yt = tyi * rows;
    const int x0 = xt + 4 * tx, y = yt + ty;
    const int zb = zci * g.zchunk;
    const int ze = min(zb + g.zchunk, g.nz);
    const int nx4 = (g.nx + 3) & ~3;
    const int ylim = g.ny + g.H;
    const int64_t sy = g.sy, sz = g.sz;
    const int W = a.sponge_w;
    const float sa = a.sponge_a;

    const bool own_ok = lane_on && (x0 <= nx4) && (y < ylim);
    const int64_t own_off = own_ok ? (int64_t)y * sy + x0 : 0;
    const int own = lane_on ? (R + ty) * lw + tx + 1 : R * lw + 1;   // idle lanes read the first
    float gown[4];
    {
        const float gy = gaxis(y, g.ny, W, sa, a.faces & 4, a.faces & 8);
#pragma unroll
        for (int e = 0; e < 4; ++e) gown[e] = gy * gaxis(x0 + e, g.nx, W, sa, a.faces & 1, a.faces & 2);
    }
    // tile word i -> row i / lw, column i % lw from (row yt - R, column xt - 4); words outside
    // the array are read from the interior origin instead (they are never used)
    const float *field = f ? a.qc : a.pc;
    const int nw = (rows + 2 * R) * lw;
    int64_t l_off[NLK];
#pragma unroll
    for (int k = 0; k < NLK; ++k) {
        const int i = tid + k * NL;
        const int row = i / lw, col = i - row * lw;
        const bool ok = (i < nw) && (yt - R + row < ylim) && (xt - 4 + 4 * col <= nx4);
        l_off[k] = ok ? (int64_t)(yt - R + row) * sy + (xt - 4 + 4 * col) : 0;
    }
    f4v stage[NLK];
    auto load_tile = [&](int z) {
        const float *p = field + (int64_t)z * sz;
#pragma unroll
        for (int k = 0; k < NLK; ++k) stage[k] = *reinterpret_cast<const f4v *>(p + l_off[k]);
    };
    auto store_tile = [&](int slot) {
#pragma unroll
        for (int k = 0; k < NLK; ++k)
            if (tid + k * NL < nw) *reinterpret_cast<f4v *>(&ring[f][slot][tid + k * NL]) = stage[k];
    };
    auto window = [&](const float4 *row, float *w) {
        const float4 L = row[-1], C = row[0], Rr = row[1];
        w[0] = L.x; w[1] = L.y; w[2] = L.z; w[3] = L.w;
        w[4] = C.x; w[5] = C.y; w[6] = C.z; w[7] = C.w;
        w[8] = Rr.x; w[9] = Rr.y; w[10] = Rr.z; w[11] = Rr.w;
    };
    auto comp = [](const float4 &v, int e) {
        return e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w;
    };

    float d1[R], c2w[R + 1];
#pragma unroll
    for (int i = 0; i < R; ++i) d1[i] = a.d1[i];
#pragma unroll
    for (int i = 0; i <= R; ++i) c2w[i] = a.c2w[i];
    // in vector registers: an FMA with a scalar-register weight never issues beside the other
    // wave's
#pragma unroll
    for (int i = 0; i < R; ++i) asm volatile("" : "+v"(d1[i]));
#pragma unroll
    for (int i = 0; i <= R; ++i) asm volatile("" : "+v"(c2w[i]));
    auto dx1 = [&](const float *w, int e) {   // first x derivative at cell e
        float d = 0.f;
#pragma unroll
        for (int j = 1; j <= R; ++j) d = fmaf(d1[j - 1], w[4 + e + j] - w[4 + e - j], d);
        return d;
    };

    load_tile(zb - R);
    store_tile(0);
    __syncthreads();

    // Dy f is also needed at the words left and right of the tile's rows (Dxy = Dx(Dy f)): the
    // first 2 rows lanes take one of these words each
    const int hrow = tid >> 1, hcol = (tid & 1) ? txa + 1 : 0;
    const bool halo_on = hrow < rows;
    const int down = lane_on ? ty * lw + tx + 1 : 1;
    auto dy_word = [&](const float4 *t) {   // Dy f of the word at t
        float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 1; k <= R; ++k) {
            const float4 u = t[k * lw], d = t[-k * lw];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = fmaf(d1[k - 1], comp(u, e) - comp(d, e), v[e]);
        }
        return make_float4(v[0], v[1], v[2], v[3]);
    };

    // pend[v][j]: sum so far, for output plane (next entering plane) - R + j, of Dz(Dx f),
    // Dz(Dy f) and Dzz f.  The entering plane's term is added while the sums move down one place, so the
    // window needs no copies.
    float pend[3][2 * R][4];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 2 * R; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) pend[i][j][e] = 0.f;

    const float srcv = a.src ? *a.src : 0.f;
    const bool zlo = a.faces & 16, zhi = a.faces & 32;
    // plane z is updated and stored one step after its derivatives, when the barrier at the
    // step's end has published the other half's part
    float h1[4], h2[4], ctr[4];
    float4 prev4, c24, med4, thn = make_float4(0.f, 0.f, 0.f, 0.f), phn = thn;
    auto finish = [&](int z) {
        const float gz = gaxis(z, g.nz, W, sa, zlo, zhi);
        const float4 other = swap[z & 1][1 - f][tid];
        float r[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float med = 1.f + 2.f * comp(med4, e), o = comp(other, e);
            const float sg = a.sigma, al = a.alpha, ia = a.inv_alpha;   // ia = 1 / alpha
            const float acc = f ? med * ia * o + h1[e] - sg * (o * ia - h2[e])
                                : med * h2[e] + al * o + sg * (h1[e] - al * o);
            const float G = gz * gown[e];
            r[e] = G * (2.0f * ctr[e] - G * comp(prev4, e) + a.c2s * comp(c24, e) * acc);
        }
        if (srcv != 0.f && z == a.src_z && y == a.src_y && a.src_x >= x0 && a.src_x < x0 + 4) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (x0 + e == a.src_x) r[e] += srcv;
        }
        if (lane_on && y < g.ny && x0 < g.nx) {
            float *po = (f ? a.qn : a.pn) + (int64_t)z * sz + own_off;
            if (x0 + 3 < g.nx) {
                const f4v v = {r[0], r[1], r[2], r[3]};
                __builtin_nontemporal_store(v, reinterpret_cast<f4v *>(po));
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (x0 + e < g.nx) po[e] = r[e];
            }
            if (f == 0 && a.traces && z == 0) {
                float *pt = a.traces + (int64_t)y * g.nx + x0;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (x0 + e < g.nx) pt[e] = ctr[e];
            }
        }
    };
    int se = 0, de = 0;   // slots of the entering plane in ring and dyr
    for (int zi = zb - R; zi < ze + R; ++zi) {
        const int z = zi - R;
        const bool more = zi + 1 < ze + R;
        const int sc = se + 2 < RP ? se + 2 : se + 2 - RP;   // ring slot of plane z
        if (more) load_tile(zi + 1);
        const int64_t zo = (int64_t)z * sz + own_off;
        const float4 th4 = thn, ph4 = phn;
        if (z + 1 >= zb && z + 1 < ze) {   // a plane ahead
            thn = *reinterpret_cast<const float4 *>(a.theta + zo + sz);
            phn = *reinterpret_cast<const float4 *>(a.phi + zo + sz);
        }
        if (z >= zb) {
            if (z > zb) finish(z - 1);
            prev4 = *reinterpret_cast<const float4 *>((f ? a.qp : a.pp) + zo);
            c24 = *reinterpret_cast<const float4 *>(a.c2 + zo);
            med4 = *reinterpret_cast<const float4 *>((f ? a.delta : a.eps) + zo);
        }
        // entering plane: Dx f and Dy f of the own cells go into the z sums
        float dz1[3][4];   // completed at plane z
        {
            const float4 *t = &ring[f][se][own];
            float w[12], v[3][4];
            window(t, w);
            const float4 dy = dy_word(t);
            if (lane_on) dyr[f][de][down] = dy;
            if (halo_on) dyr[f][de][hrow * lw + hcol] = dy_word(&ring[f][se][(R + hrow) * lw + hcol]);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[0][e] = dx1(w, e);
                v[1][e] = comp(dy, e);
                v[2][e] = w[4 + e];
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                // weight of a plane k above the output
                auto wt = [&](int k) {
                    return i == 2 ? c2w[k < 0 ? -k : k] : k == 0 ? 0.f : k > 0 ? d1[k - 1] : -d1[-k - 1];
                };
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    dz1[i][e] = fmaf(wt(R), v[i][e], pend[i][0][e]);
#pragma unroll
                    for (int j = 0; j < 2 * R - 1; ++j) {
                        const int k = R - 1 - j;
                        pend[i][j][e] = i < 2 && k == 0 ? pend[i][j + 1][e]
                                                        : fma_to(wt(k), v[i][e], pend[i][j + 1][e]);
                    }
                    pend[i][2 * R - 1][e] = wt(-R) * v[i][e];
                }
            }
        }
        if (z >= zb) {
            const float4 *t = &ring[f][sc][own];
            float w[12], dyw[12], sxx[4], syy[4];
            window(t, w);
            // slot of plane z in dyr: the next one after the entering plane's
            window(&dyr[f][de + 1 <= R ? de + 1 : 0][down], dyw);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float c0 = c2w[0] * w[4 + e];
                float s2 = c0;
#pragma unroll
                for (int j = 1; j <= R; ++j) s2 = fmaf(c2w[j], w[4 + e + j] + w[4 + e - j], s2);
                ctr[e] = w[4 + e];
                sxx[e] = s2;
                syy[e] = c0;
            }
#pragma unroll
            for (int k = 1; k <= R; ++k) {
                const float4 u = t[k * lw], d = t[-k * lw];
#pragma unroll
                for (int e = 0; e < 4; ++e) syy[e] = fmaf(c2w[k], comp(u, e) + comp(d, e), syy[e]);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float st, ct, sn, cn;
                angle_sincos(comp(th4, e), &st, &ct);
                angle_sincos(comp(ph4, e), &sn, &cn);
                const float nx_ = st * cn, ny_ = st * sn, nz_ = ct;
                // H1 = sum_ij n_i n_j D_ij, factored by the first index
                const float ny2 = 2.f * ny_, nz2 = 2.f * nz_;
                const float tx_ = fmaf(nx_, sxx[e], fmaf(ny2, dx1(dyw, e), nz2 * dz1[0][e]));
                const float ty_ = fmaf(ny_, syy[e], nz2 * dz1[1][e]);
                h1[e] = fmaf(nx_, tx_, fmaf(ny_, ty_, nz_ * (nz_ * dz1[2][e])));
                h2[e] = (sxx[e] + syy[e] + dz1[2][e]) - h1[e];
            }
            // p'' takes H1 q from the other half of the block, q'' takes H2 p
            swap[z & 1][f][tid] = f ? make_float4(h1[0], h1[1], h1[2], h1[3])
                                    : make_float4(h2[0], h2[1], h2[2], h2[3]);
        }
        // the next plane takes the ring slot of plane z - 1
        de = de + 1 <= R ? de + 1 : 0;
        se = se + 1 < RP ? se + 1 : 0;
        if (more) store_tile(se);
        __syncthreads();
    }
    finish(ze - 1);
}

template <int R>
int launch_tti(const mms_wave *w, const mms_tti *t, int n, const float *pp, const float *pc,
               float *pn, const float *qp, const float *qc, float *qn, hipStream_t s) {
    const mms_grid *gd = &w->g;
    const int64_t o = (int64_t)gd->halo * (gd->sz + gd->sy + 1);
    // (the pitch limit that the header states; this kernel's own offsets are 64-bit)
    if ((int64_t)(8 + 2 * R + 1) * gd->sy >= ((int64_t)1 << 32)) {
        set_last_error("TTI step: grid rows too long for 32-bit tile offsets");
        return MMS_EUNSUPPORTED;
    }
    TtiArgs a{};
    Geom &g = a.g;
    g.H = gd->halo;
    g.nx = (int)gd->nx;
    g.ny = (int)gd->ny;
    g.nz = (int)gd->nz;
    g.sy = gd->sy;
    g.sz = gd->sz;
    // Tiles of txa <= 30 words and as many rows as 256 lanes hold, one block per CU: of the
    // fewest x tiles and up to two more, the shape with the shortest launch.  A chunk's 2r first
    // planes only enter the z sums, about half a plane's work each.
    int words = 0, n0 = 0;
    balanced_tile_words(g.nx, 30, &n0);
    words = (g.nx + 3) / 4;
    int64_t best = -1;
    for (int n = n0; n < n0 + 3; ++n) {
        const int txa = (words + n - 1) / n < 1 ? 1 : (words + n - 1) / n;
        int rows = NL / txa < 32 ? NL / txa : 32;
        if (rows > DW / (txa + 2)) rows = DW / (txa + 2);
        if (rows > tile_words(R) / (txa + 2) - 2 * R) rows = tile_words(R) / (txa + 2) - 2 * R;
        const int ntx = (words + txa - 1) / txa, nty = (g.ny + rows - 1) / rows;
        int64_t cost;
        const int zc = pick_zchunk_rounds(g.nz, (int64_t)ntx * nty, 256, 1, 256, R + 1, &cost);
        if (best < 0 || cost < best) {
            best = cost;
            g.txa = txa;
            g.ntx = ntx;
            g.nty = nty;
            g.zchunk = zc;
            a.rows = rows;
        }
    }
    g.nzc = (g.nz + g.zchunk - 1) / g.zchunk;
    for (int k = 0; k <= R; ++k) a.c2w[k] = w->lap[k];
    for (int k = 0; k < R; ++k) a.d1[k] = t->d1[k];
    a.pc = pc + o;
    a.qc = qc + o;
    a.pp = pp + o;
    a.qp = qp + o;
    a.c2 = w->c2 + o;
    a.eps = t->eps + o;
    a.delta = t->delta + o;
    a.theta = t->theta + o;
    a.phi = t->phi + o;
    a.c2s = w->c2_scale;
    a.sigma = t->sigma;
    a.alpha = t->alpha;
    a.inv_alpha = 1.0f / t->alpha;
    a.pn = pn + o;
    a.qn = qn + o;
    a.traces = w->traces ? w->traces + (int64_t)n * gd->ny * gd->nx : nullptr;
    a.src = (w->src_dt2f && n >= 0 && n < w->nt) ? w->src_dt2f + n : nullptr;
    a.src_z = (int)w->src_z;
    a.src_y = (int)w->src_y;
    a.src_x = (int)w->src_x;
    a.sponge_w = w->sponge_width;
    a.sponge_a = w->sponge_alpha;
    a.faces = w->sponge_faces;
    const int64_t nblk = (int64_t)g.ntx * g.nty * g.nzc;
    if (nblk > 0x7fffffff) return MMS_EINVAL;
    hipLaunchKernelGGL((tti_kernel<R>), dim3((unsigned)nblk), dim3(2 * NL), 0, s, a);
    return check_launch("tti_kernel");
}

}  // namespace

int tti_step(const mms_wave *w, const mms_tti *t, int n, const float *pp, const float *pc,
             float *pn, const float *qp, const float *qc, float *qn, hipStream_t s) {
    switch (w->radius) {
        case 1: return launch_tti<1>(w, t, n, pp, pc, pn, qp, qc, qn, s);
        case 2: return launch_tti<2>(w, t, n, pp, pc, pn, qp, qc, qn, s);
        case 3: return launch_tti<3>(w, t, n, pp, pc, pn, qp, qc, qn, s);
        case 4: return launch_tti<4>(w, t, n, pp, pc, pn, qp, qc, qn, s);
        default: return MMS_EUNSUPPORTED;
    }
}

}  // namespace mms
