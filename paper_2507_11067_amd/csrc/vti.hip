// Fused pseudo-acoustic VTI step (gfx950): the two-field anisotropic update that
// RTM in VTI media runs (Sec. II-A, Sec. V-F), in the well-posed form the TTI
// system of Sec. II-A takes for zero tilt and zero shear velocity:
//   H^{n+1} = G (2 H^n - G H^{n-1} + C2 (a Sxy H^n + b Szz V^n)) + dt^2 f^n delta_src
//   V^{n+1} = G (2 V^n - G V^{n-1} + C2 (b Sxy H^n +   Szz V^n)) + dt^2 f^n delta_src
// a = 1 + 2 epsilon and b = sqrt(1 + 2 delta) are fields; Sxy = Sxx + Syy and Szz
// are the axis parts of the star.  Only H needs x and y neighbours and only V
// needs z neighbours, so (following the paper's decomposition of complex kernels
// into one-dimensional stencils on small blocks, Sec. IV-G):
//  * H travels through a double-buffered LDS tile (x/y halo);
//  * V travels through a register queue of 2r+1 planes (z terms only);
//  * both outputs are written with streaming stores.
// The step is bound by the memory system (36 bytes a point; radius 2 takes as long as radius 4 at
// 400^3), so its requests must not stop: each operand's registers are requested anew as soon as
// the plane in hand has used them (point-wise operands and the H tile one plane ahead, V two),
// after the stores, so that a wait counts younger requests only, and across the barrier.  Loads
// straight into LDS cannot stay in flight there (the barrier waits for all of them): with them
// the kernel took, us a step at radius 4, before / now: 160^3 31.5 / 28.7, 200^3 53.8 / 51.3,
// 301 x 255 x 290 186 / 177, 400^3 509 / 499 (4.6 TB/s); radius 2, 240 x 250 x 230: 115 / 108.
// Small grids take a direct kernel, narrow ones flat tiles (see DIRECT_MAX, FLAT_MAX_NX).  us a
// step, radius 4, before / with them: 64^3 13.9 / 10.8 (the host's side of a call),
// 128^3 19.6 / 17.2, 47 x 300 x 300 67.9 / 34.6, 100 x 300 x 300 87.1 / 70.3.
#include "mms_internal.h"

namespace mms {
namespace {

typedef float f4v __attribute__((ext_vector_type(4)));

constexpr int VNT = 512;

struct VtiArgs {
    Geom g;
    float c[9];            // per-axis weights, k + r (symmetric)
    const float *hc, *vc;  // H^n, V^n
    const float *hp, *vp;  // H^{n-1}, V^{n-1}
    const float *c2, *fa, *fb;
    float c2s;
    float *hn, *vn;        // outputs
    float *traces;         // [ny][nx] plane of level n, or NULL
    const float *src;
    int src_z, src_y, src_x;
    int sponge_w;
    float sponge_a;
    int faces;
};

// Point-wise operands of four cells: H^{n-1}, V^{n-1}, C2, a, b
struct Pw {
    float4 hp, vp, c2, fa, fb;
};

// New values of both fields at the cells (z, y, x0 ..) from S_xy H, S_zz V and the operands.
// The fused operations are spelt out: which product of a sum the compiler fuses, and so the
// last bit, would otherwise differ from kernel to kernel.
__device__ __forceinline__ void update_cells(const VtiArgs &a, int z, int y, int x0, float gz,
                                             const float *gown, const float4 &hc4,
                                             const float4 &vc4, const float *sxy, const float *szz,
                                             const Pw &pw, float srcv, float *rh, float *rv) {
    const float hcv[4] = {hc4.x, hc4.y, hc4.z, hc4.w};
    const float vcv[4] = {vc4.x, vc4.y, vc4.z, vc4.w};
    const float hpv[4] = {pw.hp.x, pw.hp.y, pw.hp.z, pw.hp.w};
    const float vpv[4] = {pw.vp.x, pw.vp.y, pw.vp.z, pw.vp.w};
    const float c2v[4] = {pw.c2.x, pw.c2.y, pw.c2.z, pw.c2.w};
    const float fav[4] = {pw.fa.x, pw.fa.y, pw.fa.z, pw.fa.w};
    const float fbv[4] = {pw.fb.x, pw.fb.y, pw.fb.z, pw.fb.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float G = gz * gown[e];
        const float C2 = a.c2s * c2v[e];
        rh[e] = G * fmaf(C2, fmaf(fav[e], sxy[e], fbv[e] * szz[e]),
                         fmaf(2.0f, hcv[e], -(G * hpv[e])));
        rv[e] = G * fmaf(C2, fmaf(fbv[e], sxy[e], szz[e]), fmaf(2.0f, vcv[e], -(G * vpv[e])));
    }
    if (srcv != 0.f && z == a.src_z && y == a.src_y && a.src_x >= x0 &&
        a.src_x < x0 + 4) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (x0 + e == a.src_x) {
                rh[e] += srcv;
                rv[e] += srcv;
            }
    }
}

// Streaming stores of both fields at four cells (plane offset off) and the receivers' reading.
__device__ __forceinline__ void store_cells(const VtiArgs &a, int z, int y, int x0, int64_t off,
                                            const float4 &hc4, const float *rh, const float *rv) {
    const Geom &g = a.g;
    const int64_t sz = g.sz;
    const float hcv[4] = {hc4.x, hc4.y, hc4.z, hc4.w};
    float *ph_ = a.hn + (int64_t)z * sz + off;
    float *pv_ = a.vn + (int64_t)z * sz + off;
    if (x0 + 3 < g.nx) {
        const f4v vh = {rh[0], rh[1], rh[2], rh[3]};
        const f4v vv = {rv[0], rv[1], rv[2], rv[3]};
        __builtin_nontemporal_store(vh, reinterpret_cast<f4v *>(ph_));
        __builtin_nontemporal_store(vv, reinterpret_cast<f4v *>(pv_));
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (x0 + e < g.nx) {
                ph_[e] = rh[e];
                pv_[e] = rv[e];
            }
    }
    if (a.traces && z == 0) {
        float *pt = a.traces + (int64_t)y * g.nx + x0;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (x0 + e < g.nx) pt[e] = hcv[e];
    }
}

// FLAT: the lanes cover rows of txa words one after the other; else a row has 64 lanes, of which
// txa own words.
template <int R, bool FLAT>
__global__ void __launch_bounds__(VNT) vti_kernel(VtiArgs a) {
    constexpr int Q = 2 * R + 1;
    constexpr int NT = VNT;
    constexpr int NL = flat_tile_words(R, NT);   // words of the largest H tile, row-major
    constexpr int NLK = (NL + NT - 1) / NT;
    __shared__ float4 tile[2][NL];

    const Geom &g = a.g;
    int b = mms_xcd_remap(blockIdx.x, gridDim.x);
    const int txi = b % g.ntx;
    b /= g.ntx;
    const int tyi = b % g.nty;
    const int zci = b / g.nty;
    const int tid = threadIdx.x;
    // txa lanes of a row own words; the others only help with the halo and the barriers.  pitch:
    // LDS words of a tile row
    const int txa = g.txa, lw = txa + 2, bxa = 4 * txa;
    const int rows = FLAT ? g.rows : NT / 64, pitch = FLAT ? lw : 66;
    const int ty = FLAT ? tid / txa : tid / 64, tx = FLAT ? tid - ty * txa : tid % 64;
    const bool lane_on = FLAT ? ty < rows : tx < txa;
    const int nw = FLAT ? (rows + 2 * R) * lw : NL;
    const int xt = txi * bxa, yt = tyi * rows;
    const int x0 = xt + 4 * tx, y = yt + ty;
    // (idle lanes of a flat tile read its first word)
    const int own = !FLAT || lane_on ? (R + ty) * pitch + tx + 1 : R * pitch + 1;
    const int zb = zci * g.zchunk;
    const int ze = min(zb + g.zchunk, g.nz);
    const int nx4 = (g.nx + 3) & ~3;
    const int ylim = g.ny + g.H;
    const int64_t sy = g.sy, sz = g.sz;
    const int W = a.sponge_w;
    const float sa = a.sponge_a;

    const bool own_ok = lane_on && (x0 <= nx4) && (y < ylim);
    const int64_t own_off = (int64_t)y * sy + x0;
    // lanes without cells in the array read the plane's first word (never used): an address
    // select rather than a guard, so that no branch hides the number of requests in flight
    const int64_t ld_off = own_ok ? own_off : 0;
    float gown[4];
    {
        const float gy = gaxis(y, g.ny, W, sa, a.faces & 4, a.faces & 8);
#pragma unroll
        for (int e = 0; e < 4; ++e) gown[e] = gy * gaxis(x0 + e, g.nx, W, sa, a.faces & 1, a.faces & 2);
    }
    auto ld = [&](const float *base, int z) -> float4 {
        return *reinterpret_cast<const float4 *>(base + (int64_t)z * sz + ld_off);
    };
    // H tile word i -> (row i / pitch, col i % pitch) from the tile origin (row yt - R, column
    // xt - 4); words outside this tile's lw columns or outside the array are read from the
    // origin instead (never used)
    uint32_t d_off[NLK];
#pragma unroll
    for (int k = 0; k < NLK; ++k) {
        const int i = tid + k * NT;
        const int row = i / pitch, col = i % pitch;
        const bool ok = (i < nw) && (col < lw) && (yt - R + row < ylim) && (xt - 4 + 4 * col <= nx4);
        d_off[k] = ok ? (uint32_t)row * (uint32_t)sy + 4u * (uint32_t)col : 0u;
    }
    f4v st[NLK];
    auto load_tile = [&](int z) {
        const float *p = a.hc + (int64_t)z * sz + (int64_t)(yt - R) * sy + (xt - 4);
#pragma unroll
        for (int k = 0; k < NLK; ++k) st[k] = *reinterpret_cast<const f4v *>(p + d_off[k]);
    };
    auto store_tile = [&](float4 *t) {
#pragma unroll
        for (int k = 0; k < NLK; ++k)
            if (tid + k * NT < nw) *reinterpret_cast<f4v *>(t + tid + k * NT) = st[k];
    };

    auto load_pw = [&](int z) {
        Pw p;
        p.hp = ld(a.hp, z);
        p.vp = ld(a.vp, z);
        p.c2 = ld(a.c2, z);
        p.fa = ld(a.fa, z);
        p.fb = ld(a.fb, z);
        return p;
    };

    const int zl = ze - 1;
    // V at planes z-R .. z+R, and z+R+1 (requested)
    constexpr int QS = Q + 1;
    float4 q[QS];
#pragma unroll
    for (int i = 0; i < Q; ++i) q[i] = ld(a.vc, zb - R + i);
    load_tile(zb);
    store_tile(tile[0]);
    load_tile(min(zb + 1, zl));
    Pw pw = load_pw(zb);
    q[Q] = ld(a.vc, min(zb + 1, zl) + R);
    __syncthreads();

    const float *c = a.c;
    const float srcv = a.src ? *a.src : 0.f;
    const bool zlo = a.faces & 16, zhi = a.faces & 32;
    for (int z = zb;;) {
#pragma unroll
        for (int ph = 0; ph < QS; ++ph) {
            const float4 *t = &tile[ph & 1][own];
            const float4 hc4 = t[0];
            const float4 L = t[-1];
            const float4 Rr = t[1];
            const float w[12] = {L.x,   L.y,   L.z,   L.w,  hc4.x, hc4.y,
                                 hc4.z, hc4.w, Rr.x, Rr.y, Rr.z,  Rr.w};
            float sxy[4] = {0.f, 0.f, 0.f, 0.f}, szz[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = -R; k <= R; ++k) {
                const float ck = c[R + k];
                const float4 vy = k == 0 ? hc4 : t[k * pitch];
                const float4 vz = q[(ph + R + k) % QS];
                const float yv[4] = {vy.x, vy.y, vy.z, vy.w};
                const float zv[4] = {vz.x, vz.y, vz.z, vz.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    sxy[e] = fmaf(ck, yv[e] + w[4 + e + k], sxy[e]);
                    szz[e] = fmaf(ck, zv[e], szz[e]);
                }
            }
            const float gz = gaxis(z, g.nz, W, sa, zlo, zhi);
            float rh[4], rv[4];
            update_cells(a, z, y, x0, gz, gown, hc4, q[(ph + R) % QS], sxy, szz, pw, srcv, rh, rv);
            store_tile(tile[(ph & 1) ^ 1]);
            if (lane_on && y < g.ny && x0 < g.nx) store_cells(a, z, y, x0, own_off, hc4, rh, rv);
            if (++z >= ze) return;
            pw = load_pw(z);
            load_tile(min(z + 1, zl));
            q[ph] = ld(a.vc, min(z + 1, zl) + R);
            __syncthreads();
        }
    }
}

// Small grids: one lane per 16-byte word reads its words of H (row and column) and V (z) straight
// from memory (the operations, and their order, are those of vti_kernel).
template <int R>
__global__ void __launch_bounds__(256) vti_direct_kernel(VtiArgs a, unsigned nwords, unsigned nxw) {
    const unsigned i = (unsigned)mms_xcd_remap(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
    if (i >= nwords) return;
    const Geom &g = a.g;
    const unsigned row = i / nxw;
    const int x0 = 4 * (int)(i % nxw), y = (int)(row % (unsigned)g.ny), z = (int)(row / (unsigned)g.ny);
    const int64_t off = (int64_t)y * g.sy + x0, zoff = (int64_t)z * g.sz + off;
    auto ld = [](const float *q) { return *reinterpret_cast<const float4 *>(q); };
    const float *h = a.hc + zoff, *v = a.vc + zoff;
    const float4 L = ld(h - 4), hc4 = ld(h), Rr = ld(h + 4), vc4 = ld(v);
    float4 vy[2 * R + 1], vz[2 * R + 1];
#pragma unroll
    for (int k = -R; k <= R; ++k) {
        vy[k + R] = k == 0 ? hc4 : ld(h + k * g.sy);
        vz[k + R] = k == 0 ? vc4 : ld(v + k * g.sz);
    }
    Pw pw;
    pw.hp = ld(a.hp + zoff);
    pw.vp = ld(a.vp + zoff);
    pw.c2 = ld(a.c2 + zoff);
    pw.fa = ld(a.fa + zoff);
    pw.fb = ld(a.fb + zoff);
    const float srcv = a.src ? *a.src : 0.f;
    const int W = a.sponge_w;
    const float sa = a.sponge_a;
    float gown[4];
    const float gy = gaxis(y, g.ny, W, sa, a.faces & 4, a.faces & 8);
#pragma unroll
    for (int e = 0; e < 4; ++e) gown[e] = gy * gaxis(x0 + e, g.nx, W, sa, a.faces & 1, a.faces & 2);
    const float gz = gaxis(z, g.nz, W, sa, a.faces & 16, a.faces & 32);
    const float w[12] = {L.x,   L.y,   L.z,   L.w,  hc4.x, hc4.y,
                         hc4.z, hc4.w, Rr.x, Rr.y, Rr.z,  Rr.w};
    float sxy[4] = {0.f, 0.f, 0.f, 0.f}, szz[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = -R; k <= R; ++k) {
        const float ck = a.c[R + k];
        const float yv[4] = {vy[R + k].x, vy[R + k].y, vy[R + k].z, vy[R + k].w};
        const float zv[4] = {vz[R + k].x, vz[R + k].y, vz[R + k].z, vz[R + k].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            sxy[e] = fmaf(ck, yv[e] + w[4 + e + k], sxy[e]);
            szz[e] = fmaf(ck, zv[e], szz[e]);
        }
    }
    float rh[4], rv[4];
    update_cells(a, z, y, x0, gz, gown, hc4, vc4, sxy, szz, pw, srcv, rh, rv);
    store_cells(a, z, y, x0, off, hc4, rh, rv);
}

}  // namespace

int vti_step(const mms_wave *w, int n, const float *fa, const float *fb, const float *hp,
             const float *hc, float *hn, const float *vp, const float *vc, float *vn,
             hipStream_t s) {
    VtiArgs a{};
    Geom &g = a.g;
    const mms_grid *gd = &w->g;
    g.H = gd->halo;
    g.nx = (int)gd->nx;
    g.ny = (int)gd->ny;
    g.nz = (int)gd->nz;
    g.sy = gd->sy;
    g.sz = gd->sz;
    // the H tile is addressed with 32-bit offsets from its origin
    if (!tile_offsets_fit(VNT / 64, w->radius, g.sy)) {
        set_last_error("VTI step: grid rows too long for 32-bit tile offsets");
        return MMS_EUNSUPPORTED;
    }
    g.txa = balanced_tile_words(g.nx, 64, &g.ntx);
    g.nty = (g.ny + 7) / 8;
    // one 512-thread block per CU (VGPR-bound), 256 CUs; the V queue fill costs
    // about one plane of traffic
    g.zchunk = pick_zchunk_rounds(g.nz, (int64_t)g.ntx * g.nty, 256, 8, 128, 1);
    g.nzc = (g.nz + g.zchunk - 1) / g.zchunk;
    const bool flat = g.nx <= FLAT_MAX_NX && flat_tile32(g, w->radius, VNT, 256, 8);
    const int r = w->radius;
    for (int k = -r; k <= r; ++k) a.c[k + r] = w->lap[k < 0 ? -k : k];
    const int64_t o = (int64_t)gd->halo * (gd->sz + gd->sy + 1);
    a.hc = hc + o;
    a.vc = vc + o;
    a.hp = hp + o;
    a.vp = vp + o;
    a.c2 = w->c2 + o;
    a.fa = fa + o;
    a.fb = fb + o;
    a.c2s = w->c2_scale;
    a.hn = hn + o;
    a.vn = vn + o;
    a.traces = w->traces ? w->traces + (int64_t)n * gd->ny * gd->nx : nullptr;
    a.src = (w->src_dt2f && n >= 0 && n < w->nt) ? w->src_dt2f + n : nullptr;
    a.src_z = (int)w->src_z;
    a.src_y = (int)w->src_y;
    a.src_x = (int)w->src_x;
    a.sponge_w = w->sponge_width;
    a.sponge_a = w->sponge_alpha;
    a.faces = w->sponge_faces;
    if ((int64_t)g.nx * g.ny * g.nz <= DIRECT_MAX) {
        const unsigned nxw = (unsigned)(g.nx + 3) / 4;
        const unsigned nwords = nxw * (unsigned)g.ny * (unsigned)g.nz;
        const dim3 grid((nwords + 255) / 256), block(256);
        switch (r) {
            case 1: hipLaunchKernelGGL((vti_direct_kernel<1>), grid, block, 0, s, a, nwords, nxw); break;
            case 2: hipLaunchKernelGGL((vti_direct_kernel<2>), grid, block, 0, s, a, nwords, nxw); break;
            case 3: hipLaunchKernelGGL((vti_direct_kernel<3>), grid, block, 0, s, a, nwords, nxw); break;
            case 4: hipLaunchKernelGGL((vti_direct_kernel<4>), grid, block, 0, s, a, nwords, nxw); break;
            default: return MMS_EUNSUPPORTED;
        }
        return check_launch("vti_direct_kernel");
    }
    const int64_t nblk = (int64_t)g.ntx * g.nty * g.nzc;
    if (nblk > 0x7fffffff) return MMS_EINVAL;
    const dim3 grid((unsigned)nblk), block(VNT);
    switch (2 * r + flat) {
        case 2: hipLaunchKernelGGL((vti_kernel<1, false>), grid, block, 0, s, a); break;
        case 3: hipLaunchKernelGGL((vti_kernel<1, true>), grid, block, 0, s, a); break;
        case 4: hipLaunchKernelGGL((vti_kernel<2, false>), grid, block, 0, s, a); break;
        case 5: hipLaunchKernelGGL((vti_kernel<2, true>), grid, block, 0, s, a); break;
        case 6: hipLaunchKernelGGL((vti_kernel<3, false>), grid, block, 0, s, a); break;
        case 7: hipLaunchKernelGGL((vti_kernel<3, true>), grid, block, 0, s, a); break;
        case 8: hipLaunchKernelGGL((vti_kernel<4, false>), grid, block, 0, s, a); break;
        case 9: hipLaunchKernelGGL((vti_kernel<4, true>), grid, block, 0, s, a); break;
        default: return MMS_EUNSUPPORTED;
    }
    return check_launch("vti_kernel");
}

}  // namespace mms
