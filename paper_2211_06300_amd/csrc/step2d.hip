// Time steps of the 2D 8th-order acoustic scheme (Sec. 4.1) with the fused
// work of the hot path: point / dense source injection (Sec. 2.1, eq. newq2),
// receiver recording R and adjoint injection R^T (Sec. 2.1, Sec. 3), the CG
// direction update (Algorithm 1), the normal-operator output N p = mu + beta
// B^2 p with its p.Np partials (eq. axb), and the zero-lag correlations of the
// gradient (eq. gradewi).
//
// State per shot: u (two slots) and the increment d = u^n - u^{n-1} (two
// slots), each on a storage grid with a zero ghost frame of GH = 8 cells
// around the padded grid (rows XS floats apart), so stencil loads of a tile
// grown by two stencil radii never need bounds checks.  A launch reads the
// current slots and writes the other ones.
//
// k_step2d<FL>:    one step; a 256-thread workgroup owns a 64 x 32 tile.  The
//                  tile of u^n plus a 4-cell halo is staged in LDS, each lane
//                  owns a column and 8 rows, z neighbours from registers, x
//                  neighbours from LDS.
// k_step2d_t2<FL, TH>: two steps per launch (time blocking) on tiles of 56
//                  columns and TH rows.  u^n is staged on the tile grown by 8
//                  cells, the first step is computed on the tile grown by 4
//                  cells (64 columns: one wave across) into LDS, the second on
//                  the tile.  The wavefield state crosses HBM once per two steps.
//
// Workgroup ids are remapped so that consecutive tiles land on the same XCD
// (8 XCDs take workgroups round-robin), keeping halo neighbours in one L2.
#include <type_traits>

#include "esi_internal.h"

namespace esi {

namespace {

#ifndef ESI_RZ
#define ESI_RZ 8
#endif
#ifndef ESI_TX
#define ESI_TX 64
#endif
#ifndef ESI_MINW
#define ESI_MINW 1
#endif
constexpr int TX = ESI_TX;   // tile width: WX waves of 64 lanes side by side
constexpr int WX = TX / 64;
constexpr int WZ = 4 / WX;   // waves stacked along z (4 waves per workgroup)
constexpr int RZ = ESI_RZ;   // rows per lane
static_assert(TX % 64 == 0 && 4 % WX == 0, "tile width must be 64, 128 or 256");
constexpr int TZ = WZ * RZ;
// one-step kernel: tile + one radius
constexpr int LW = TX + 2 * HALO;
constexpr int LH = TZ + 2 * HALO;

__device__ __forceinline__ int xcd_remap(int b, int nblocks) {
    const int per = nblocks / XCDS, rem = nblocks % XCDS;
    const int xcd = b % XCDS, idx = b / XCDS;
    return xcd < rem ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
}

// A 64-bit value of another lane, through the vector unit
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
    union { double d; int w[2]; } u;
    u.d = v;
    u.w[0] = __builtin_amdgcn_mov_dpp(u.w[0], CTRL, 0xF, 0xF, true);
    u.w[1] = __builtin_amdgcn_mov_dpp(u.w[1], CTRL, 0xF, 0xF, true);
    return u.d;
}

// Sum over the wave (all lanes active), in every lane: v += v of lane ^ o for o =
// 32, 16, 8, 4, 2, 1.  The exchanges stay in the vector unit: through LDS
// (shuffles), two a step one after another, they took 0.2 us more at the end of every
// launch that keeps a partial sum (CG on one 201 x 201 shot: 6.1 and 5.8 us a launch).
__device__ __forceinline__ double wave_sum(double v) {
    union { double d; uint32_t w[2]; } u, x, y;
    u.d = v;
#pragma unroll
    for (int h = 0; h < 2; ++h) {   // lower and upper 32 lanes, each in both halves
        const auto r = __builtin_amdgcn_permlane32_swap(u.w[h], u.w[h], false, false);
        x.w[h] = r[0]; y.w[h] = r[1];
    }
    u.d = x.d + y.d;
#pragma unroll
    for (int h = 0; h < 2; ++h) {   // even and odd rows of 16 lanes
        const auto r = __builtin_amdgcn_permlane16_swap(u.w[h], u.w[h], false, false);
        x.w[h] = r[0]; y.w[h] = r[1];
    }
    v = x.d + y.d;
    v += dpp<0x128>(v);               // row_ror:8
    v += dpp<0x1B>(dpp<0x141>(v));    // ^ 7 (row_half_mirror), ^ 3 (quad_perm)
    v += dpp<0x4E>(v);                // ^ 2
    v += dpp<0xB1>(v);                // ^ 1
    return v;
}

// Laplacian (times dx^2) at an LDS cell from neighbour differences: the centre
// weight is -2 sum_k a_k, and for a smooth field each u_{+-k} - u is exact in
// float32, so the weighted sum carries no cancellation error.  `p` points at
// the cell, `stride` is the LDS row pitch.
__device__ __forceinline__ float lap_lds(const StepArgs& a, const float* p, int stride) {
    const float cv = p[0];
    float lx = a.w1 * ((p[-1] - cv) + (p[1] - cv));
    lx = fmaf(a.w2, (p[-2] - cv) + (p[2] - cv), lx);
    lx = fmaf(a.w3, (p[-3] - cv) + (p[3] - cv), lx);
    lx = fmaf(a.w4, (p[-4] - cv) + (p[4] - cv), lx);
    float lz = a.w1 * ((p[-stride] - cv) + (p[stride] - cv));
    lz = fmaf(a.w2, (p[-2 * stride] - cv) + (p[2 * stride] - cv), lz);
    lz = fmaf(a.w3, (p[-3 * stride] - cv) + (p[3 * stride] - cv), lz);
    lz = fmaf(a.w4, (p[-4 * stride] - cv) + (p[4 * stride] - cv), lz);
    return lx + lz;
}

// (1+k) u^{n+1} = 2u^n - (1-k) u^{n-1} + c lq advanced through the increment
// d^n = u^n - u^{n-1}: (1+k) d^{n+1} = (1-k) d^n + c lq, u^{n+1} = u^n + d^{n+1}.
// Keeping d in its own array stops the rounding of u from leaking into the
// velocity, where it would persist.
// The division by 1 + k uses the hardware reciprocal (within 1 ulp): k = 0 on
// every physical cell, where rcp(1) = 1 exactly and the update is unchanged.
__device__ __forceinline__ float incr(float c2v, float lq, float dv, float kap) {
    return fmaf(c2v, lq, (1.f - kap) * dv) * __builtin_amdgcn_rcpf(1.f + kap);
}

// Element access through a uniform base and a 32-bit byte offset, so that the
// compiler can use scalar-base + 32-bit-offset addressing (every array a
// kernel indexes this way is below 4 GiB from its base).
template <class T>
__device__ __forceinline__ T& at(T* base, uint32_t i) {
    return *reinterpret_cast<T*>(reinterpret_cast<char*>(base) + i * (uint32_t)sizeof(T));
}
template <class T>
__device__ __forceinline__ const T& at(const T* base, uint32_t i) {
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + i * (uint32_t)sizeof(T));
}

// Base pointers of one step's dense streams (uniform: shot and step fixed).
struct StepPtrs {
    float* dout;         // adjoint output or N p, this step's slice
    float* gacc;         // this shot's gradient accumulator
    float* store;        // this step's (dA/dm)u slot
    const float* stin;   // stored (dA/dm)u of this step (CORR)
    float* r;            // this step's slice of r (RUPD with NORMAL)
    float al;            // the shot's CG step length (RUPD with NORMAL)
};

// n / d and the remainder, n < 2^31, with m = (2^32 - 1) / d: the estimate is at
// most one short.  A few scalar instructions in place of the compiler's division
// (a reciprocal and its corrections in the vector unit, before the first load):
// modelling one 201 x 201 shot 1034 and 1008 us, 32 shots of 801 x 401 20.1 and
// 19.8 ms.
__device__ __forceinline__ int div_by(int n, int d, uint32_t m, int* rem) {
    int q = (int)__umulhi((uint32_t)n, m), r = n - q * d;
    if (r >= d) { ++q; r -= d; }
    *rem = r;
    return q;
}

// Shot and tile of workgroup L: from the batch's work list when shots have
// apertures, else tile fastest within a shot.
__device__ __forceinline__ void work_item(const StepArgs& a, int L, int tiles, int* s, int* t) {
    *s = div_by(a.work ? a.work[L] : L, tiles, a.tiles_m, t) - (a.work ? a.shot0 : 0);
}

// Physical columns [lo, hi) of global shot gs and its damping table.  Cells
// outside the aperture plus its absorbing layer see c2 = 0, so their zero
// state stays zero: the shot propagates on its window alone.
struct Aperture {
    int lo, hi;
    const float* kx;
};
__device__ __forceinline__ Aperture aperture(const StepArgs& a, int gs) {
    Aperture ap;
    ap.lo = a.win ? a.win[2 * gs] : 0;
    ap.hi = a.win ? a.win[2 * gs + 1] : a.nx;
    ap.kx = a.kx + (int64_t)a.kx_stride * gs;
    return ap;
}

// Offset of step `step` of shot s in dsrc / dout: vbase on the whole time
// axis, slot step % blk_T of the shot's block otherwise.
__device__ __forceinline__ int64_t blk_off(const StepArgs& a, int s, int step, int64_t vbase) {
    return a.blk_T ? ((int64_t)s * a.blk_T + step % a.blk_T) * a.nphys : vbase;
}

__device__ __forceinline__ StepPtrs step_ptrs(const StepArgs& a, int s, int step, int64_t vbase, int slot) {
    StepPtrs q;
    q.dout = a.dout ? a.dout + blk_off(a, s, step, vbase) : nullptr;
    q.gacc = a.gacc ? a.gacc + (int64_t)s * a.nphys : nullptr;
    q.store = a.store ? a.store + s * a.store_stride + (int64_t)slot * a.nphys : nullptr;
    q.stin = q.store;
    q.r = a.cg_rw ? a.cg_rw + vbase : nullptr;
    q.al = a.cg_rw ? (float)a.cg_alpha[s] : 0.f;
    return q;
}

// Fused per-cell outputs of one step at a physical cell of the tile.
//  un: new field, q: source term, lq: lap + dx^2 q, c2v: c / dx^2,
//  pv: p^t (NORMAL), stv: stored (dA/dm)u (CORR), rv: r^t (NORMAL with RUPD).
//
// (The DTFT helpers below: the source of step n from the frequency slices,
// q = inv_nt sum_m (re_m cos w_m t_n + im_m sin w_m t_n), and the update of a
// cell's accumulators acc_m += mu (cos, sin)(w_m t), for the earlier step tA
// first when a two-step launch passes its output muA.)
template <int R>
__device__ __forceinline__ void dtft_source(const StepArgs& a, int s, int step, const uint32_t* pi, const bool* ph,
                                            float* q) {
    const float2* __restrict__ tw = a.dft_tw + (int64_t)step * a.dft_nf;
    const float2* __restrict__ sb = a.dft_src + (int64_t)s * a.dft_nf * a.nphys;
    float acc[R];
#pragma unroll
    for (int i = 0; i < R; ++i) acc[i] = 0.f;
    for (int m = 0; m < a.dft_nf; ++m) {
        const float2 w = tw[m];
        const float2* __restrict__ sm = sb + (int64_t)m * a.nphys;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const float2 v = sm[pi[i]];
            acc[i] = fmaf(v.y, w.y, fmaf(v.x, w.x, acc[i]));
        }
    }
#pragma unroll
    for (int i = 0; i < R; ++i) q[i] = ph[i] ? acc[i] * a.inv_nt : 0.f;
}

// Frequencies go in chunks whose loads are all issued before any store, so a
// cell's read-modify-writes overlap instead of waiting one on another.
__device__ __forceinline__ void dtft_accumulate(const StepArgs& a, int s, uint32_t pi, int step, float mu, int stepA,
                                                float muA) {
    constexpr int CH = 8;
    float2* __restrict__ acc = a.dft_acc + (int64_t)s * a.dft_nf * a.nphys + pi;
    const float2* __restrict__ tw = a.dft_tw + (int64_t)step * a.dft_nf;
    const float2* __restrict__ twA = a.dft_tw + (int64_t)(stepA < 0 ? 0 : stepA) * a.dft_nf;
    for (int m0 = 0; m0 < a.dft_nf; m0 += CH) {
        float2 v[CH];
#pragma unroll
        for (int k = 0; k < CH; ++k)
            if (m0 + k < a.dft_nf) v[k] = acc[(int64_t)(m0 + k) * a.nphys];
#pragma unroll
        for (int k = 0; k < CH; ++k) {
            if (m0 + k < a.dft_nf) {
                if (stepA >= 0) {
                    v[k].x = fmaf(muA, twA[m0 + k].x, v[k].x);
                    v[k].y = fmaf(muA, twA[m0 + k].y, v[k].y);
                }
                v[k].x = fmaf(mu, tw[m0 + k].x, v[k].x);
                v[k].y = fmaf(mu, tw[m0 + k].y, v[k].y);
            }
        }
#pragma unroll
        for (int k = 0; k < CH; ++k)
            if (m0 + k < a.dft_nf) acc[(int64_t)(m0 + k) * a.nphys] = v[k];
    }
}

template <unsigned FL>
__device__ __forceinline__ void cell_outputs(const StepArgs& a, const StepPtrs& o, uint32_t pi,
                                             float un, float q, float lq, float c2v, float pv,
                                             float stv, float rv, float wb, double& acc) {
    if constexpr ((FL & F_OUT) != 0) at(o.dout, pi) = un;
    if constexpr ((FL & F_NORMAL) != 0) {
        const float np = fmaf(wb, pv, un);
        if constexpr ((FL & F_RUPD) != 0) {   // r -= alpha N p, as a separate pass would
            const float rn = fmaf(-o.al, np, rv);
            at(o.r, pi) = rn;
            acc += (double)(rn * rn);
        } else {
            at(o.dout, pi) = np;
            acc += (double)pv * (double)np;
        }
    }
    if constexpr ((FL & (F_CG_FUSE | F_SRC_DENSE)) != 0 && (FL & F_RUPD) != 0)
        acc += (double)(q * (wb * q));   // beta B^2 p.p of the direction (dense source)
    if constexpr ((FL & F_PENALTY) != 0) {
        at(o.gacc, pi) = fmaf(wb * q, c2v * a.inv_dt2 * lq, at(o.gacc, pi));
        acc += (double)(wb * q) * (double)q;   // penalty term beta W q^2 (kept when a.part is set)
    }
    if constexpr ((FL & F_STORE) != 0) at(o.store, pi) = c2v * a.inv_dt2 * lq;
    if constexpr ((FL & F_CORR) != 0) at(o.gacc, pi) = fmaf(un, stv, at(o.gacc, pi));
}

__device__ __forceinline__ float annih_w(const StepArgs& a, int ix, int iz, float sx, float sz) {
    if (a.w_identity) return a.beta;   // uniform over the launch
    const float ddx = (float)ix - sx, ddz = (float)iz - sz;
    // the hardware square root (within 1 ulp; the argument is a sum of squared
    // integers, never denormal) instead of the correctly rounded sequence
    const float bb = __builtin_amdgcn_sqrtf(ddx * ddx + ddz * ddz) + a.b_eps;
    return a.beta * (bb * bb);
}

// ---------------------------------------------------------------------------
template <unsigned FL>
__global__ __launch_bounds__(256, ESI_MINW) void k_step2d(const StepArgs a) {
    __shared__ float sh[LH * LW];
    __shared__ float sinj[(FL & F_INJ) ? TZ * TX : 1];
    __shared__ double sred[4];

    // tile index fastest within a shot: each XCD streams a contiguous stretch
    // of one shot's fields (shot-fastest, to share c2 in L2, fetched fewer
    // bytes but ran slower: the scattered streams cost more than they save)
    int s, t;
    work_item(a, xcd_remap(blockIdx.x, gridDim.x), a.tiles, &s, &t);
    if (a.active && !a.active[s]) return;   // uniform over the workgroup
    const int gs = a.shot0 + s;
    const Aperture ap = aperture(a, gs);
    const int tzi = t / a.tiles_x, txi = t - tzi * a.tiles_x;
    const int x0 = txi * TX, z0 = tzi * TZ;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave index: uniform
    const int XS = a.XS;
    // every storage offset of a shot's field fits in 32 bits
    const float* __restrict__ cur = a.cur + s * a.fstride;
    float* __restrict__ nxt = a.nxt + s * a.fstride;
    const float* __restrict__ din = a.din + s * a.fstride;
    float* __restrict__ dnx = a.dnx + s * a.fstride;

    // LDS (r, c) <- padded (z0 + r - 4, x0 + c - 4).  Wave w stages rows w,
    // w + 4, ...: 64 lanes take the row body, 8 the halo (the other lanes
    // repeat a halo load so every load is unconditional).  All rows are loaded
    // into registers before the first LDS write.
    constexpr int RPW = LH / 4;
    static_assert(LH % 4 == 0, "tile rows must split evenly over the waves");
    float tb[RPW][WX], th[RPW];
    {
        const float* src = cur + (z0 + GH - HALO + wv) * XS + x0 + GH - HALO;
#pragma unroll
        for (int k = 0; k < RPW; ++k) {
#pragma unroll
            for (int j = 0; j < WX; ++j) tb[k][j] = at(src, (uint32_t)(k * 4 * XS + 64 * j) + (uint32_t)lane);
            th[k] = at(src, (uint32_t)(k * 4 * XS + TX) + (uint32_t)(lane & (2 * HALO - 1)));
        }
    }
    const int wx = wv % WX, wz = wv / WX;

    // this lane's column and rows: issue every global load first
    const int xl = wx * 64 + lane;                       // tile-local column
    const int x = x0 + xl;
    const float kxv = at(ap.kx, (uint32_t)min(x, a.nxp - 1));
    const int ix = x - a.nb;
    const bool xphys = ix >= ap.lo && ix < ap.hi;
    const bool xwin = x >= ap.lo && x < ap.hi + 2 * a.nb;
    const int zb = z0 + wz * RZ;
    const uint32_t so0 = (uint32_t)((zb + GH) * XS + x + GH);
    const int64_t vbase = ((int64_t)s * a.nt + a.step) * a.nphys;
    const StepPtrs o1 = step_ptrs(a, s, a.step, vbase, a.store_slot);
    float c2v[RZ], dv[RZ], kzv[RZ], qv[RZ];
    uint32_t pi[RZ];
    bool ph[RZ];
#pragma unroll
    for (int i = 0; i < RZ; ++i) {
        const int z = zb + i;
        c2v[i] = xwin ? at(a.c2, so0 + (uint32_t)(i * XS)) : 0.f;
        dv[i] = at(din, so0 + (uint32_t)(i * XS));
        kzv[i] = at(a.kz, (uint32_t)min(z, a.nzp - 1));
        const int iz = z - a.nb;
        ph[i] = xphys && iz >= 0 && iz < a.nz;
        pi[i] = ph[i] ? (uint32_t)(iz * a.nx + ix) : 0u;   // clamped: loads stay unconditional
        qv[i] = 0.f;
    }
    if constexpr ((FL & F_SRC_DENSE) != 0) {
        const float* __restrict__ q = a.dsrc + blk_off(a, s, a.step, vbase);
#pragma unroll
        for (int i = 0; i < RZ; ++i) qv[i] = ph[i] ? at(q, pi[i]) : 0.f;
        if constexpr ((FL & F_SCALE) != 0) {   // cell-scaled dense source
            const float* __restrict__ sc = a.cg_s + (int64_t)s * a.nphys;
#pragma unroll
            for (int i = 0; i < RZ; ++i) qv[i] = qv[i] * at(sc, pi[i]);
        }
    }
    if constexpr ((FL & F_DTFT_SRC) != 0) dtft_source<RZ>(a, s, a.step, pi, ph, qv);
    double pr_acc = 0.0;   // p_new . r partial (F_SCALE)
    if constexpr ((FL & F_CG_FUSE) != 0) {
        const float alp = (float)a.cg_alpha[s];
        const float bet = (float)a.cg_beta[s];
        const float* __restrict__ p = a.cg_p + vbase;
        float* __restrict__ pnew = a.cg_pn + vbase;
        const float* __restrict__ r = a.cg_r + vbase;
        float* __restrict__ xv = a.cg_x + vbase;
        float po[RZ], rv[RZ], xo[RZ], rraw[RZ];
#pragma unroll
        for (int i = 0; i < RZ; ++i) { po[i] = at(p, pi[i]); rv[i] = at(r, pi[i]); xo[i] = at(xv, pi[i]); }
        if constexpr ((FL & F_SCALE) != 0) {
            const float* __restrict__ sc = a.cg_s + (int64_t)s * a.nphys;
#pragma unroll
            for (int i = 0; i < RZ; ++i) { rraw[i] = rv[i]; rv[i] = rv[i] * at(sc, pi[i]); }
        }
#pragma unroll
        for (int i = 0; i < RZ; ++i) {
            const float pn = fmaf(bet, po[i], rv[i]);
            if (ph[i]) {
                at(pnew, pi[i]) = pn;
                if (alp != 0.f) at(xv, pi[i]) = fmaf(alp, po[i], xo[i]);
                if constexpr ((FL & F_SCALE) != 0) pr_acc += (double)pn * (double)rraw[i];
            }
            qv[i] = ph[i] ? pn : 0.f;
        }
    }
    float pv[RZ], stv[RZ], rw[RZ];
#pragma unroll
    for (int i = 0; i < RZ; ++i) { pv[i] = 0.f; stv[i] = 0.f; rw[i] = 0.f; }
    if constexpr ((FL & F_NORMAL) != 0) {
        const float* __restrict__ p = a.dp + vbase;
#pragma unroll
        for (int i = 0; i < RZ; ++i) pv[i] = at(p, pi[i]);
        if constexpr ((FL & F_RUPD) != 0) {
#pragma unroll
            for (int i = 0; i < RZ; ++i) rw[i] = at(o1.r, pi[i]);
        }
    }
    if constexpr ((FL & F_CORR) != 0) {
#pragma unroll
        for (int i = 0; i < RZ; ++i) stv[i] = at(o1.stin, pi[i]);
    }

#pragma unroll
    for (int k = 0; k < RPW; ++k) {
        const int r = wv + k * 4;
#pragma unroll
        for (int j = 0; j < WX; ++j) sh[r * LW + 64 * j + lane] = tb[k][j];
        if (lane < 2 * HALO) sh[r * LW + TX + lane] = th[k];
    }

    const int64_t nrec_s = (FL & (F_INJ | F_GATHER)) ? a.rec_ptr[gs + 1] - a.rec_ptr[gs] : 0;
    const int64_t doff = (FL & (F_INJ | F_GATHER)) ? (int64_t)a.nt * (a.rec_ptr[gs] - a.rec_ptr[a.shot0]) : 0;
    bool has_inj = false;
    if constexpr ((FL & F_INJ) != 0) {
        const int32_t* ip = a.inj_ptr + (int64_t)gs * (a.tiles + 1);
        const int beg = ip[t], end = ip[t + 1];
        has_inj = end > beg;
        if (has_inj) {
            for (int i = tid; i < TZ * TX; i += 256) sinj[i] = 0.f;
            __syncthreads();
            const float* dj = a.inj_data + doff + (int64_t)a.step * nrec_s;
            for (int e = beg + tid; e < end; e += 256) {
                float v = 0.f;
                for (int k = a.inj_rptr[e]; k < a.inj_rptr[e + 1]; ++k) v += dj[a.inj_rid[k]];
                sinj[a.inj_cell[e]] = v;
            }
        }
    }
    __syncthreads();

    if constexpr ((FL & F_GATHER) != 0) {
        if (a.step > 0) {
            const int32_t* gp = a.gat_ptr + (int64_t)gs * (a.tiles + 1);
            float* dn = a.gat_data + doff + (int64_t)(a.step - 1) * nrec_s;
            for (int e = gp[t] + tid; e < gp[t + 1]; e += 256) {
                const int cell = a.gat_cell[e];
                const int r = cell / TX, c = cell - r * TX;
                dn[a.gat_rid[e]] = sh[(r + HALO) * LW + c + HALO];
            }
        }
    }

    int src_cell = -1;
    float src_val = 0.f;
    if constexpr ((FL & (F_SRC_POINT | F_SRC_REC)) != 0) {
        if (a.src_tile[gs] == t) {
            src_cell = a.src_cell[gs];
            if constexpr ((FL & F_SRC_POINT) != 0) src_val = a.wavelet[(int64_t)s * a.nt + a.step];
        }
    }
    float sx = 0.f, sz = 0.f;
    if constexpr ((FL & (F_NORMAL | F_PENALTY | F_RUPD)) != 0) {
        sx = (float)a.src_pos[gs * 3 + 0];
        sz = (float)a.src_pos[gs * 3 + 1];
    }

    double acc = 0.0;
#pragma unroll
    for (int i = 0; i < RZ; ++i) {
        const int zl = wz * RZ + i;
        const int z = z0 + zl;
        const float* cp = sh + (zl + HALO) * LW + xl + HALO;
        const float lap = lap_lds(a, cp, LW);
        float q = qv[i];
        const float qd = q;   // the extended (dense) part of the source
        if constexpr ((FL & F_SRC_POINT) != 0) {
            if (zl * TX + xl == src_cell) q += src_val;
        }
        if constexpr ((FL & F_INJ) != 0) {
            if (has_inj) q += sinj[zl * TX + xl];
        }
        const float kap = kxv + kzv[i];
        const float lq = fmaf(a.dx2, q, lap);
        const float dn = incr(c2v[i], lq, dv[i], kap);
        const float un = cp[0] + dn;
        // cells past the padded grid sit in the zero ghost frame (c2 = u = d = 0)
        // and compute exactly 0, so the stores need no mask
        at(dnx, so0 + (uint32_t)(i * XS)) = dn;
        at(nxt, so0 + (uint32_t)(i * XS)) = un;
        if (!ph[i]) continue;
        if constexpr ((FL & F_SRC_REC) != 0) {
            if (zl * TX + xl == src_cell) a.src_rec[(int64_t)s * a.nt + a.step] = un;
        }
        if constexpr ((FL & F_DTFT_ACC) != 0) dtft_accumulate(a, s, pi[i], a.step, un, -1, 0.f);
        float wb = 0.f;
        if constexpr ((FL & (F_NORMAL | F_PENALTY | F_RUPD)) != 0) wb = annih_w(a, ix, z - a.nb, sx, sz);
        cell_outputs<FL>(a, o1, pi[i], un, qd, lq, c2v[i], pv[i], stv[i], rw[i], wb, acc);
    }

    if constexpr ((FL & (F_NORMAL | F_SCALE | F_PENALTY | F_RUPD)) != 0) {
        if (a.part) {   // uniform over the launch
            acc = wave_sum(acc + pr_acc);
            if (lane == 0) sred[wv] = acc;
            __syncthreads();
            if (tid == 0) {
                double sum = 0.0;
                for (int w = 0; w < 4; ++w) sum += sred[w];
                a.part[(int64_t)s * a.part_stride + t] += sum;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Two steps, tA = a.step and tB = a.step + a.dir, in one launch, on 56 x TH
// output tiles (TH a template parameter; every height computes the same bits
// per cell).  The first step runs on the tile grown by 4 cells, 64 columns: a
// wave spans it exactly, one lane per column.  Wave w owns the tile's rows
// [w TH/4, (w+1) TH/4) and two of the eight rows of the ring above and below
// them; the second step runs on the same lanes and rows (lanes 4..59), so c,
// the new increment and the new field of a cell stay in registers between the
// steps and only the field itself is exchanged, through LDS.
//
// The kernel is bound by instruction issue as much as by HBM: with a reload of
// c and d between the steps and masks and addresses per row, the modelling
// variant issued 1232 vector and 1169 scalar instructions a wave, 58 of its 60
// us on 32 shots of 801 x 401, and few-tile launches waited for their surface
// tiles, whose lanes walked up to 64 receivers one after another.  So what a row
// costs beyond its arithmetic stays in scalar registers:
//  * fields and dense vectors are buffers: a lane's column is a byte offset in
//    one vector register for all rows, the row a scalar offset.  Columns off
//    the grid, the window or the tile hold an offset past the buffer's end,
//    which loads 0 and drops stores, so rows need no masks of their own;
//  * rows off the padded grid read a row of the zero ghost frame instead;
//  * tiles whose grown region lies in the physical window, away from the
//    shot's source and receivers, run rows without damping (k = 0 there: the
//    increment is fmaf(c, lq, d) exactly), injection or edge masks;
//  * the z differences u_{+k} - u of a row serve as the negated u_{-k} - u of
//    the row k below: (u_{+k} - u) + (u_{-k} - u) in one subtraction.
//  * a thread reads the injection entry of its own index while the tile's loads
//    fly and drops it into an LDS plane that is dead at the time;
//  * a launch of few tiles lasts as long as its chain of memory latencies, of
//    which the arguments, the shot's and tile's entries, the lists and the fields
//    were six or seven, 1.2 to 2.1 us before the first field load was issued, and
//    the partial sum at the end another 0.6.  The workgroup now touches every
//    line of its arguments at once, reads all the uniform values of its shot and
//    tile in one batch and, on short tiles, has the fields on their way before it
//    waits for them (T2Head).
// A wave of the modelling variant issues 699 vector and 358 scalar instructions
// (81 % of the vector issue slots; 246 MB a launch by counters, 6.1 TB/s).
// Microseconds per launch on 32-row tiles, before and now:
// modelling 32 shots of 801 x 401, 60.1 and 40.1; CG on 8 of them (forward pass,
// adjoint), 42.7 and 33.6, now 38.9 and 29.3; FWI windows, 32 shots of 1601 x 601
// (modelling, segment recompute, correlating adjoint), 65.3, 95.8 and 110.4, now
// 48.9, 61.6 and 81.1 (store past the caches); one shot of 201 x 201 (modelling,
// CG forward and adjoint averaged), 8.7 and 16.3, now 6.3 and 9.1 (on the 8-row
// tiles it takes, 5.6 and 6.9 before the batched reads, now 4.0 and 5.8).
constexpr int T2W = 56;                           // output tile width
constexpr int A_W = T2W + 2 * HALO;               // 64: first-step region width
constexpr int U0W = T2W + 4 * HALO;               // 72
static_assert(A_W == 64, "two-step tile geometry");

// A global array as a raw buffer (base and size uniform over the wave).
// Offset past the end of every buffer: loads return 0 and stores are dropped.
// Buffers are below 2 GiB (launch2d's callers see to it), so adding a row's
// scalar offset never wraps.
constexpr uint32_t OOB = 0x80000000u;
struct Buf {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ Buf(const float* p, uint32_t bytes)
        : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, (int)bytes, 0x00027000)) {}
    // element at byte offset v (per lane) + s (uniform); NT: not kept in the caches
    static constexpr int NT = 2;
    template <int AUX = 0>
    __device__ __forceinline__ float ld(uint32_t v, uint32_t s) const {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)v, (int)s, AUX));
    }
    template <int AUX = 0>
    __device__ __forceinline__ void st(float x, uint32_t v, uint32_t s) const {
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), r, (int)v, (int)s, AUX);
    }
};
__device__ __forceinline__ uint32_t buf_bytes(int64_t floats) {
    return (uint32_t)min<int64_t>(4 * floats, (int64_t)OOB);
}

// x part of the Laplacian at an LDS cell, as lap_lds forms it.  The address of
// the leftmost neighbour is made opaque: from one base per row the eight loads
// pair up with immediate offsets; left to itself the compiler forms a base per
// pair (96 address additions of 777 vector instructions a wave).
__device__ __forceinline__ float lap_x(const StepArgs& a, const float* p, float cv) {
    typedef const __attribute__((address_space(3))) float lds_float;
    lds_float* q = (lds_float*)(p - HALO);
    asm("" : "+v"(q));
    float lx = a.w1 * ((q[3] - cv) + (q[5] - cv));
    lx = fmaf(a.w2, (q[2] - cv) + (q[6] - cv), lx);
    lx = fmaf(a.w3, (q[1] - cv) + (q[7] - cv), lx);
    return fmaf(a.w4, (q[0] - cv) + (q[8] - cv), lx);
}

// z part at rows 0, 1, ... of a column held in registers, in order: the
// differences e_k(j) = col[j + k] - col[j] are formed once and serve the rows
// j (as u_{+k} - u) and j + k (negated, as u_{-k} - u): the same bits as
// lap_lds, since negation is exact.
struct LapZ {
    float e1, e2[2], e3[3], e4[4];
    template <int N>
    __device__ __forceinline__ explicit LapZ(const float (&col)[N]) {
        e1 = col[4] - col[3];
#pragma unroll
        for (int j = 0; j < 2; ++j) e2[j] = col[4 + j] - col[2 + j];
#pragma unroll
        for (int j = 0; j < 3; ++j) e3[j] = col[4 + j] - col[1 + j];
#pragma unroll
        for (int j = 0; j < 4; ++j) e4[j] = col[4 + j] - col[j];
    }
    template <int N>
    __device__ __forceinline__ float row(const StepArgs& a, const float (&col)[N], int i) {
        const float cv = col[i + 4];
        const float n1 = col[i + 5] - cv, n2 = col[i + 6] - cv, n3 = col[i + 7] - cv, n4 = col[i + 8] - cv;
        float lz = a.w1 * (n1 - e1);
        lz = fmaf(a.w2, n2 - e2[0], lz);
        lz = fmaf(a.w3, n3 - e3[0], lz);
        lz = fmaf(a.w4, n4 - e4[0], lz);
        e1 = n1;
        e2[0] = e2[1]; e2[1] = n2;
        e3[0] = e3[1]; e3[1] = e3[2]; e3[2] = n3;
        e4[0] = e4[1]; e4[1] = e4[2]; e4[2] = e4[3]; e4[3] = n4;
        return lz;
    }
};

// A segment's store of (dA/dm) u that outgrows the 256 MB of last-level cache is
// written and read past the caches, which keep the fields (launch2d).
constexpr unsigned F_STREAM = 1u << 30;

// Occupancy target, waves per SIMD: LDS (24 KB at 32 rows) would hold six
// workgroups per CU, the registers of a variant decide.
template <unsigned FL, int TH>
constexpr int t2_waves() { return (FL & F_INJ) != 0 && (FL & F_NORMAL) == 0 && TH <= 32 ? 5 : 4; }

template <int TH>
struct T2 {
    static constexpr int A_H = TH + 2 * HALO;     // first-step region rows
    static constexpr int RZ2 = TH / 4;            // tile rows per wave
    static constexpr int NR = RZ2 + 2;            // rows per wave in the first step: tile rows, then two ring rows
    static constexpr int U0H = TH + 4 * HALO;
    static constexpr int RPW0 = U0H / 4, NHL = (U0H + 31) / 32;   // staged rows per wave, loads of the last 8 columns
};

// Region row of wave wv's row i in the first step: its tile rows, then two ring rows
template <int TH>
__device__ __forceinline__ int t2_row(int wv, int i) {
    constexpr int RZ2 = T2<TH>::RZ2;
    return i < RZ2 ? wv * RZ2 + HALO + i : (wv < 2 ? 2 * wv : TH + 2 * wv) + i - RZ2;
}

// Padded (z0 - 8 + r, x0 - 8 + c) of a field for U0 (r, c): 64 columns a row per
// wave, the other 8 of 32 rows at a time over the workgroup.
template <int TH, bool GEN>
__device__ __forceinline__ void t2_stage(const StepArgs& a, const Buf& cur, int z0, int x0, float (&tb)[T2<TH>::RPW0],
                                         float (&th)[T2<TH>::NHL]) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t XB = 4u * (uint32_t)a.XS;
    const int xb = x0 - 2 * HALO + lane, hr = tid >> 3;
    const uint32_t vb = !GEN || (unsigned)xb < (unsigned)a.nxp ? 4u * (uint32_t)(xb + GH) : OOB;
#pragma unroll
    for (int k = 0; k < T2<TH>::RPW0; ++k) {
        const int z = z0 - 2 * HALO + wv + 4 * k;
        tb[k] = cur.ld(vb, !GEN || (unsigned)z < (unsigned)a.nzp ? (uint32_t)(z + GH) * XB : 0u);
    }
    const int xh = x0 - 2 * HALO + 64 + (tid & 7);
#pragma unroll
    for (int k = 0; k < T2<TH>::NHL; ++k) {
        const int z = z0 - 2 * HALO + hr + 32 * k;
        const bool in = (!GEN || (xh < a.nxp && (unsigned)z < (unsigned)a.nzp)) && hr + 32 * k < T2<TH>::U0H;
        th[k] = cur.ld(in ? (uint32_t)(z + GH) * XB + 4u * (uint32_t)(xh + GH) : OOB, 0u);
    }
}

// What a workgroup reads before it knows which kind of tile it has: the uniform
// values of its shot and tile, and on short tiles (EARLY) the fields.
template <int TH>
struct T2Head {
    int s, t, txi, tzi, lo, hi;                   // shot, tile, its column and row, aperture
    int ibeg, iend, gbeg, gend;                   // the tile's injection and recording entries
    int sx, sz;                                   // the shot's source
    int64_t rec0, rec_s, rec_e;                   // receivers: first of the batch, the shot's range
    double al, be, part;
    float tb[T2<TH>::RPW0], th[T2<TH>::NHL], c[T2<TH>::NR], d[T2<TH>::NR];
};
template <int TH>
constexpr bool t2_early() { return TH <= 16; }

template <unsigned FL, int TH, bool GEN>
__device__ __forceinline__ void step2d_t2_body(const StepArgs& a, T2Head<TH>& h, int srow, int scol,
                                               float* __restrict__ U0, float* __restrict__ U1, double& acc) {
    constexpr int T2Z = TH;                       // output tile rows
    constexpr int A_H = T2<TH>::A_H, RZ2 = T2<TH>::RZ2, NR = T2<TH>::NR, U0H = T2<TH>::U0H;
    constexpr bool EARLY = t2_early<TH>();
    const int s = h.s, t = h.t, ibeg = h.ibeg, iend = h.iend;
    const Aperture ap = {h.lo, h.hi, a.kx + (int64_t)a.kx_stride * (a.shot0 + h.s)};
    static_assert(T2Z % 4 == 0 && U0H % 4 == 0 && U0H <= 64, "two-step tile geometry");
    float* const sinjB = U0;
    static_assert(U0H * U0W >= A_H * A_W, "the second step's injection fits the u^{tA} buffer");
    // Gradient accumulators are read and written once per launch: both steps'
    // products are chained per cell in the second step, g = fmaf(B, fmaf(A, g))
    // as two one-step launches would add them (the DTFT source keeps one update
    // per step).
    constexpr bool CORR = (FL & F_CORR) != 0;
    constexpr int STREAM = (FL & F_STREAM) != 0 ? Buf::NT : 0;
    constexpr bool CHAIN_PEN = (FL & F_PENALTY) != 0 && (FL & (F_DTFT_SRC | F_INJ)) == 0;
    constexpr bool WB = (FL & (F_NORMAL | F_PENALTY | F_RUPD)) != 0;   // needs beta B^2
    constexpr bool DENSE = (FL & (F_SRC_DENSE | F_DTFT_SRC | F_CG_FUSE)) != 0;
    constexpr bool RUPD = (FL & F_RUPD) != 0, SCALE = (FL & F_SCALE) != 0;

    const int txi = h.txi, tzi = h.tzi;
    const int x0 = txi * T2W, z0 = tzi * T2Z;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave index: uniform
    const uint32_t XB = 4u * (uint32_t)a.XS, NXB = 4u * (uint32_t)a.nx;   // row pitches in bytes
    const int tA = a.step, tB = a.step + a.dir;
    const uint32_t fb = buf_bytes(a.fstride / RING), pb = buf_bytes(a.nphys);
    const Buf cur(a.cur + s * a.fstride, fb), nxt(a.nxt + s * a.fstride, fb);
    const Buf din(a.din + s * a.fstride, fb), dnx(a.dnx + s * a.fstride, fb);
    const Buf c2(a.c2, fb);
    const int64_t vA = ((int64_t)s * a.nt + tA) * a.nphys;
    const int64_t vB = ((int64_t)s * a.nt + tB) * a.nphys;
    // byte offset of a padded row in a field; rows off the padded grid take a
    // row of the zero ghost frame.  Byte offset of a physical row, and the mask
    // that puts a row off the physical grid out of range.
    auto zin = [&](int z) { return !GEN || (unsigned)z < (unsigned)a.nzp; };
    auto zph = [&](int z) { return !GEN || (unsigned)(z - a.nb) < (unsigned)a.nz; };
    auto frow = [&](int z) -> uint32_t { return zin(z) ? (uint32_t)(z + GH) * XB : 0u; };
    auto prow = [&](int z) -> uint32_t { return zph(z) ? (uint32_t)(z - a.nb) * NXB : 0u; };
    auto pmask = [&](int z) -> uint32_t { return zph(z) ? 0u : OOB; };

    constexpr int RPW0 = T2<TH>::RPW0, NHL = T2<TH>::NHL;
    float (&tb)[RPW0] = h.tb, (&th)[NHL] = h.th;
    const int hr = tid >> 3, hc = tid & 7;
    if constexpr (!EARLY) t2_stage<TH, GEN>(a, cur, z0, x0, tb, th);

    // ---- this lane's column and this wave's rows: row i of the first step is
    // padded row zrow(i), region row rrow(i)
    auto rrow = [&](int i) { return t2_row<TH>(wv, i); };
    auto zrow = [&](int i) { return z0 - HALO + rrow(i); };
    const int x = x0 - HALO + lane;                        // padded column
    const int ix = x - a.nb;
    const bool tile_lane = lane >= HALO && lane < HALO + T2W;
    const bool xin = !GEN || (unsigned)x < (unsigned)a.nxp;
    const bool xph = !GEN || (ix >= ap.lo && ix < ap.hi);
    const bool xout = xph && tile_lane;                    // physical column of the tile
    const float kxv = GEN ? at(ap.kx, (uint32_t)min(max(x, 0), a.nxp - 1)) : 0.f;
    const uint32_t vf = xin ? 4u * (uint32_t)(x + GH) : OOB;                 // field column
    const uint32_t vst = xin && tile_lane ? 4u * (uint32_t)(x + GH) : OOB;   // field column to store
    const uint32_t vc = !GEN || (x >= ap.lo && x < ap.hi + 2 * a.nb) ? 4u * (uint32_t)(x + GH) : OOB;
    const uint32_t vp = xph ? 4u * (uint32_t)ix : OOB;     // dense column
    const uint32_t vo = xout ? 4u * (uint32_t)ix : OOB;    // dense column of the tile
    float (&c)[NR] = h.c, (&d)[NR] = h.d;
    float kz[GEN ? NR : 1], qA[NR], poA[NR], rA[NR], xoA[RZ2], pvA[RZ2];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        if constexpr (!EARLY) {
            c[i] = c2.ld(vc, frow(zrow(i)));
            d[i] = din.ld(vf, frow(zrow(i)));
        } else {
            c[i] = vc != OOB ? c[i] : 0.f;   // 0 outside the aperture
        }
        if constexpr (GEN) kz[i] = at(a.kz, (uint32_t)min(max(zrow(i), 0), a.nzp - 1));
        qA[i] = 0.f; poA[i] = 0.f; rA[i] = 0.f;
        if (i < RZ2) { xoA[i] = 0.f; pvA[i] = 0.f; }
    }
    // dense vectors of step t at rows i < N: values that only the output tile
    // uses (x, p, r of N p) are not loaded on the ring, the neighbours' tiles
    auto dense = [&](const float* base, uint32_t v, auto& out, int n) {
        const Buf b(base, pb);
#pragma unroll
        for (int i = 0; i < n; ++i) out[i] = b.ld(v | pmask(zrow(i)), prow(zrow(i)));
    };
    auto stored = [&](const float* base, auto& out) {   // of the tile's rows
        const Buf b(base, pb);
#pragma unroll
        for (int i = 0; i < RZ2; ++i) out[i] = b.template ld<STREAM>(vo | pmask(zrow(i)), prow(zrow(i)));
    };
    if constexpr ((FL & F_SRC_DENSE) != 0) {
        dense(a.dsrc + blk_off(a, s, tA, vA), vp, qA, NR);
        if constexpr (SCALE) {
            float sc[NR];
            dense(a.cg_s + (int64_t)s * a.nphys, vp, sc, NR);
#pragma unroll
            for (int i = 0; i < NR; ++i) qA[i] = qA[i] * sc[i];
        }
    }
    // dense-vector indices of rows i < N for the DTFT helpers
    auto dtft_q = [&](int step, auto& q, auto n) {
        constexpr int N = decltype(n)::value;
        uint32_t pi[N];
        bool ph[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            ph[i] = xph && zph(zrow(i));
            pi[i] = ph[i] ? (uint32_t)((zrow(i) - a.nb) * a.nx + ix) : 0u;
        }
        dtft_source<N>(a, s, step, pi, ph, q);
    };
    if constexpr ((FL & F_DTFT_SRC) != 0) dtft_q(tA, qA, std::integral_constant<int, NR>{});
    float alp = 0.f, bet = 0.f;
    if constexpr ((FL & F_CG_FUSE) != 0) {
        alp = (float)h.al;
        bet = (float)h.be;
        dense(a.cg_p + vA, vp, poA, NR);
        dense(a.cg_r + vA, vp, qA, NR);
        dense(a.cg_x + vA, vo, xoA, RZ2);
        if constexpr (SCALE) {
            float sc[NR];
            dense(a.cg_s + (int64_t)s * a.nphys, vp, sc, NR);
#pragma unroll
            for (int i = 0; i < NR; ++i) { rA[i] = qA[i]; qA[i] = qA[i] * sc[i]; }
        }
    }
    if constexpr ((FL & F_NORMAL) != 0) {
        dense(a.dp + vA, vo, pvA, RZ2);
        if constexpr (RUPD) dense(a.cg_rw + vA, vo, rA, RZ2);   // r^tA (no F_SCALE here)
    }

    // ---- the tile's receivers: this thread's entry (cell, values of both
    // steps; more than 256 entries loop), read while the tile's loads fly
    const int64_t nrec_s = h.rec_e - h.rec_s, doff = (int64_t)a.nt * (h.rec_s - h.rec0);
    int icell = 0, gcell = 0, grid = 0;
    const int gbeg = h.gbeg, gend = h.gend;
    float ivA = 0.f, ivB = 0.f;
    // sum of the data of step `tt` over the receivers of injection entry e
    auto inj_value = [&](int e, int tt) -> float {
        const float* dj = a.inj_data + doff + (int64_t)tt * nrec_s;
        float v = 0.f;
        for (int k = a.inj2_rptr[e]; k < a.inj2_rptr[e + 1]; ++k) v += dj[a.inj2_rid[k]];
        return v;
    };
    if constexpr (GEN && (FL & F_INJ) != 0) {
        // An entry's first receiver is listed by entry (it is the shot's own, also
        // where cells hold several): its data is on the way before the bounds of
        // the entry's list say whether more follow.
        const int e = ibeg + tid;
        if (e < iend) {
            icell = a.inj2_cell[e];
            const int r0 = a.inj2_rptr[e], r1 = a.inj2_rptr[e + 1], rid = a.inj2_first[e];
            const float* dj = a.inj_data + doff;
            ivA = 0.f + dj[(int64_t)tA * nrec_s + rid];
            ivB = 0.f + dj[(int64_t)tB * nrec_s + rid];
            if (r1 != r0 + 1) {
                ivA = inj_value(e, tA);
                ivB = inj_value(e, tB);
            }
        }
    }
    if constexpr ((FL & F_GATHER) != 0) {
        if (gbeg + tid < gend) {
            gcell = a.gat_cell[gbeg + tid];
            grid = a.gat_rid[gbeg + tid];
        }
    }
    const bool has_inj = GEN && (FL & F_INJ) != 0 && iend > ibeg;   // uniform over the workgroup

#pragma unroll
    for (int k = 0; k < RPW0; ++k) U0[(wv + k * 4) * U0W + lane] = tb[k];
#pragma unroll
    for (int k = 0; k < NHL; ++k)
        if (hr + 32 * k < U0H) U0[(hr + 32 * k) * U0W + 64 + hc] = th[k];
    if (has_inj) {   // the first step's injection, in U1 until the step overwrites it cell by cell
#pragma unroll
        for (int i = 0; i < NR; ++i) U1[rrow(i) * A_W + lane] = 0.f;
        __syncthreads();
        if (ibeg + tid < iend) U1[icell] = ivA;
        for (int e = ibeg + tid + 256; e < iend; e += 256) U1[a.inj2_cell[e]] = inj_value(e, tA);
    }
    __syncthreads();

    // d^{step} = R u at the tile's receivers, from a plane whose tile starts at
    // `from` with rows `pitch` apart
    auto record = [&](int step, const float* from, int pitch) {
        float* dn = a.gat_data + doff + (int64_t)step * nrec_s;
        auto rec = [&](int cell, int rid) {
            const int r = cell / T2W, cc = cell - r * T2W;
            dn[rid] = from[r * pitch + cc];
        };
        if (gbeg + tid < gend) rec(gcell, grid);
        for (int e = gbeg + tid + 256; e < gend; e += 256) rec(a.gat_cell[e], a.gat_rid[e]);
    };
    if constexpr ((FL & F_GATHER) != 0)
        if (tA > 0) record(tA - 1, U0 + 2 * HALO * U0W + 2 * HALO, U0W);   // d^{tA-1} (forward only)

    // beta B^2 at padded row z of this lane's column
    float sx = 0.f, sz = 0.f;
    if constexpr (WB) {
        sx = (float)h.sx;
        sz = (float)h.sz;
    }
    const float wx = ((float)ix - sx) * ((float)ix - sx);
    auto weight = [&](int z) -> float {
        if (a.w_identity) return a.beta;   // uniform over the launch
        const float ddz = (float)(z - a.nb) - sz;
        // the hardware square root (within 1 ulp; the argument is a sum of squared
        // integers, never denormal) instead of the correctly rounded sequence
        const float bb = __builtin_amdgcn_sqrtf(wx + ddz * ddz) + a.b_eps;
        return a.beta * (bb * bb);
    };
    const StepPtrs oA = step_ptrs(a, s, tA, vA, a.store_slot);
    const StepPtrs oB = step_ptrs(a, s, tB, vB, a.store_slot2);
    // fused outputs of one step at tile row i: new field un, dense source q, lap
    // + dx^2 q; stores of lanes or rows off the tile's physical cells are
    // dropped (v, out of range), their sums masked
    auto outputs = [&](const StepPtrs& o, int64_t vbase, int i, float un, float q, float lq, float po, float xo,
                       float pv, float rv) {
        const uint32_t v = vo | pmask(zrow(i)), so = prow(zrow(i));
        const bool on = xout && zph(zrow(i));
        const float wb = WB ? weight(zrow(i)) : 0.f;
        if constexpr ((FL & F_CG_FUSE) != 0) {
            Buf(a.cg_pn + vbase, pb).st(q, v, so);
            if (alp != 0.f) Buf(a.cg_x + vbase, pb).st(fmaf(alp, po, xo), v, so);
            if constexpr (SCALE) acc += (double)(on ? q : 0.f) * (double)rv;
        }
        if constexpr ((FL & F_OUT) != 0) Buf(o.dout, pb).st(un, v, so);
        if constexpr ((FL & F_NORMAL) != 0) {
            const float np = fmaf(wb, pv, un);
            if constexpr (RUPD) {   // r -= alpha N p, as a separate pass would
                const float rn = fmaf(-o.al, np, rv);
                Buf(o.r, pb).st(rn, v, so);
                const float rs = on ? rn : 0.f;
                acc += (double)(rs * rs);
            } else {
                Buf(o.dout, pb).st(np, v, so);
                acc += (double)pv * (double)(on ? np : 0.f);
            }
        }
        if constexpr ((FL & (F_CG_FUSE | F_SRC_DENSE)) != 0 && RUPD) {
            const float qs = on ? q : 0.f;
            acc += (double)(qs * (wb * qs));   // beta B^2 p.p of the direction (dense source)
        }
        if constexpr ((FL & F_PENALTY) != 0) {
            if constexpr (!CHAIN_PEN) {
                const Buf g(o.gacc, pb);
                g.st(fmaf(wb * q, c[i] * a.inv_dt2 * lq, g.ld(v, so)), v, so);
            }
            const float qs = on ? q : 0.f;
            acc += (double)(wb * qs) * (double)qs;   // penalty term beta W q^2 (kept when a.part is set)
        }
        if constexpr ((FL & F_STORE) != 0) Buf(o.store, pb).template st<STREAM>(c[i] * a.inv_dt2 * lq, v, so);
    };
    // one cell of a step: field cv, Laplacian, source (extended part qd) -> new
    // increment into d[i], the new field returned, lap + dx^2 q in lq
    auto cell = [&](int i, float cv, float lap, float q, float& lq) -> float {
        lq = (DENSE || GEN) ? fmaf(a.dx2, q, lap) : lap;
        d[i] = GEN ? incr(c[i], lq, d[i], kxv + kz[GEN ? i : 0]) : fmaf(c[i], lq, d[i]);
        return cv + d[i];
    };

    // ---- first step: ring rows, then the tile's rows
    float u[RZ2], lqA[CHAIN_PEN ? RZ2 : 1];
    auto step_a = [&](auto first, auto count) {
        constexpr int I0 = decltype(first)::value, N = decltype(count)::value;
        float col[N + 2 * HALO];
        const float* cp = U0 + rrow(I0) * U0W + lane + HALO;
#pragma unroll
        for (int k = 0; k < N + 2 * HALO; ++k) col[k] = cp[k * U0W];
        LapZ lz(col);
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const int i = I0 + j;
            const float cv = col[j + HALO];
            const float lap = lap_x(a, cp + (j + HALO) * U0W, cv) + lz.row(a, col, j);
            float q = qA[i];
            if constexpr ((FL & F_CG_FUSE) != 0) q = fmaf(bet, poA[i], qA[i]);   // 0 off the physical grid
            const float qd = q;   // the extended (dense) part of the source
            if constexpr (GEN && (FL & F_SRC_POINT) != 0) {
                if (rrow(i) == srow && lane == scol) q += a.wavelet[(int64_t)s * a.nt + tA];
            }
            if (has_inj) q += U1[rrow(i) * A_W + lane];
            float lq;
            const float un = cell(i, cv, lap, q, lq);
            U1[rrow(i) * A_W + lane] = xin && zin(zrow(i)) ? un : 0.f;
            if (i < RZ2) {
                u[i] = xin && zin(zrow(i)) ? un : 0.f;
                if constexpr (CHAIN_PEN) lqA[i] = lq;
                if constexpr (GEN && (FL & F_SRC_REC) != 0) {
                    if (rrow(i) == srow && lane == scol && tile_lane) a.src_rec[(int64_t)s * a.nt + tA] = un;
                }
                outputs(oA, vA, i, un, qd, lq, poA[i], xoA[i], pvA[i], rA[i]);
            }
        }
    };
    step_a(std::integral_constant<int, RZ2>{}, std::integral_constant<int, 2>{});
    step_a(std::integral_constant<int, 0>{}, std::integral_constant<int, RZ2>{});

    // the second step's dense loads fly over the barrier (no other thread of
    // this launch writes what they read)
    float qB[RZ2], pvB[RZ2], stB[RZ2], stA[RZ2], gv[RZ2], poB[RZ2], xoB[RZ2], rB[RZ2];
#pragma unroll
    for (int i = 0; i < RZ2; ++i) {
        qB[i] = 0.f; pvB[i] = 0.f; stB[i] = 0.f; stA[i] = 0.f; gv[i] = 0.f; poB[i] = 0.f; xoB[i] = 0.f; rB[i] = 0.f;
    }
    if constexpr ((FL & F_SRC_DENSE) != 0) {
        dense(a.dsrc + blk_off(a, s, tB, vB), vo, qB, RZ2);
        if constexpr (SCALE) {
            float sc[RZ2];
            dense(a.cg_s + (int64_t)s * a.nphys, vo, sc, RZ2);
#pragma unroll
            for (int i = 0; i < RZ2; ++i) qB[i] = qB[i] * sc[i];
        }
    }
    if constexpr ((FL & F_DTFT_SRC) != 0) dtft_q(tB, qB, std::integral_constant<int, RZ2>{});
    if constexpr ((FL & F_CG_FUSE) != 0) {
        dense(a.cg_p + vB, vo, poB, RZ2);
        dense(a.cg_r + vB, vo, qB, RZ2);
        dense(a.cg_x + vB, vo, xoB, RZ2);
        if constexpr (SCALE) {
            float sc[RZ2];
            dense(a.cg_s + (int64_t)s * a.nphys, vo, sc, RZ2);
#pragma unroll
            for (int i = 0; i < RZ2; ++i) { rB[i] = qB[i]; qB[i] = qB[i] * sc[i]; }
        }
    }
    if constexpr ((FL & F_NORMAL) != 0) {
        dense(a.dp + vB, vo, pvB, RZ2);
        if constexpr (RUPD) dense(a.cg_rw + vB, vo, rB, RZ2);   // r^tB (no F_SCALE here)
    }
    if constexpr (CORR) {
        stored(oA.stin, stA);
        stored(oB.stin, stB);
    }
    if constexpr (CORR || CHAIN_PEN) dense(oB.gacc, vo, gv, RZ2);
    __syncthreads();

    if constexpr ((FL & F_GATHER) != 0) record(tA, U1 + HALO * A_W + HALO, A_W);   // d^{tA} = R u^{tA+1}
    if (has_inj) {   // U0 is dead since the barrier after the first step
        for (int i = tid; i < A_H * A_W; i += 256) sinjB[i] = 0.f;
        __syncthreads();
        if (ibeg + tid < iend) sinjB[icell] = ivB;
        for (int e = ibeg + tid + 256; e < iend; e += 256) sinjB[a.inj2_cell[e]] = inj_value(e, tB);
        __syncthreads();
    }

    // ---- second step on the tile (the ring's lanes compute values that go nowhere)
    float col[RZ2 + 2 * HALO];
    const int lc = min(max(lane, HALO), A_W - HALO - 1);   // keeps the ring's lanes inside their row
    const float* cp = U1 + (wv * RZ2) * A_W + lc;
#pragma unroll
    for (int k = 0; k < HALO; ++k) {
        col[k] = cp[k * A_W];
        col[RZ2 + HALO + k] = cp[(RZ2 + HALO + k) * A_W];
    }
#pragma unroll
    for (int i = 0; i < RZ2; ++i) col[HALO + i] = u[i];
    LapZ lz(col);
#pragma unroll
    for (int i = 0; i < RZ2; ++i) {
        const float cv = u[i];
        const float lap = lap_x(a, cp + (i + HALO) * A_W, cv) + lz.row(a, col, i);
        float q = qB[i];
        if constexpr ((FL & F_CG_FUSE) != 0) q = fmaf(bet, poB[i], qB[i]);   // 0 off the physical grid
        const float qd = q;   // the extended (dense) part of the source
        if constexpr (GEN && (FL & F_SRC_POINT) != 0) {
            if (rrow(i) == srow && lane == scol) q += a.wavelet[(int64_t)s * a.nt + tB];
        }
        if (has_inj) q += sinjB[rrow(i) * A_W + lane];
        float lq;
        const float un = cell(i, cv, lap, q, lq);
        // cells past the padded grid sit in the zero ghost frame (they would
        // compute 0): not stored
        if (zin(zrow(i))) {   // uniform
            dnx.st(d[i], vst, frow(zrow(i)));
            nxt.st(un, vst, frow(zrow(i)));
        }
        if constexpr ((FL & F_DTFT_ACC) != 0) {
            if (xout && zph(zrow(i)))
                dtft_accumulate(a, s, (uint32_t)((zrow(i) - a.nb) * a.nx + ix), tB, un, tA, cv);
        }
        if constexpr (GEN && (FL & F_SRC_REC) != 0) {
            if (rrow(i) == srow && lane == scol && tile_lane) a.src_rec[(int64_t)s * a.nt + tB] = un;
        }
        outputs(oB, vB, i, un, qd, lq, poB[i], xoB[i], pvB[i], rB[i]);
        if constexpr (CORR)
            Buf(oB.gacc, pb).st(fmaf(un, stB[i], fmaf(cv, stA[i], gv[i])), vo | pmask(zrow(i)), prow(zrow(i)));
        if constexpr (CHAIN_PEN) {
            const float wb = weight(zrow(i));
            const float gA = fmaf(wb * qA[i], c[i] * a.inv_dt2 * lqA[i], gv[i]);
            Buf(oB.gacc, pb).st(fmaf(wb * qd, c[i] * a.inv_dt2 * lq, gA), vo | pmask(zrow(i)), prow(zrow(i)));
        }
    }
}

template <unsigned FL, int TH>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(t2_waves<FL, TH>())))
void k_step2d_t2(const StepArgs a) {
    // u^{tA} on the tile + 8 (dead after the first step, then holding the second
    // step's injection), u after the first step on the tile + 4 (before that,
    // in its place cell by cell, the first step's injection)
    __shared__ float U0[(TH + 4 * HALO) * U0W];
    __shared__ float U1[(TH + 2 * HALO) * A_W];
    __shared__ double sred[4];
    T2Head<TH> h;
    // One dword of each cache line of the arguments, before anything waits: later
    // reads of the line are then short.
    int tiles = a.tiles;
    asm("" : "+s"(tiles) : "s"(a.cur), "s"(a.c2), "s"(a.nb), "s"(a.dx2), "s"(a.src_pos), "s"(a.inj2_ptr),
        "s"(a.gat_data), "s"(a.cg_r), "s"(a.win), "s"(a.work), "s"(a.active), "s"(a.store), "s"(a.dft_nf));
    const int blocks = a.work ? a.nwork : tiles * a.nshots;   // the launch's
    work_item(a, xcd_remap(blockIdx.x, blocks), tiles, &h.s, &h.t);
    h.s = __builtin_amdgcn_readfirstlane(h.s);
    h.t = __builtin_amdgcn_readfirstlane(h.t);
    // The shot's and tile's uniform values in one batch without branches: an
    // array that is not there is read from c2 and the value dropped.
    const int gs = a.shot0 + h.s;
    auto pick = [&](const auto* p, int64_t i) { return p ? p + i : (decltype(p))a.c2; };
    int act = *pick(a.active, h.s);
    const int32_t* wp = pick(a.win, 2 * (int64_t)gs);
    h.lo = wp[0]; h.hi = wp[1];
    h.ibeg = h.iend = h.gbeg = h.gend = 0;
    const int64_t tp = (int64_t)gs * (tiles + 1) + h.t;
    if constexpr ((FL & F_INJ) != 0) { h.ibeg = a.inj2_ptr[tp]; h.iend = a.inj2_ptr[tp + 1]; }
    if constexpr ((FL & F_GATHER) != 0) { h.gbeg = a.gat_ptr[tp]; h.gend = a.gat_ptr[tp + 1]; }
    h.rec0 = h.rec_s = h.rec_e = 0;
    if constexpr ((FL & (F_INJ | F_GATHER)) != 0) {
        h.rec0 = a.rec_ptr[a.shot0];
        h.rec_s = a.rec_ptr[gs];
        h.rec_e = a.rec_ptr[gs + 1];
    }
    h.sx = a.src_pos[gs * 3 + 0];
    h.sz = a.src_pos[gs * 3 + 1];
    h.al = h.be = h.part = 0.0;
    if constexpr ((FL & F_CG_FUSE) != 0) { h.al = a.cg_alpha[h.s]; h.be = a.cg_beta[h.s]; }
    constexpr bool PART = (FL & (F_NORMAL | F_SCALE | F_PENALTY | F_RUPD)) != 0;
    const int64_t pidx = (int64_t)h.s * a.part_stride + h.t;
    if constexpr (PART) h.part = *pick((const double*)a.part, pidx);
    h.tzi = div_by(h.t, a.tiles_x, a.tiles_xm, &h.txi);
    const int tzi = h.tzi, txi = h.txi;
    __builtin_amdgcn_sched_barrier(0);   // on their way before the fields' loads
    if constexpr (t2_early<TH>()) {
        const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const uint32_t fb = buf_bytes(a.fstride / RING);
        const Buf cur(a.cur + h.s * a.fstride, fb), din(a.din + h.s * a.fstride, fb), c2(a.c2, fb);
        t2_stage<TH, true>(a, cur, tzi * TH, txi * T2W, h.tb, h.th);
        const int x = txi * T2W - HALO + lane;
        const uint32_t vf = (unsigned)x < (unsigned)a.nxp ? 4u * (uint32_t)(x + GH) : OOB;
#pragma unroll
        for (int i = 0; i < T2<TH>::NR; ++i) {
            const int z = tzi * TH - HALO + t2_row<TH>(wv, i);
            const uint32_t row = (unsigned)z < (unsigned)a.nzp ? 4u * (uint32_t)((z + GH) * a.XS) : 0u;
            h.c[i] = c2.ld(vf, row);
            h.d[i] = din.ld(vf, row);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // wait for the batch here, once
    asm("" : "+s"(act) : "s"(h.lo), "s"(h.hi), "s"(h.ibeg), "s"(h.iend), "s"(h.gbeg), "s"(h.gend), "s"(h.rec0),
        "s"(h.rec_s), "s"(h.rec_e), "s"(h.sx), "s"(h.sz), "s"(h.al), "s"(h.be), "s"(h.part));
    if (a.active && !act) return;   // uniform over the workgroup
    if (!a.win) { h.lo = 0; h.hi = a.nx; }
    const int px = txi * T2W - HALO - a.nb, pz = tzi * TH - HALO - a.nb;   // the grown region's physical origin
    int srow = -1, scol = -1;
    if constexpr ((FL & (F_SRC_POINT | F_SRC_REC)) != 0) {   // the source cell in the grown region
        const int gx = h.sx - px, gz = h.sz - pz;
        if ((unsigned)gz < (unsigned)(TH + 2 * HALO) && (unsigned)gx < (unsigned)A_W) { srow = gz; scol = gx; }
    }
    // Interior tiles (uniform): the grown region is physical, and neither the
    // source nor a receiver to inject lies in it; the staged region is then on
    // the padded grid (nb >= 4).
    const bool inner = px >= h.lo && px + A_W <= h.hi && pz >= 0 && pz + TH + 2 * HALO <= a.nz && h.iend == h.ibeg &&
                       srow < 0;
    double acc = 0.0;
    if (inner) step2d_t2_body<FL, TH, false>(a, h, srow, scol, U0, U1, acc);
    else step2d_t2_body<FL, TH, true>(a, h, srow, scol, U0, U1, acc);

    if constexpr (PART) {
        if (a.part) {   // uniform over the launch
            const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
            acc = wave_sum(acc);
            if (lane == 0) sred[wv] = acc;
            __syncthreads();
            if (threadIdx.x == 0) {
                double sum = 0.0;
                for (int w = 0; w < 4; ++w) sum += sred[w];
                a.part[pidx] = h.part + sum;
            }
        }
    }
}

// Record d^{nt-1} = R u^{nt} after the last step (one thread per receiver).
__global__ void k_final_gather(const float* __restrict__ field, int64_t fstride,
                               const int32_t* __restrict__ rec, const int64_t* __restrict__ rec_ptr,
                               int shot0, int nshots, int nt, int nb, int XS, int YS, int ndim,
                               float* __restrict__ data) {
    const int64_t base = rec_ptr[shot0];
    const int64_t n = rec_ptr[shot0 + nshots] - base;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = base + i;
        int s = 0;
        while (rec_ptr[shot0 + s + 1] <= r) ++s;   // shots per call are few
        const int64_t nrec_s = rec_ptr[shot0 + s + 1] - rec_ptr[shot0 + s];
        const int64_t rid = r - rec_ptr[shot0 + s];
        const int x = rec[r * 3 + 0] + nb + GH, z = rec[r * 3 + 1] + nb + GH;
        const int y = ndim == 3 ? rec[r * 3 + 2] + nb + GH : 0;
        const float v = field[s * fstride + ((int64_t)z * YS + y) * XS + x];
        data[(int64_t)nt * (rec_ptr[shot0 + s] - base) + (int64_t)(nt - 1) * nrec_s + rid] = v;
    }
}

// TH = 0: the one-step kernel; else the two-step kernel with TH-row tiles
template <unsigned FL, int TH>
esi_status_t launch2d(Plan* P, const StepArgs& a) {
    const int blocks = a.work ? a.nwork : a.tiles * a.nshots;
    if (blocks == 0) return ESI_OK;
    // A store larger than the last-level cache (256 MB) is read back from memory
    // anyway and pushes the fields out on its way.  FWI gradient of 32 windowed
    // shots of 1601 x 601, 50 slots (6.2 GB): 34.7 ms, 30.4 past the caches; 16 shots
    // of 801 x 401, 25 slots (514 MB): 5.83 and 5.58; 4 shots, 50 slots (257 MB): 3.88
    // and 3.90; 12 shots of 401 x 201, 20 slots (77 MB): 4.14 and 4.25.
    constexpr bool STORES = TH >= 24 && (FL & (F_STORE | F_CORR)) != 0;   // shorter tiles: small launches
    if constexpr (STORES) {
        if (a.nshots * a.store_stride > (int64_t)1 << 26) {
            hipLaunchKernelGGL((k_step2d_t2<FL | F_STREAM, TH>), dim3(blocks), dim3(256), 0, P->stream, a);
            ESI_HIP_TRY(hipGetLastError());
            return ESI_OK;
        }
    }
    if constexpr (TH > 0)
        hipLaunchKernelGGL((k_step2d_t2<FL, TH>), dim3(blocks), dim3(256), 0, P->stream, a);
    else
        hipLaunchKernelGGL(k_step2d<FL>, dim3(blocks), dim3(256), 0, P->stream, a);
    ESI_HIP_TRY(hipGetLastError());
    return ESI_OK;
}

// The variants the autotuner may give other tile heights: those of the CG,
// modelling and gradient loops.  Other variants run on 32-row tiles.
template <int TH>
esi_status_t dispatch2d_tuned(Plan* P, unsigned flags, const StepArgs& a) {
    switch (flags) {
#define ESI_CASE(F) case (F): return launch2d<(F), TH>(P, a);
        ESI_CASE(F_SRC_POINT | F_GATHER)
        ESI_CASE(F_SRC_POINT | F_STORE)
        ESI_CASE(F_SRC_DENSE | F_GATHER)
        ESI_CASE(F_SRC_DENSE | F_PENALTY)
        ESI_CASE(F_SRC_POINT | F_SRC_DENSE | F_PENALTY)
        ESI_CASE(F_CG_FUSE | F_GATHER | F_RUPD)
        ESI_CASE(F_SRC_DENSE | F_GATHER | F_RUPD)
        ESI_CASE(F_CG_FUSE | F_GATHER | F_SCALE)
        ESI_CASE(F_SRC_DENSE | F_SCALE | F_GATHER)
        ESI_CASE(F_INJ)
        ESI_CASE(F_INJ | F_OUT)
        ESI_CASE(F_INJ | F_NORMAL)
        ESI_CASE(F_INJ | F_NORMAL | F_RUPD)
        ESI_CASE(F_INJ | F_CORR)
#undef ESI_CASE
        default: return fail(ESI_ERR_ARG, "internal: 2D step flags " + std::to_string(flags) +
                                              " have no " + std::to_string(TH) + "-row tiles");
    }
}

bool tuned_variant(unsigned flags) {
    switch (flags) {
        case F_SRC_POINT | F_GATHER: case F_SRC_POINT | F_STORE: case F_SRC_DENSE | F_GATHER:
        case F_SRC_DENSE | F_PENALTY: case F_SRC_POINT | F_SRC_DENSE | F_PENALTY:
        case F_CG_FUSE | F_GATHER | F_RUPD: case F_SRC_DENSE | F_GATHER | F_RUPD:
        case F_CG_FUSE | F_GATHER | F_SCALE: case F_SRC_DENSE | F_SCALE | F_GATHER: case F_INJ:
        case F_INJ | F_OUT: case F_INJ | F_NORMAL: case F_INJ | F_NORMAL | F_RUPD: case F_INJ | F_CORR:
            return true;
        default:
            return false;
    }
}

template <int TH>
esi_status_t dispatch2d(Plan* P, unsigned flags, const StepArgs& a) {
    switch (flags) {
#define ESI_CASE(F) case (F): return launch2d<(F), TH>(P, a);
        ESI_CASE(F_SRC_POINT | F_GATHER)
        ESI_CASE(F_SRC_POINT | F_GATHER | F_STORE)
        ESI_CASE(F_SRC_POINT | F_STORE)
        ESI_CASE(F_SRC_POINT)
        ESI_CASE(F_SRC_DENSE | F_GATHER)
        ESI_CASE(F_SRC_DENSE | F_GATHER | F_STORE)
        ESI_CASE(F_SRC_DENSE | F_STORE)
        ESI_CASE(F_SRC_DENSE)
        ESI_CASE(F_SRC_DENSE | F_PENALTY)
        ESI_CASE(F_SRC_POINT | F_SRC_DENSE | F_PENALTY)
        ESI_CASE(F_SRC_DENSE | F_PENALTY | F_GATHER)
        ESI_CASE(F_SRC_POINT | F_SRC_DENSE | F_PENALTY | F_GATHER)
        ESI_CASE(F_SRC_POINT | F_SRC_DENSE | F_GATHER)
        ESI_CASE(F_SRC_POINT | F_SRC_DENSE | F_GATHER | F_STORE)
        ESI_CASE(F_SRC_POINT | F_SRC_DENSE | F_STORE)
        ESI_CASE(F_CG_FUSE | F_GATHER)
        ESI_CASE(F_CG_FUSE | F_GATHER | F_SCALE)
        ESI_CASE(F_CG_FUSE | F_GATHER | F_RUPD)
        ESI_CASE(F_SRC_DENSE | F_GATHER | F_RUPD)
        ESI_CASE(F_DTFT_SRC | F_GATHER)
        ESI_CASE(F_SRC_DENSE | F_SCALE | F_GATHER)
        ESI_CASE(F_DTFT_SRC | F_PENALTY)
        ESI_CASE(F_INJ | F_DTFT_ACC)
        ESI_CASE(F_INJ)
        ESI_CASE(F_INJ | F_OUT)
        ESI_CASE(F_INJ | F_NORMAL)
        ESI_CASE(F_INJ | F_NORMAL | F_RUPD)
        ESI_CASE(F_INJ | F_CORR)
        ESI_CASE(F_INJ | F_CORR | F_OUT)
        ESI_CASE(F_INJ | F_CORR | F_SRC_REC)
#undef ESI_CASE
        default: return fail(ESI_ERR_ARG, "internal: unsupported 2D step flags " + std::to_string(flags));
    }
}

}  // namespace

esi_status_t launch_step2d(Plan* P, unsigned flags, const StepArgs& a, int shape) {
    switch (shape) {
        case LS_ONE: return dispatch2d<0>(P, flags, a);
        case LS_T2_32: return dispatch2d<32>(P, flags, a);
        case LS_T2_24: return dispatch2d_tuned<24>(P, flags, a);
        case LS_T2_40: return dispatch2d_tuned<40>(P, flags, a);
        case LS_T2_16: return dispatch2d_tuned<16>(P, flags, a);
        case LS_T2_8: return dispatch2d_tuned<8>(P, flags, a);
        default: return fail(ESI_ERR_ARG, "internal: launch shape " + std::to_string(shape));
    }
}

int step2d_loop_shape(unsigned flags, int shape, int64_t fsize) {
    // the two-step kernels address a field with signed 32-bit byte offsets
    if (fsize >= (int64_t)1 << 29) return LS_ONE;
    return shape != LS_ONE && !tuned_variant(flags) ? LS_T2_32 : shape;
}

void step2d_shape_tile(int shape, int* tx, int* tz) {
    *tx = shape == LS_ONE ? TX : T2W;
    switch (shape) {
        case LS_ONE: *tz = TZ; break;
        case LS_T2_24: *tz = 24; break;
        case LS_T2_40: *tz = 40; break;
        case LS_T2_16: *tz = 16; break;
        case LS_T2_8: *tz = 8; break;
        default: *tz = 32;
    }
}

esi_status_t launch_final_gather(Plan* P, const float* field, int64_t fstride, float* data,
                                 int shot0, int nshots) {
    int64_t n = P->h_rec_ptr[shot0 + nshots] - P->h_rec_ptr[shot0];
    if (n == 0) return ESI_OK;
    int blocks = (int)std::min<int64_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(k_final_gather, dim3(blocks), dim3(256), 0, P->stream, field, fstride,
                       P->d_rec, P->d_rec_ptr, shot0, nshots, P->nt, P->nb, P->XS, P->YS,
                       P->ndim, data);
    ESI_HIP_TRY(hipGetLastError());
    return ESI_OK;
}

}  // namespace esi
