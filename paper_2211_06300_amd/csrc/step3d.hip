// One time step of the 3D 8th-order acoustic scheme (Sec. 4.1) with the same
// fused work as the 2D kernels (injection, recording, CG direction update,
// N p with p.Np partials, gradient correlations).
//
// 2.5D sweep: a 512-thread workgroup owns a 64 (x) x 16 (y) block of columns
// and a chunk of z-planes (step3d_chunk); a thread owns two columns, the
// adjacent rows 2 ly and 2 ly + 1, whose y neighbours overlap.  Each thread
// keeps the z windows of its columns in registers; the current plane of the
// block plus a 4-cell x/y halo is staged in a double-buffered LDS plane, so one
// barrier per plane suffices.
// Receiver injection is applied per plane through a small LDS plane; the
// recording reads u^n straight from memory.  Storage is the padded grid with
// a zero ghost frame of GH cells, planes YS x XS floats apart.
//
// Fields and dense vectors are raw buffers that start at the chunk's first
// plane: a column is a byte offset in a vector register for all planes, the
// plane a scalar offset, and columns off the grid hold an offset past the
// buffer's end, which loads 0 and drops stores.  Planes of blocks inside the
// physical grid run without damping (k = 0 there: the increment is fmaf(c, lq,
// d) exactly), injection or source.  The march advances UZ planes at a time,
// so that the windows move once per UZ planes.  Microseconds per launch, before
// (addresses and masks per plane, receivers counted one by one, 32-plane
// chunks) and now, modelling / segment recompute / adjoint / correlating
// adjoint: one shot of 64^3, 32.4 / 35.6 / 52.4 / 60.8, now 8.5 / 8.9 / 9.8 / 11.1;
// 4 shots of 256^3, 560 / 662 / 591 / 888, now 509 / 589 / 530 / 755.  The latter
// moves 2.79 GB a modelling launch by counters (20 B a cell are 2.07), 5.5 TB/s:
// halo planes that neither L2 nor a neighbour still holds.  Non-temporal loads
// or stores of the streams without reuse were slower by 7 to 27 % (they pass
// the memory-side cache by), loads two planes ahead by nothing.
#include <type_traits>

#include "esi_internal.h"

namespace esi {

namespace {

constexpr int TX = 64, WY = 8, RY = 2;     // threads: 64 x 8, two rows each
constexpr int TY = WY * RY, TZC = 32;      // block of columns; storage rounds z to TZC planes
constexpr int UZ = 4;                      // planes per turn of the march
constexpr int NTH = TX * WY;               // 512 threads
constexpr int PW = TX + 2 * HALO, PH = TY + 2 * HALO;   // staged plane 72 x 24
constexpr int NHALO = PW * PH - TX * TY;   // 704 halo cells per plane
constexpr int WIN = 2 * HALO + UZ;         // z window of a turn
static_assert(NHALO <= 2 * NTH && NHALO >= NTH, "two halo cells per thread");
static_assert(UZ == 4, "the march spells out four planes; LDS planes alternate by their place in a turn");

__device__ __forceinline__ int xcd_remap(int b, int nblocks) {
    const int per = nblocks / XCDS, rem = nblocks % XCDS;
    const int xcd = b % XCDS, idx = b / XCDS;
    return xcd < rem ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
}

template <class T>
__device__ __forceinline__ const T& at(const T* base, uint32_t i) {
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + i * (uint32_t)sizeof(T));
}

// A global array as a raw buffer (base and size uniform over the wave).  OOB is
// past the end of every buffer; buffers are cut below 2 GiB, which no chunk of
// planes reaches, so adding a plane's scalar offset never wraps.
constexpr uint32_t OOB = 0x80000000u;
struct Buf {
    __amdgpu_buffer_rsrc_t r;
    // (the size is formed by scalar instructions alone: in a vector register the
    // compiler would loop over the lanes' descriptors at every access)
    __device__ __forceinline__ Buf(const float* p, int64_t floats)
        : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0,
                                              (int)(((uint64_t)floats >> 29) != 0 ? OOB : 4u * (uint32_t)floats),
                                              0x00027000)) {}
    __device__ __forceinline__ float ld(uint32_t v, uint32_t s) const {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)v, (int)s, 0));
    }
    __device__ __forceinline__ void st(float x, uint32_t v, uint32_t s) const {
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), r, (int)v, (int)s, 0);
    }
};

template <unsigned FL>
__global__ __launch_bounds__(NTH) void k_step3d(const StepArgs a) {
    __shared__ float P[2][PH * PW];
    __shared__ float sinj[(FL & F_INJ) ? TX * TY : 1];
    __shared__ double sred[NTH / 64];
    constexpr bool DENSE = (FL & (F_SRC_DENSE | F_CG_FUSE)) != 0;
    constexpr bool RUPD = (FL & F_RUPD) != 0, CORR = (FL & F_CORR) != 0;
    constexpr bool WB = (FL & (F_NORMAL | F_PENALTY | F_RUPD)) != 0;

    const int L = xcd_remap(blockIdx.x, gridDim.x);
    const int s = __builtin_amdgcn_readfirstlane(L / a.tiles);
    const int t = L - s * a.tiles;
    if (a.active && !a.active[s]) return;   // uniform over the workgroup
    const int gs = a.shot0 + s;
    const int tzi = __builtin_amdgcn_readfirstlane(t / (a.tiles_x * a.tiles_y));
    const int rem = t - tzi * a.tiles_x * a.tiles_y;
    const int tyi = __builtin_amdgcn_readfirstlane(rem / a.tiles_x), txi = rem - tyi * a.tiles_x;
    const int x0 = txi * TX, y0 = tyi * TY, zc0 = tzi * a.chunk;
    const int zend = min(zc0 + a.chunk, a.nzp);
    const int tid = threadIdx.x, lx = tid & 63;
    const int ly = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int XS = a.XS, YS = a.YS;
    const uint32_t PB = 4u * (uint32_t)(YS * XS);            // bytes of a field plane
    const uint32_t QB = 4u * (uint32_t)(a.ny * a.nx);        // bytes of a dense plane

    // fields from storage plane zc0 - 4 + GH on; padded plane z is plane z - zc0 + 4 there
    const int64_t f0 = (int64_t)(zc0 - HALO + GH) * YS * XS, fn = a.fstride / 4 - f0;
    const Buf cur(a.cur + s * a.fstride + f0, fn), nxt(a.nxt + s * a.fstride + f0, fn);
    const Buf din(a.din + s * a.fstride + f0, fn), dnx(a.dnx + s * a.fstride + f0, fn);
    const Buf c2(a.c2 + f0, fn);
    // dense vectors from the chunk's first physical plane on
    const int iz0 = min(max(zc0 - a.nb, 0), a.nz - 1);
    const int64_t q0 = (int64_t)iz0 * a.ny * a.nx, qn = a.nphys - q0;
    const int64_t vbase = ((int64_t)s * a.nt + a.step) * a.nphys;
    // dsrc / dout hold the whole time axis, or blk_T steps (step n in slot n % blk_T)
    const int64_t vblk = a.blk_T ? ((int64_t)s * a.blk_T + a.step % a.blk_T) * a.nphys : vbase;
    const int64_t sbase = (int64_t)s * a.nphys;
    auto dense = [&](const float* base, int64_t off) { return Buf(base + off + q0, qn); };
    const Buf bq = dense((FL & F_SRC_DENSE) ? a.dsrc : a.c2, (FL & F_SRC_DENSE) ? vblk : 0);
    const Buf bout = dense((FL & (F_OUT | F_NORMAL)) ? a.dout : a.nxt, (FL & (F_OUT | F_NORMAL)) ? vblk : 0);
    const Buf bsc = dense((FL & F_SCALE) ? a.cg_s : a.c2, (FL & F_SCALE) ? sbase : 0);
    const Buf bp = dense((FL & F_NORMAL) ? a.dp : (FL & F_CG_FUSE) ? a.cg_p : a.c2,
                         (FL & (F_NORMAL | F_CG_FUSE)) ? vbase : 0);
    const Buf br = dense((FL & F_NORMAL) && RUPD ? a.cg_rw : (FL & F_CG_FUSE) ? a.cg_r : a.c2,
                         ((FL & F_NORMAL) && RUPD) || (FL & F_CG_FUSE) ? vbase : 0);
    const Buf bpn = dense((FL & F_CG_FUSE) ? a.cg_pn : a.c2, (FL & F_CG_FUSE) ? vbase : 0);
    const Buf bx = dense((FL & F_CG_FUSE) ? a.cg_x : a.c2, (FL & F_CG_FUSE) ? vbase : 0);
    const Buf bg = dense((FL & (F_PENALTY | F_CORR)) ? a.gacc : a.c2, (FL & (F_PENALTY | F_CORR)) ? sbase : 0);
    constexpr bool ST = (FL & (F_STORE | F_CORR)) != 0;
    const Buf bst = dense(ST ? a.store : a.c2, ST ? s * a.store_stride + (int64_t)a.store_slot * a.nphys : 0);
    // paired correlation: this launch also adds the previous step's product,
    // its input field times store slot store_slot2, first (uniform)
    const bool pair = CORR && a.corr_pair;
    const Buf bst2 = dense(CORR ? a.store : a.c2,
                           CORR && pair ? s * a.store_stride + (int64_t)a.store_slot2 * a.nphys : 0);
    const float ral = ((FL & F_NORMAL) && RUPD) ? (float)a.cg_alpha[s] : 0.f;
    const float alp = (FL & F_CG_FUSE) ? (float)a.cg_alpha[s] : 0.f, bet = (FL & F_CG_FUSE) ? (float)a.cg_beta[s] : 0.f;

    // this thread's columns: rows yl + r of the block
    const int x = x0 + lx, ix = x - a.nb, yl = ly * RY;
    uint32_t vf[RY], vp[RY];    // byte offsets in a field and a dense plane, OOB off the grid
    float kxy[RY];
#pragma unroll
    for (int r = 0; r < RY; ++r) {
        const int y = y0 + yl + r, iy = y - a.nb;
        vf[r] = x < a.nxp && y < a.nyp ? 4u * (uint32_t)((y + GH) * XS + x + GH) : OOB;
        vp[r] = ix >= 0 && ix < a.nx && iy >= 0 && iy < a.ny ? 4u * (uint32_t)(iy * a.nx + ix) : OOB;
        kxy[r] = at(a.kx, (uint32_t)min(x, a.nxp - 1)) + at(a.ky, (uint32_t)min(y, a.nyp - 1));
    }
    // the block's columns are physical: no damping on its physical planes
    const bool inner = x0 >= a.nb && x0 + TX <= a.nx + a.nb && y0 >= a.nb && y0 + TY <= a.ny + a.nb;
    // halo cells this thread stages (the second one: threads below NHALO - NTH)
    int hl[2];
    uint32_t ho[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        int h = min(tid + k * NTH, NHALO - 1);
        int ry, rx;
        if (h < 2 * HALO * PW) {                          // y-halo slabs, full width
            ry = h / PW;
            rx = h - ry * PW;
            if (ry >= HALO) ry += TY;
        } else {                                          // x-halo, body rows
            h -= 2 * HALO * PW;
            ry = HALO + h / (2 * HALO);
            rx = h % (2 * HALO);
            if (rx >= HALO) rx += TX;
        }
        const int hx = x0 - HALO + rx, hy = y0 - HALO + ry;
        hl[k] = ry * PW + rx;
        ho[k] = (tid + k * NTH < NHALO && hx >= 0 && hx < a.nxp && hy >= 0 && hy < a.nyp)
                    ? 4u * (uint32_t)((hy + GH) * XS + hx + GH) : OOB;
    }
    const bool halo2 = ly < (NHALO - NTH) / 64;           // uniform over the wave
    static_assert((NHALO - NTH) % 64 == 0, "whole waves stage the second halo cells");

    // z windows: w[r][k] = u at z - 4 + k for the turn's first plane z; planes
    // off the padded grid are the zero ghost frame.  A plane's own loads (the
    // windows' new values, the halo cells, c, d) are issued one plane ahead,
    // before the barrier of the plane in between, so their latency overlaps
    // that plane's stencil work.
    float w[RY][WIN];
#pragma unroll
    for (int k = 0; k < 2 * HALO; ++k)
#pragma unroll
        for (int r = 0; r < RY; ++r) w[r][k] = cur.ld(vf[r], (uint32_t)k * PB);
    float nw[RY], nc[RY], nd[RY], nh[2], nk;   // the next plane's loads
    const Buf bk(a.kz, a.nzp);
    auto fetch = [&](int z) {
        const uint32_t pz = (uint32_t)(z - zc0 + HALO) * PB;
        nk = bk.ld(0u, 4u * (uint32_t)z);
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            nw[r] = cur.ld(vf[r], pz + 4u * PB);
            nc[r] = c2.ld(vf[r], pz);
            nd[r] = din.ld(vf[r], pz);
        }
        nh[0] = cur.ld(ho[0], pz);
        nh[1] = cur.ld(ho[1], pz);
    };
    fetch(zc0);

    const int64_t nrec_s = (FL & (F_INJ | F_GATHER)) ? a.rec_ptr[gs + 1] - a.rec_ptr[gs] : 0;
    const int64_t doff = (FL & (F_INJ | F_GATHER)) ? (int64_t)a.nt * (a.rec_ptr[gs] - a.rec_ptr[a.shot0]) : 0;
    if constexpr ((FL & F_GATHER) != 0) {
        // d^{n-1} = R u^n for the receivers of this block, straight from u^n
        if (a.step > 0) {
            const int32_t* gp = a.gat_ptr + (int64_t)gs * (a.tiles + 1);
            const float* u = a.cur + s * a.fstride;
            float* dn = a.gat_data + doff + (int64_t)(a.step - 1) * nrec_s;
            for (int e = gp[t] + tid; e < gp[t + 1]; e += NTH) {
                const int cell = a.gat_cell[e];
                const int lz = cell / (TX * TY), r2 = cell - lz * TX * TY;
                const int cy = r2 / TX, cx = r2 - cy * TX;
                dn[a.gat_rid[e]] = u[((int64_t)(zc0 + lz + GH) * YS + y0 + cy + GH) * XS + x0 + cx + GH];
            }
        }
    }
    // injection entries are sorted by cell, i.e. by plane first: `ie` is the
    // first one not yet injected, ilz its plane of the chunk.  This thread's
    // entry of the first NTH is read here; later ones when their plane comes.
    int ie = 0, ibeg = 0, iend = 0, ilz = -1, pcell = -1;
    float pval = 0.f;
    const float* dj = nullptr;
    auto inj_value = [&](int e) -> float {
        float v = 0.f;
        for (int k = a.inj_rptr[e]; k < a.inj_rptr[e + 1]; ++k) v += dj[a.inj_rid[k]];
        return v;
    };
    if constexpr ((FL & F_INJ) != 0) {
        const int32_t* ip = a.inj_ptr + (int64_t)gs * (a.tiles + 1);
        ie = ibeg = ip[t];
        iend = ip[t + 1];
        dj = a.inj_data + doff + (int64_t)a.step * nrec_s;
        if (ie < iend) ilz = a.inj_cell[ie] / (TX * TY);
        if (ie + tid < iend) {
            pcell = a.inj_cell[ie + tid];
            pval = inj_value(ie + tid);
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
    const int src_lz = src_cell < 0 ? -1 : src_cell / (TX * TY);
    float sx = 0.f, sy = 0.f, sz = 0.f;
    if constexpr (WB) {
        sx = (float)a.src_pos[gs * 3 + 0];
        sz = (float)a.src_pos[gs * 3 + 1];
        sy = (float)a.src_pos[gs * 3 + 2];
    }

    double acc = 0.0;
    // plane z, the K-th of its turn
    auto plane = [&](int z, auto place) {
        constexpr int K = decltype(place)::value;
        const int lz = z - zc0, iz = z - a.nb;
        const uint32_t pz = (uint32_t)(lz + HALO) * PB;
        float* Pb = P[K & 1];
        float c2v[RY], dv[RY];
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            w[r][K + 2 * HALO] = nw[r];
            Pb[(yl + r + HALO) * PW + lx + HALO] = w[r][K + HALO];
            c2v[r] = nc[r];
            dv[r] = nd[r];
        }
        Pb[hl[0]] = nh[0];
        if (halo2) Pb[hl[1]] = nh[1];
        const float kz = nk;
        // this plane's dense loads
        const bool zp = iz >= 0 && iz < a.nz;               // uniform
        const uint32_t zm = zp ? 0u : OOB, qz = zp ? (uint32_t)(iz - iz0) * QB : 0u;
        float q[RY], po[RY], xo[RY], pv[RY], stv[RY], rv[RY], gv[RY], stp[RY];
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            const uint32_t v = vp[r] | zm;
            q[r] = 0.f; po[r] = 0.f; xo[r] = 0.f; pv[r] = 0.f; stv[r] = 0.f; rv[r] = 0.f; gv[r] = 0.f; stp[r] = 0.f;
            if constexpr ((FL & F_SRC_DENSE) != 0) {
                q[r] = bq.ld(v, qz);
                if constexpr ((FL & F_SCALE) != 0) q[r] = q[r] * bsc.ld(v, qz);   // cell-scaled dense source
            }
            if constexpr ((FL & F_CG_FUSE) != 0) {
                po[r] = bp.ld(v, qz);
                xo[r] = bx.ld(v, qz);
                q[r] = fmaf(bet, po[r], br.ld(v, qz));   // 0 off the physical grid
            }
            if constexpr ((FL & F_NORMAL) != 0) {
                pv[r] = bp.ld(v, qz);
                if constexpr (RUPD) rv[r] = br.ld(v, qz);
            }
            // the accumulator is read here, with the other dense loads, so that
            // its latency overlaps the plane's stencil work
            if constexpr ((FL & (F_PENALTY | F_CORR)) != 0) gv[r] = bg.ld(v, qz);
            if constexpr (CORR) {
                stv[r] = bst.ld(v, qz);
                if (pair) stp[r] = bst2.ld(v, qz);
            }
        }
        bool inj_here = false;
        if constexpr ((FL & F_INJ) != 0) {
            if (lz == ilz) {   // uniform: entries of this plane
                inj_here = true;
                __syncthreads();                  // the last injection plane has been read
                for (int i = tid; i < TX * TY; i += NTH) sinj[i] = 0.f;
                __syncthreads();
                for (int n = NTH; n == NTH;) {
                    // entries ie + tid below ibeg + NTH are held by the threads that read them
                    const bool held = ie < ibeg + NTH;
                    const int e = held ? ibeg + tid : ie + tid;
                    const int cell = e < iend ? (held ? pcell : a.inj_cell[e]) : -1;
                    const bool here = e >= ie && e < iend && cell / (TX * TY) == lz;
                    if (here) sinj[cell - lz * TX * TY] = held ? pval : inj_value(e);
                    const int got = __syncthreads_count(here);
                    ie += got;
                    // more of this plane may follow the last entry looked at
                    n = ie == (held ? ibeg + NTH : e - tid + NTH) ? NTH : 0;
                }
                ilz = ie < iend ? a.inj_cell[ie] / (TX * TY) : -1;
            }
        }
        if (z + 1 < zend) fetch(z + 1);           // uniform over the workgroup
        __syncthreads();
        const float* cpl = Pb + (yl + HALO) * PW + lx + HALO;
        float yv[RY + 2 * HALO];   // the column pair's plane values, rows yl - 4 .. yl + RY + 3
#pragma unroll
        for (int k = 0; k < HALO; ++k) {
            yv[k] = cpl[(k - HALO) * PW];
            yv[RY + HALO + k] = cpl[(RY + k) * PW];
        }
#pragma unroll
        for (int r = 0; r < RY; ++r) yv[HALO + r] = w[r][K + HALO];
        auto cells = [&](auto general) {
            constexpr bool GEN = decltype(general)::value;
#pragma unroll
            for (int r = 0; r < RY; ++r) {
                const float* cp = cpl + r * PW;
                const float* ww = &w[r][K];
                const float* yy = &yv[r];
                const float cv = ww[HALO];
                float lx_ = a.w1 * ((cp[-1] - cv) + (cp[1] - cv));
                lx_ = fmaf(a.w2, (cp[-2] - cv) + (cp[2] - cv), lx_);
                lx_ = fmaf(a.w3, (cp[-3] - cv) + (cp[3] - cv), lx_);
                lx_ = fmaf(a.w4, (cp[-4] - cv) + (cp[4] - cv), lx_);
                float ly_ = a.w1 * ((yy[3] - cv) + (yy[5] - cv));
                ly_ = fmaf(a.w2, (yy[2] - cv) + (yy[6] - cv), ly_);
                ly_ = fmaf(a.w3, (yy[1] - cv) + (yy[7] - cv), ly_);
                ly_ = fmaf(a.w4, (yy[0] - cv) + (yy[8] - cv), ly_);
                float lz_ = a.w1 * ((ww[3] - cv) + (ww[5] - cv));
                lz_ = fmaf(a.w2, (ww[2] - cv) + (ww[6] - cv), lz_);
                lz_ = fmaf(a.w3, (ww[1] - cv) + (ww[7] - cv), lz_);
                lz_ = fmaf(a.w4, (ww[0] - cv) + (ww[8] - cv), lz_);
                const float lap = (lx_ + ly_) + lz_;
                const int pcl = (yl + r) * TX + lx;             // cell within the plane
                float qq = q[r];
                const float qd = qq;   // the extended (dense) part of the source
                bool src = false;
                if constexpr (GEN && (FL & (F_SRC_POINT | F_SRC_REC)) != 0) src = lz * TX * TY + pcl == src_cell;
                if constexpr (GEN && (FL & F_SRC_POINT) != 0) {
                    if (src) qq += src_val;
                }
                if constexpr (GEN && (FL & F_INJ) != 0) {
                    if (inj_here) qq += sinj[pcl];
                }
                const float lq = (DENSE || GEN) ? fmaf(a.dx2, qq, lap) : lap;
                const float kap = kxy[r] + kz;
                const float dn = GEN ? fmaf(c2v[r], lq, (1.f - kap) * dv[r]) * __builtin_amdgcn_rcpf(1.f + kap)
                                     : fmaf(c2v[r], lq, dv[r]);
                const float un = cv + dn;
                // cells past the padded grid sit in the zero ghost frame (they
                // would compute 0): neither loaded nor stored
                dnx.st(dn, vf[r], pz);
                nxt.st(un, vf[r], pz);
                // outputs on physical cells: stores elsewhere are dropped, sums masked
                const uint32_t v = vp[r] | zm;
                const bool on = vp[r] != OOB && zp;
                if constexpr ((FL & F_CG_FUSE) != 0) {
                    bpn.st(qd, v, qz);
                    if (alp != 0.f) bx.st(fmaf(alp, po[r], xo[r]), v, qz);
                }
                if constexpr ((FL & F_OUT) != 0) bout.st(un, v, qz);
                if constexpr (GEN && (FL & F_SRC_REC) != 0) {
                    if (src) a.src_rec[(int64_t)s * a.nt + a.step] = un;
                }
                float wb = 0.f;
                if constexpr (WB) {
                    if (a.w_identity) {
                        wb = a.beta;
                    } else {
                        // the hardware square root (within 1 ulp; the argument
                        // is a sum of squared integers, never denormal)
                        const float ddx = (float)ix - sx, ddy = (float)(y0 + yl + r - a.nb) - sy, ddz = (float)iz - sz;
                        const float bb = __builtin_amdgcn_sqrtf(ddx * ddx + ddy * ddy + ddz * ddz) + a.b_eps;
                        wb = a.beta * (bb * bb);
                    }
                }
                if constexpr (DENSE && RUPD)
                    acc += (double)(qd * (wb * qd));   // beta B^2 p.p of the direction (0 off the grid)
                if constexpr ((FL & F_NORMAL) != 0) {
                    const float np = fmaf(wb, pv[r], un);
                    if constexpr (RUPD) {   // r -= alpha N p, as a separate pass would
                        const float rn = fmaf(-ral, np, rv[r]);
                        br.st(rn, v, qz);
                        const float rs = on ? rn : 0.f;
                        acc += (double)(rs * rs);
                    } else {
                        bout.st(np, v, qz);
                        acc += (double)pv[r] * (double)(on ? np : 0.f);
                    }
                }
                if constexpr ((FL & F_PENALTY) != 0) {
                    bg.st(fmaf(wb * qd, c2v[r] * a.inv_dt2 * lq, gv[r]), v, qz);
                    acc += (double)(wb * qd) * (double)qd;   // penalty term (kept when a.part is set)
                }
                if constexpr ((FL & F_STORE) != 0) bst.st(c2v[r] * a.inv_dt2 * lq, v, qz);
                if constexpr (CORR) {
                    // the previous step's product first, as a two-step launch chains them
                    const float g = pair ? fmaf(cv, stp[r], gv[r]) : gv[r];
                    bg.st(fmaf(un, stv[r], g), v, qz);
                }
            }
        };
        if (inner && zp && !inj_here && lz != src_lz) cells(std::false_type{});
        else cells(std::true_type{});
    };
    for (int z = zc0; z < zend; z += UZ) {
        plane(z, std::integral_constant<int, 0>{});
        if (z + 1 < zend) plane(z + 1, std::integral_constant<int, 1>{});
        if (z + 2 < zend) plane(z + 2, std::integral_constant<int, 2>{});
        if (z + 3 < zend) plane(z + 3, std::integral_constant<int, 3>{});
#pragma unroll
        for (int r = 0; r < RY; ++r)
#pragma unroll
            for (int k = 0; k < 2 * HALO; ++k) w[r][k] = w[r][k + UZ];
    }

    if constexpr (WB) {
        if (a.part) {   // uniform over the launch
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
            if (lx == 0) sred[ly] = acc;
            __syncthreads();
            if (tid == 0) {
                double sum = 0.0;
                for (int k = 0; k < NTH / 64; ++k) sum += sred[k];
                a.part[(int64_t)s * a.part_stride + t] += sum;
            }
        }
    }
}

template <unsigned FL>
esi_status_t launch3d(Plan* P, const StepArgs& a) {
    const int blocks = a.tiles * a.nshots;
    hipLaunchKernelGGL(k_step3d<FL>, dim3(blocks), dim3(NTH), 0, P->stream, a);
    ESI_HIP_TRY(hipGetLastError());
    return ESI_OK;
}

}  // namespace

esi_status_t launch_step3d(Plan* P, unsigned flags, const StepArgs& a) {
    switch (flags) {
#define ESI_CASE(F) case (F): return launch3d<(F)>(P, a);
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
        ESI_CASE(F_CG_FUSE | F_GATHER | F_RUPD)
        ESI_CASE(F_SRC_DENSE | F_GATHER | F_RUPD)
        ESI_CASE(F_SRC_DENSE | F_SCALE | F_GATHER)
        ESI_CASE(F_INJ)
        ESI_CASE(F_INJ | F_OUT)
        ESI_CASE(F_INJ | F_SRC_REC)
        ESI_CASE(F_INJ | F_NORMAL)
        ESI_CASE(F_INJ | F_NORMAL | F_RUPD)
        ESI_CASE(F_INJ | F_CORR)
        ESI_CASE(F_INJ | F_CORR | F_OUT)
        ESI_CASE(F_INJ | F_CORR | F_SRC_REC)
#undef ESI_CASE
        default: return fail(ESI_ERR_ARG, "internal: unsupported 3D step flags " + std::to_string(flags));
    }
}

// Planes per chunk for a plan of `nshots` shots, `plane` floats per field plane.
// A launch takes as long as the CU with most workgroups: their count over the
// CUs, rounded up, times the planes of each and 0.7 for the 8 planes of u that a
// chunk reads beyond its own.  Alone on its CU a workgroup hides little of its
// latency, and two hold together.  Microseconds per step, modelling / gradient
// (averaged over its three passes), n^3 grids with nb 20, by planes (workgroups):
//   40, 1 shot:    3 (270)  8.2 / 8.8    4 (200)  7.3 / 8.0    8 (100) 10.1 / 11.2
//   48, 1 shot:    3 (360)  8.5 / 9.2    4 (264)  9.2 / 10.1   5 (216)  8.3 / 9.2
//   64, 1 shot:    3 (490)  8.7 / 9.5    4 (364)  9.6 / 10.6   6 (252)  9.1 / 10.1
//   64, 2 shots:   4 (728) 13.7 / 16.2   6 (504) 13.0 / 15.1   8 (364) 15.3 / 17.3
//   96, 1 shot:    4 (918) 16.0 / 18.3   6 (621) 16.9 / 19.5   8 (459) 15.2 / 17.5
//   163, 1 shot:   4 (2652) 39.7 / 52.3  7 (1508) 36.6 / 51.3  8 (1352) 40.7 / 53.6
//   256, 4 shots:  4 (28120)  565 / 638  8 (14060)  524 / 609  16 (7220)  545 / 640
int step3d_chunk(int nxp, int nyp, int nzp, int64_t plane, int nshots) {
    constexpr int64_t CUS = 256;
    const int64_t columns = (int64_t)nshots * ((nxp + TX - 1) / TX) * ((nyp + TY - 1) / TY);
    // a chunk with its halo must not pass 2 GiB, which buffers cannot: shorter
    // chunks where 3 planes would, none (0) where one would (planes of 53 million floats)
    auto fits = [&](int ch) { return (ch + 2 * HALO + 1) * 4 * plane < (int64_t)1 << 31; };
    int best = fits(2) ? 2 : fits(1) ? 1 : 0;
    int64_t least = INT64_MAX;
    for (int ch = 3; ch <= 8 && fits(ch); ++ch) {
        const int64_t rounds = (columns * ((nzp + ch - 1) / ch) + CUS - 1) / CUS;
        const int64_t cost = rounds * (10 * ch + 7) * (rounds == 1 ? 117 : rounds == 2 ? 97 : 100);
        if (cost <= least) { least = cost; best = ch; }
    }
    return best;
}

// (host only, for tests)
extern "C" int esi_host_step3d_chunk(int nxp, int nyp, int nzp, int64_t plane, int nshots) {
    return step3d_chunk(nxp, nyp, nzp, plane, nshots);
}

void step3d_tile_shape(int* tx, int* ty, int* tz) { *tx = TX; *ty = TY; *tz = TZC; }

}  // namespace esi
