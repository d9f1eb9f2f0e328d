// Learned preconditioner network: a four-level U-Net (channels 16/32/64/128)
// with bfloat16 weights and activations and float32 accumulation, trained and
// run entirely by the kernels below.  The paper leaves the preconditioner of
// its CG open (Sec. 4.2 and Sec. 6: fewer inner iterations need an efficient
// preconditioner); the network, its loss and its use are this library's.
//
// Activations are NHWC bfloat16 (channels contiguous, 16-byte aligned groups
// of eight).  A decoder level's concatenation [upsampled, skip] is one buffer
// of two planar halves, each a dense NHWC tensor of ch channels: the
// transposed convolution writes the first, the encoder's second convolution
// writes its output straight into the second, and the decoder's first
// convolution reads the pair as 2 ch channels.  The skip costs no copy, and
// no kernel writes part of another's cache lines.
//
// 3x3 convolutions (forward and data gradient) are implicit GEMMs on
// v_mfma_f32_16x16x32_bf16: D[cout][pixel] = sum_{tap, ci} W[tap][cout][ci]
// X[pixel + tap][ci], with each input tile staged in LDS once and read by all
// nine taps, and the weights packed in the instruction's operand order.  The
// data gradient is the same kernel with taps reversed and weights transposed.
// Transposed convolutions use the same instruction with operands loaded
// straight from memory (each input pixel is read once); their data gradient
// uses v_mfma_f32_16x16x16_bf16.  The weight gradients are GEMMs over pixels on
// the K = 32 instruction, with NHWC tiles in LDS read pixel-major by transposing
// loads (split into fixed chunks, partials summed in a fixed order).
#include <cmath>
#include <cstring>
#include <type_traits>
#include <vector>

#include "esi_internal.h"

namespace esi {
namespace {

typedef uint16_t bf16_t;
typedef short s4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
union bf8u {   // eight bf16 values as one 16-byte load or store
    uint4 u;
    uint16_t h[8];
};

constexpr int NT = 256;

__device__ __forceinline__ float bf2f(bf16_t h) { return __uint_as_float((uint32_t)h << 16); }
// round to nearest even (finite inputs)
__device__ __forceinline__ bf16_t f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}
static uint16_t f2bf_host(float f) {
    uint32_t u;
    std::memcpy(&u, &f, 4);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// ---------------------------------------------------------------------------
// 3x3 convolution, same size, zero padding, as an implicit GEMM on
// v_mfma_f32_16x16x32_bf16: D[m][pixel] = sum over (tap, k) of
// A[tap][m][k] X[pixel + tap][k].  X and Y are NHWC views with pixel strides
// sx, sy (elements); K input and M output channels, multiples of 16.  A view
// may hold its channels as two planar halves: channels from xsplit on
// (ysplit for Y) live xhs (yhs) elements further on, at channel c - xsplit.
//
// The contraction runs in blocks of 32: (tap, 32 channels) when K is a
// multiple of 32 (CK = 32, nine blocks per chunk of 32 channels), else (two
// taps, 16 channels) (CK = 16, five blocks, the tenth tap with zero weights).
// Lane l of a block holds the 8 consecutive contraction indices of k-group
// l / 16, for row (A) or pixel (B) l % 16; A is packed in that order by
// k_pack_frag, so a lane's weights are one coalesced 16-byte load.
//
// Workgroup (x, y): NWV waves, each RPW output rows of PG groups of 16 of the tile's
// 64 pixels, the 16 CB output channels of group y.  Per chunk of CK input channels
// the (rows + 2) x 66 input tile is staged in LDS once and every tap reads its
// shifted operands from there: at two rows a wave and CK = 32 an operand read
// serves the taps of both rows.  The weights stay in registers for the whole
// launch where a layer has one chunk and they fit (RES), else they are staged in
// LDS with the chunk.
//
// The grid is persistent: workgroup x takes tiles x, x + gridDim.x, ...  The
// global loads of the next (tile, chunk) are issued before the current one's
// MFMAs and land in registers, so memory latency overlaps the arithmetic; a
// tile's outputs are stored after its last chunk.
//
// Around the MFMAs it is the vector instructions that cost (a 64-wide one takes
// as long as a quarter of an MFMA), so there are few: tiles are walked by scalar
// additions, loads and stores are raw buffers with a per-lane offset that is
// fixed but for the image's edges and a scalar one per row, and outputs are
// rounded two at a time by the instruction.  Stores are 16 bytes a lane (8 bytes
// left four partial writes in a line: 467 us for the pass below against 428).
// The layers of 16 channels are bound by memory (37 us for 223 MB by counters, 6 TB/s), the
// others by the last wave of tiles and what it leaves exposed: 64 channels on 8
// images of 102 x 202 have 416 tiles for 256 CUs (28 us, of which 8 MFMAs).
// The forward pass on 8 images of 408 x 808 takes 428 to 441 us; with 1369 vector
// instructions for 144 MFMAs (now 513), pooling and first and last layer as
// kernels of their own, it took 652.
constexpr int frag_ck(int K) { return K % 32 == 0 ? 32 : 16; }
constexpr int frag_nkb(int ck) { return ck == 32 ? 9 : 5; }

enum Epi {
    E_FWD,    // bias, ReLU
    E_POOL,   // and the 2x2 average of the outputs (of their bf16 values) into `pool`
    E_OUT,    // and the 1x1 output layer (16 -> 1) of the outputs into `o`; Y only if given
    E_GRAD,   // data gradient: as it is
    E_MASK    // outputs where `act` (laid out as Y, no halves) is not positive are 0
};

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
constexpr uint32_t OOB = 0x80000000u;   // byte offset beyond every buffer: loads 0, stores nothing

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* p) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)OOB, 0x00027000);
}
// two floats to bf16, round to nearest even
__device__ __forceinline__ uint32_t pk_bf16(float a, float b) {
    union { bf16x2 v; uint32_t u; } r;
    r.v = bf16x2{(__bf16)a, (__bf16)b};
    return r.u;
}
__device__ __forceinline__ float bf_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf_hi(uint32_t u) { return __uint_as_float(u & 0xFFFF0000u); }
// the value of lane l ^ 1
__device__ __forceinline__ uint32_t lane_pair(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true);
}

// Lane 16 g + j of u and v holds outputs 4 g .. 4 g + 3 (8 bytes) of pixel j of a
// block of 16 outputs each; now 8 consecutive outputs of one: g = 0 and 2 the
// halves of u, g = 1 and 3 those of v.
__device__ __forceinline__ u32x4 merge_blocks(u32x2 u, u32x2 v) {
    const auto x = __builtin_amdgcn_permlane16_swap(u.x, v.x, false, false);
    const auto y = __builtin_amdgcn_permlane16_swap(u.y, v.y, false, false);
    return u32x4{x[0], y[0], x[1], y[1]};
}

// 16-byte buffer stores go without a scalar offset: with one, the compiler puts
// no wait between the store and the next write of its data registers, and the
// first dword of half the lanes was then stored with that next value.
__device__ __forceinline__ void store16(u32x4 v, __amdgpu_buffer_rsrc_t r, uint32_t off) {
    __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)off, 0, 0);
}
// the inverse of merge_blocks
__device__ __forceinline__ void split_blocks(u32x4 m, u32x2& u, u32x2& v) {
    const auto x = __builtin_amdgcn_permlane16_swap(m.x, m.z, false, false);
    const auto y = __builtin_amdgcn_permlane16_swap(m.y, m.w, false, false);
    u = u32x2{x[0], y[0]};
    v = u32x2{x[1], y[1]};
}

struct ConvArgs {
    const bf16_t* X;
    int sx;
    int64_t xhs;
    int xsplit, K;
    const bf16_t* Af;
    int ncb;                // 16-row blocks of A
    const float* bias;
    bf16_t* Y;
    int sy;
    int64_t yhs;
    int ysplit, H, W, N;
    const bf16_t* act;      // E_MASK
    bf16_t* pool;           // E_POOL: [N][H/2][W/2][sy]
    const bf16_t* wo;       // E_OUT: weights, bias, output [N][H][W]
    const float* bo;
    float* o;
    const float* xin;       // IN: the network's input [N][3][H][W] in place of X
};

template <int CB, int CK, int PG>
struct Conv3Tile {
    static constexpr int RPW = 2, ROWS = 8;               // output rows of a wave and of a tile
    static constexpr int NWV = 4 * ROWS / (RPW * PG);     // waves: 4 groups of pixels a row, PG a wave
    static constexpr int NTW = 64 * NWV;                  // threads of a workgroup
    static constexpr int NKB = frag_nkb(CK);
    static constexpr int TR = ROWS + 2, TC = 66, SUB = CK / 8;
    static constexpr int RPL = NTW / (64 * SUB);          // tile rows per load, but for the last two columns
    static constexpr int NL = (TR + RPL - 1) / RPL;
    static constexpr int NWL = (NKB * CB + NWV - 1) / NWV;   // weight blocks a wave stages
};

template <int CB, int CK, int PG, int EPI, bool RES, bool IN>
__global__ __launch_bounds__(64 * (16 / PG)) __attribute__((amdgpu_waves_per_eu(2))) void k_conv3(const ConvArgs A) {
    using T = Conv3Tile<CB, CK, PG>;
    constexpr int RPW = T::RPW, NWV = T::NWV;
    constexpr int TC = T::TC, TR = T::TR, SUB = T::SUB, NKB = T::NKB;
    static_assert(T::RPL >= 1 && TR * 2 * SUB <= T::NTW, "tile staging");
    static_assert(EPI != E_OUT || (CB == 1 && PG == 4), "the output layer reads 16 channels");
    static_assert(!IN || CK == 16, "the input is padded to 16 channels");
    __shared__ __align__(16) bf16_t xs[TR * TC * CK];
    __shared__ __align__(16) bf16_t ws[RES ? 8 : NKB * CB * 512];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int jl = lane & 15, g = lane >> 4;
    const int wy = wave / (4 / PG) * RPW, wx = wave % (4 / PG) * (PG * 16);   // the wave's first row and pixel
    const int H = A.H, W = A.W, nchunk = RES ? 1 : A.K / CK, cb0 = blockIdx.y * CB;
    const int ntx = (W + 63) / 64, nty = (H + T::ROWS - 1) / T::ROWS;
    const int nmine = (ntx * nty * A.N - 1 - (int)blockIdx.x) / (int)gridDim.x + 1;   // gridDim.x <= tiles

    // tile walk: this workgroup's tile and the stride gridDim.x, as (x, y, image)
    int tx = blockIdx.x % ntx, ty = (blockIdx.x / ntx) % nty, tn = blockIdx.x / (ntx * nty);
    const int gx = gridDim.x % ntx, gy = (gridDim.x / ntx) % nty, gn = gridDim.x / (ntx * nty);

    // ---- staging: thread -> (row of a load, column, 16-byte piece); one more
    // load for the tile's last two columns
    uint4 st[T::NL + 1], sw[T::NWL];
    float fi[T::NL + 1][3];
    constexpr int IL = (TR + NWV - 1) / NWV;
    const int wrow = IN ? wave : wave / SUB;
    const int mpx = IN ? lane : (tid % (64 * SUB)) / SUB, msub = IN ? 0 : tid % SUB;
    const int hrow = IN ? tid >> 1 : tid / (2 * SUB);
    const int hpx = IN ? 64 + (tid & 1) : 64 + (tid % (2 * SUB)) / SUB;
    uint32_t moff, hoff;
    if constexpr (IN) {
        moff = 4 * mpx;
        hoff = 4 * (hrow * W + hpx);
    } else {
        // channels at or past xsplit inside the only chunk: second half
        const uint32_t sec = A.xsplit < CK && msub * 8 >= A.xsplit ? (uint32_t)(2 * (A.xhs - A.xsplit)) : 0u;
        moff = 2 * (mpx * A.sx + msub * 8) + sec;
        hoff = 2 * ((hrow * W + hpx) * A.sx + msub * 8) + sec;
    }
    const bool hin = hrow < TR;
    const __amdgpu_buffer_rsrc_t ra = rsrc(A.Af);
    // (unconditional, with every lane out of bounds when there is nothing to load:
    // registers loaded on one path only are copied, and waited for, at the join)
    auto fetch = [&](int x, int y, int n, int chunk, bool any) {
        const int x0 = x * 64, y0 = y * T::ROWS;
        const uint32_t mo = any && (uint32_t)(x0 - 1 + mpx) < (uint32_t)W ? moff : OOB;
        const uint32_t ho = any && hin && (uint32_t)(y0 - 1 + hrow) < (uint32_t)H && x0 - 1 + hpx < W ? hoff : OOB;
        if constexpr (IN) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const __amdgpu_buffer_rsrc_t rx = rsrc(A.xin + ((int64_t)n * 3 + c) * H * W - 1 - W);
#pragma unroll
                for (int l = 0; l < IL; ++l) {
                    const int row = l * NWV + wave, yy = y0 - 1 + row;
                    const bool ok = (uint32_t)yy < (uint32_t)H && row < TR;
                    fi[l][c] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                        rx, (int)(ok ? mo : OOB), 4 * ((yy + 1) * W + x0), 0));
                }
                fi[IL][c] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rx, (int)ho, 4 * (y0 * W + x0), 0));
            }
        } else {
            const int ch = chunk * CK;
            // from one pixel and one row before the tile's first: offsets stay positive
            const __amdgpu_buffer_rsrc_t rx =
                rsrc(A.X + ((int64_t)n * H * W - 1 - W) * A.sx + ch + (ch >= A.xsplit ? A.xhs - A.xsplit : 0));
#pragma unroll
            for (int l = 0; l < T::NL; ++l) {
                const int row = l * T::RPL + wrow, yy = y0 - 1 + row;
                const bool ok = (uint32_t)yy < (uint32_t)H && row < TR;
                const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)(ok ? mo : OOB),
                                                                     2 * ((yy + 1) * W + x0) * A.sx, 0);
                st[l] = uint4{v.x, v.y, v.z, v.w};
            }
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)ho, 2 * (y0 * W + x0) * A.sx, 0);
            st[T::NL] = uint4{v.x, v.y, v.z, v.w};
        }
    };
    // the workgroup's weight blocks of a chunk: [kb][c][lane][8]
    auto wblock = [&](int chunk, int f, int off) -> uint4 {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(
            ra, off, (((chunk * NKB + f / CB) * A.ncb + cb0 + f % CB) * 1024), 0);
        return uint4{v.x, v.y, v.z, v.w};
    };
    auto wfetch = [&](int chunk, bool any) {
        const int off = any ? lane * 16 : (int)OOB;
#pragma unroll
        for (int l = 0; l < T::NWL; ++l) sw[l] = wblock(chunk, min(l * NWV + wave, NKB * CB - 1), off);
    };
    auto put = [&]() {
        if constexpr (IN) {
#pragma unroll
            for (int l = 0; l <= IL; ++l) {
                const int row = l < IL ? l * NWV + wave : hrow, px = l < IL ? mpx : hpx;
                if ((l < IL && (l + 1) * NWV <= TR) || row < TR)
                    *reinterpret_cast<u32x2*>(xs + (row * TC + px) * CK) =
                        u32x2{pk_bf16(fi[l][0], fi[l][1]), pk_bf16(fi[l][2], 0.f)};
            }
        } else {
#pragma unroll
            for (int l = 0; l < T::NL; ++l) {
                const int row = l * T::RPL + wrow;
                if ((l + 1) * T::RPL <= TR || row < TR) *reinterpret_cast<uint4*>(xs + (row * TC + mpx) * CK + msub * 8) = st[l];
            }
            if (hin) *reinterpret_cast<uint4*>(xs + (hrow * TC + hpx) * CK + msub * 8) = st[T::NL];
        }
        if constexpr (!RES)
#pragma unroll
            for (int l = 0; l < T::NWL; ++l) {
                const int f = l * NWV + wave;
                if ((l + 1) * NWV <= NKB * CB || f < NKB * CB) *reinterpret_cast<uint4*>(ws + f * 512 + lane * 8) = sw[l];
            }
    };

    union { uint4 u; bf16x8 v; } wr[RES ? NKB * CB : 1];
    if constexpr (RES) {
#pragma unroll
        for (int f = 0; f < NKB * CB; ++f) wr[f].u = wblock(0, f, lane * 16);
    }
    auto weight = [&](int kb, int c) -> bf16x8 {
        if constexpr (RES) return wr[kb * CB + c].v;
        else return *reinterpret_cast<const bf16x8*>(ws + ((kb * CB + c) * 64 + lane) * 8);
    };
    f4 bias[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) bias[c][e] = EPI <= E_OUT ? A.bias[(cb0 + c) * 16 + 4 * g + e] : 0.f;
    float wo[16], bo = 0.f;
    if constexpr (EPI == E_OUT) {
#pragma unroll
        for (int c = 0; c < 16; ++c) wo[c] = bf2f(A.wo[c]);
        bo = A.bo[0];
    }
    if constexpr (IN) {   // channels 3 to 15 of the input stay 0
        for (int q = tid; q < TR * TC * 2; q += T::NTW) *reinterpret_cast<uint4*>(xs + q * 8) = uint4{0u, 0u, 0u, 0u};
        __syncthreads();
    }

    // this lane's operand in the tile; CK = 16: the offset of the lane's tap of each block
    const bf16_t* bp = xs + (wy * TC + wx + jl) * CK + (CK == 32 ? 8 * g : 8 * (g & 1));
    int toff[NKB];
    if constexpr (CK == 16)
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
            const int t0 = 2 * kb, t1 = kb == 4 ? 8 : 2 * kb + 1;
            toff[kb] = ((g >> 1) ? (t1 / 3) * TC + t1 % 3 : (t0 / 3) * TC + t0 % 3) * CK;
        }

    f4 acc[RPW][PG][CB];
    fetch(tx, ty, tn, 0, true);
    if (!RES) wfetch(0, true);
    for (int i = 0; i < nmine; ++i) {
        const int x0 = tx * 64, y0 = ty * T::ROWS, n = tn;
#pragma unroll
        for (int r = 0; r < RPW; ++r)
#pragma unroll
            for (int p = 0; p < PG; ++p)
#pragma unroll
                for (int c = 0; c < CB; ++c) acc[r][p][c] = f4{0.f, 0.f, 0.f, 0.f};
        for (int chunk = 0; chunk < nchunk; ++chunk) {
            __syncthreads();   // every wave is done reading the previous step's LDS
            put();
            __syncthreads();
            // the next step's loads land while this one computes
            const bool last = chunk + 1 == nchunk, any = !last || i + 1 < nmine;
            if (last) {
                tx += gx;
                if (tx >= ntx) tx -= ntx, ++ty;
                ty += gy;
                if (ty >= nty) ty -= nty, ++tn;
                tn += gn;
            }
            const int next = last ? 0 : chunk + 1;
            fetch(tx, ty, tn, next, any);
            if (!RES) wfetch(next, any);
            __builtin_amdgcn_sched_barrier(0);   // issued here, not where registers are free
            if constexpr (CK == 16) {
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb) {
                    bf16x8 a[CB];
#pragma unroll
                    for (int c = 0; c < CB; ++c) a[c] = weight(kb, c);
                    const bf16_t* q = bp + toff[kb];
#pragma unroll
                    for (int r = 0; r < RPW; ++r)
#pragma unroll
                        for (int p = 0; p < PG; ++p) {
                            const bf16x8 b = *reinterpret_cast<const bf16x8*>(q + (r * TC + p * 16) * CK);
#pragma unroll
                            for (int c = 0; c < CB; ++c)
                                acc[r][p][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[c], b, acc[r][p][c], 0, 0, 0);
                        }
                }
            } else {
                // tile row t of the wave's RPW + 2 serves tap row t of its first
                // output row and t - 1 of its second: every sum runs over the taps in order
                bf16x8 a[2][3][CB];
#pragma unroll
                for (int t = 0; t < RPW + 2; ++t)
#pragma unroll
                    for (int dx = 0; dx < 3; ++dx) {
#pragma unroll
                        for (int c = 0; c < CB; ++c) {
                            if (t) a[1][dx][c] = a[0][dx][c];
                            if (t < 3) a[0][dx][c] = weight(t * 3 + dx, c);
                        }
#pragma unroll
                        for (int p = 0; p < PG; ++p) {
                            const bf16x8 b = *reinterpret_cast<const bf16x8*>(bp + (t * TC + p * 16 + dx) * CK);
#pragma unroll
                            for (int r = 0; r < RPW; ++r)
                                if (t - r >= 0 && t - r < 3)
#pragma unroll
                                    for (int c = 0; c < CB; ++c)
                                        acc[r][p][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[r][dx][c], b, acc[r][p][c], 0, 0, 0);
                        }
                    }
            }
        }
        // ---- the tile's outputs
        uint32_t po[PG];   // byte offsets of the lane's 8 channels of a pixel
#pragma unroll
        for (int p = 0; p < PG; ++p) {
            const int px = wx + (CB == 1 ? 2 * p + (g & 1) : p) * 16 + jl;
            po[p] = x0 + px < W ? 2 * (px * A.sy + (CB == 1 ? 0 : 16 * (g & 1)) + 8 * (g >> 1)) : OOB;
        }
        const int64_t img = (int64_t)n * H * W;
        const __amdgpu_buffer_rsrc_t ry = rsrc(A.Y + img * A.sy), rm = rsrc(EPI == E_MASK ? A.act + img * A.sy : nullptr);
        auto cbase = [&](int c, int yo) -> int {   // byte offset of row yo's first pixel, channel block c
            const int co = (cb0 + c) * 16;
            return 2 * (int)((yo * W + x0) * A.sy + co + (co >= A.ysplit ? A.yhs - A.ysplit : 0));
        };
        u32x2 on[RPW][PG][CB], out[RPW][PG][CB];
        if constexpr (EPI == E_MASK)
#pragma unroll
            for (int r = 0; r < RPW; ++r) {
                const int yo = y0 + wy + r;
#pragma unroll
                for (int p = 0; p < PG; p += CB == 1 ? 2 : 1)
#pragma unroll
                    for (int c = 0; c < CB; c += 2)
                        split_blocks(__builtin_amdgcn_raw_buffer_load_b128(
                                         rm, (int)(yo < H ? po[CB == 1 ? p >> 1 : p] : OOB), cbase(c, yo), 0),
                                     on[r][p][c], CB == 1 ? on[r][p + 1][c] : on[r][p][c + 1]);
            }
#pragma unroll
        for (int r = 0; r < RPW; ++r) {
            const int yo = y0 + wy + r;
#pragma unroll
            for (int p = 0; p < PG; ++p)
#pragma unroll
                for (int c = 0; c < CB; ++c) {
                    f4 v = acc[r][p][c];
                    if constexpr (EPI <= E_OUT)
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e] + bias[c][e], 0.f);
                    if constexpr (EPI == E_MASK) {
                        const u32x2 m = on[r][p][c];
                        v[0] = bf_lo(m.x) > 0.f ? v[0] : 0.f;
                        v[1] = bf_hi(m.x) > 0.f ? v[1] : 0.f;
                        v[2] = bf_lo(m.y) > 0.f ? v[2] : 0.f;
                        v[3] = bf_hi(m.y) > 0.f ? v[3] : 0.f;
                    }
                    out[r][p][c] = u32x2{pk_bf16(v[0], v[1]), pk_bf16(v[2], v[3])};
                }
            // 16 bytes a lane, of two channel blocks or (CB = 1) of two pixel groups.
            // No branches: the count of stores after the next step's loads is fixed
            const bool in = yo < H, yes = in && (EPI != E_OUT || A.Y);
            if constexpr (CB == 1) {
#pragma unroll
                for (int p = 0; p < PG; p += 2)
                    store16(merge_blocks(out[r][p][0], out[r][p + 1][0]), ry, (yes ? po[p >> 1] : OOB) + cbase(0, yo));
            } else {
#pragma unroll
                for (int p = 0; p < PG; ++p)
#pragma unroll
                    for (int c = 0; c < CB; c += 2) {
                        const int hop = A.ysplit == (cb0 + c + 1) * 16 ? 2 * (int)(A.yhs - A.ysplit) : 0;
                        const uint32_t vo = po[p] + (g & 1 ? hop : 0);
                        store16(merge_blocks(out[r][p][c], out[r][p][c + 1]), ry, (yes ? vo : OOB) + cbase(c, yo));
                    }
            }
            if constexpr (EPI == E_OUT) {
                // transpose over the four 16-lane rows: lane 16 g + j gets the 16
                // channels of pixel j of group g
                uint32_t ch[4][2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    auto v = [&](int p) { return h ? out[r][p][0].y : out[r][p][0].x; };
                    const auto s0 = __builtin_amdgcn_permlane32_swap(v(0), v(2), false, false);
                    const auto s1 = __builtin_amdgcn_permlane32_swap(v(1), v(3), false, false);
                    const auto t0 = __builtin_amdgcn_permlane16_swap(s0[0], s1[0], false, false);
                    const auto t1 = __builtin_amdgcn_permlane16_swap(s0[1], s1[1], false, false);
                    ch[0][h] = t0[0]; ch[1][h] = t0[1]; ch[2][h] = t1[0]; ch[3][h] = t1[1];
                }
                float s = bo;
#pragma unroll
                for (int c = 0; c < 16; ++c) {
                    const uint32_t w2 = ch[c >> 2][(c >> 1) & 1];
                    s += wo[c] * (c & 1 ? bf_hi(w2) : bf_lo(w2));
                }
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(s), rsrc(A.o + img),
                                                      (int)(in && x0 + lane < W ? 4 * lane : OOB), 4 * (yo * W + x0), 0);
            }
        }
        if constexpr (EPI == E_POOL) {
            // a lane pair holds two columns of pixel groups p and p + 1: the even lane
            // averages its pair's block of group p, the odd lane that of p + 1
            const int yo = y0 + wy;
            {
                const bool odd = lane & 1;
                const __amdgpu_buffer_rsrc_t rp = rsrc(A.pool + (img >> 2) * A.sy);
#pragma unroll
                for (int p = 0; p < PG; p += 2) {
                    const int px = wx + (p + (odd ? 1 : 0)) * 16 + jl;
                    const uint32_t vo = yo < H && x0 + px < W ? 2 * ((px >> 1) * A.sy + 4 * g) : OOB;
#pragma unroll
                    for (int c = 0; c < CB; ++c) {
                        uint32_t v[4][2];   // rows x columns, packed channels
#pragma unroll
                        for (int r = 0; r < 2; ++r)
#pragma unroll
                            for (int h = 0; h < 2; ++h) {
                                const uint32_t u0 = h ? out[r][p][c].y : out[r][p][c].x;
                                const uint32_t u1 = h ? out[r][p + 1][c].y : out[r][p + 1][c].x;
                                const uint32_t mine = odd ? u1 : u0, theirs = lane_pair(odd ? u0 : u1);
                                v[2 * r][h] = odd ? theirs : mine;
                                v[2 * r + 1][h] = odd ? mine : theirs;
                            }
                        float m[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            auto f = [&](int k) { return e & 1 ? bf_hi(v[k][e >> 1]) : bf_lo(v[k][e >> 1]); };
                            m[e] = 0.25f * (f(0) + f(1) + f(2) + f(3));
                        }
                        __builtin_amdgcn_raw_buffer_store_b64(
                            u32x2{pk_bf16(m[0], m[1]), pk_bf16(m[2], m[3])}, rp, (int)vo,
                            2 * (((yo >> 1) * (W >> 1) + (x0 >> 1)) * A.sy + (cb0 + c) * 16), 0);
                    }
                }
            }
        }
    }
}

// ---- weight gradients --------------------------------------------------------
// A weight gradient is a GEMM over pixels: D[co][ci] = sum_p GY[p][co] X[p'][ci]
// per tap, p' the tap's input pixel.  Both operands are wanted pixel-major (a
// lane holds eight pixels of one channel) while the tensors are channel-major,
// so tiles are staged in LDS as they are and read by the transposing loads of
// gfx950: ds_read_tr16_b64 gives lane l = 16 g + i of a wave column i (a
// channel) of the four rows (pixels) whose 32 bytes its group's lanes address,
// lane i at row i / 4, columns 4 (i % 4).  A tap is then an offset in pixels.
typedef __attribute__((address_space(3))) s4 lds_s4;

// Eight pixels of channel l % 16 for lane l: pixels p, .., p + 3 at `lo` and at
// `hi`, each lane passing the address of its pixel and channel quarter.
__device__ __forceinline__ bf16x8 tr_operand(const bf16_t* lo, const bf16_t* hi) {
    union { s4 h[2]; bf16x8 v; } u;
    u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(lo));
    u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(hi));
    return u.v;
}
__device__ __forceinline__ bf16x8 bf_ones() {
    union { s4 h[2]; bf16x8 v; } u;
    u.h[0] = u.h[1] = s4{0x3F80, 0x3F80, 0x3F80, 0x3F80};
    return u.v;
}

// Staging of an NHWC tile (C channels of ROWS rows of 64 CW pixels, with HALO one
// more row and column on each side) by a workgroup: a thread keeps its column
// and channels, a load is 16 bytes, its row a scalar; the HALO's last two columns
// are one more load.  Loads off the image, and all of them without `any`, give 0:
// no branches, whose joins would wait for the loads.
template <int C, int ROWS, int CW, bool HALO>
struct Stage {
    static constexpr int SUB = C / 8, RPL = NT / (64 * SUB), TR = ROWS + (HALO ? 2 : 0);
    static constexpr int PW = 64 * CW + (HALO ? 2 : 0), NL = (TR * CW + RPL - 1) / RPL;
    static_assert(RPL >= 1 && (!HALO || (CW == 1 && TR * 2 * SUB <= NT)), "tile staging");
    u32x4 v[NL + (HALO ? 1 : 0)];
    uint32_t moff, hoff;
    int wrow, mpx, msub, hrow, hpx;

    // s: pixel stride, W: row pitch (pixels), add: bytes from the base to this thread's channels
    __device__ __forceinline__ void init(int s, int W, uint32_t add) {
        const int tid = threadIdx.x;
        wrow = __builtin_amdgcn_readfirstlane(tid >> 6) / SUB;
        mpx = (tid % (64 * SUB)) / SUB;
        msub = tid % SUB;
        hrow = tid / (2 * SUB);
        hpx = 64 + (tid % (2 * SUB)) / SUB;
        moff = 2 * mpx * s + add;
        hoff = 2 * (hrow * W + hpx) * s + add;
    }
    // tile at (x0, y0) of the H x W image at `img`, its base at the first of the
    // thread's channel group
    __device__ __forceinline__ void load(const bf16_t* img, int s, int H, int W, int x0, int y0, bool any) {
        constexpr int O = HALO ? 1 : 0;
        const __amdgpu_buffer_rsrc_t r = rsrc(img - (int64_t)O * (1 + W) * s);   // offsets stay positive
        uint32_t mo[CW];
#pragma unroll
        for (int k = 0; k < CW; ++k) mo[k] = (uint32_t)(x0 - O + 64 * k + mpx) < (uint32_t)W ? moff : OOB;
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const int h = l * RPL + wrow, row = h / CW, half = h % CW, yy = y0 - O + row;
            const bool in = any & ((uint32_t)yy < (uint32_t)H) & (row < TR);
            v[l] = __builtin_amdgcn_raw_buffer_load_b128(r, (int)(in ? (half ? mo[CW - 1] : mo[0]) : OOB),
                                                         2 * ((yy + O) * W + x0 + 64 * half) * s, 0);
        }
        if constexpr (HALO) {
            const bool in = any & (hrow < TR) & ((uint32_t)(y0 - 1 + hrow) < (uint32_t)H) & (x0 - 1 + hpx < W);
            v[NL] = __builtin_amdgcn_raw_buffer_load_b128(r, (int)(in ? hoff : OOB), 2 * (y0 * W + x0) * s, 0);
        }
    }
    __device__ __forceinline__ void put(bf16_t* lds) const {
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const int h = l * RPL + wrow, row = h / CW, half = 64 * (h % CW);
            if ((l + 1) * RPL <= TR * CW || row < TR)
                *reinterpret_cast<u32x4*>(lds + (row * PW + half + mpx) * C + msub * 8) = v[l];
        }
        if constexpr (HALO)
            if (hrow < TR) *reinterpret_cast<u32x4*>(lds + (hrow * PW + hpx) * C + msub * 8) = v[NL];
    }
};

// Tiles b, b + step, ... of an image batch, as (x, y, image): scalar additions
struct TileWalk {
    int x, y, n, gx, gy, gn, ntx, nty;
    __device__ __forceinline__ TileWalk(int b, int step, int ntx_, int nty_) : ntx(ntx_), nty(nty_) {
        x = b % ntx; y = (b / ntx) % nty; n = b / (ntx * nty);
        gx = step % ntx; gy = (step / ntx) % nty; gn = step / (ntx * nty);
    }
    __device__ __forceinline__ void next() {
        x += gx;
        if (x >= ntx) x -= ntx, ++y;
        y += gy;
        if (y >= nty) y -= nty, ++n;
        n += gn;
    }
};

// Sum the four waves' accumulators of a workgroup in a fixed order and write
// them as part[tap][co][ci] of this chunk (TAPS x CO x CI of the layer's TAPS x
// Cout x Cin, at co0, ci0), the bias sums (column 0 of bacc) after them.
template <int TAPS, int CB, int IB>
__device__ __forceinline__ void wgrad_out(const f4 (&acc)[TAPS][CB][IB], const f4 (&bacc)[CB], float* sm, int co0,
                                          int ci0, int Cout, int Cin, float* __restrict__ part,
                                          float* __restrict__ bpart) {
    constexpr int CO = 16 * CB, CI = 16 * IB;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int jl = lane & 15, g = lane >> 4;
    float* sb = sm + TAPS * CO * CI;
    for (int w = 0; w < 4; ++w) {
        __syncthreads();
        if (wave != w) continue;
#pragma unroll
        for (int t = 0; t < TAPS; ++t)
#pragma unroll
            for (int c = 0; c < CB; ++c)
#pragma unroll
                for (int b = 0; b < IB; ++b)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        float* q = sm + (t * CO + 16 * c + 4 * g + e) * CI + 16 * b + jl;
                        *q = w ? *q + acc[t][c][b][e] : acc[t][c][b][e];
                    }
        if (jl == 0)
#pragma unroll
            for (int c = 0; c < CB; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float* q = sb + 16 * c + 4 * g + e;
                    *q = w ? *q + bacc[c][e] : bacc[c][e];
                }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < TAPS * CO * CI; i += NT) {
        const int ci = i % CI, co = (i / CI) % CO, t = i / (CI * CO);
        part[((int64_t)t * Cout + co0 + co) * Cin + ci0 + ci] = sm[i];
    }
    if (ci0 == 0 && threadIdx.x < CO) bpart[co0 + threadIdx.x] = sb[threadIdx.x];
}

// Weight gradient of a 3x3 convolution, with the bias gradient sum_p GY[p][co]
// (a product with ones).  Workgroup (chunk, channel tile): four waves, 16 CB
// output x 16 IB input channels, all nine taps, over the chunk's tiles of
// ROWS x 64 pixels (chunk, chunk + gridDim.x, ...); a tile's GY and its X with
// a 1-pixel halo are staged in LDS while the next tile's loads are in flight,
// and wave w takes rows w, w + 4, ...  Pixels off the image are 0.
//
// One wave per 16 x 16 channels fetching every operand element by itself (two
// bytes a load) and a thread per output adding up to 1664 chunks took 183 and 143
// us a layer on average on 16 images of 208 x 408.  Now 22 us at 16 x 16 channels
// (87 MB once, 107 moved by counters, 4.9 TB/s), 27 us at 32 x 32 and above (35 with an index, a branch and
// a wait per staged piece), 6 us for the sum; the whole training gradient went
// from 6.58 to 1.55 ms, and with the convolutions' new kernel to 1.24 ms.
template <int CB, int IB, int ROWS>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2))) void k_conv3_wgrad(
    const bf16_t* __restrict__ GY, int sg, int Cout, const bf16_t* __restrict__ X, int sx, int64_t xhs, int xsplit,
    int Cin, int H, int W, int N, float* __restrict__ part, float* __restrict__ bpart) {
    constexpr int CO = 16 * CB, CI = 16 * IB, TW = 64, XW = TW + 2;
    constexpr int SM_TILE = (ROWS * TW * CO + (ROWS + 2) * XW * CI) * 2, SM_OUT = (9 * CO * CI + CO) * 4;
    __shared__ __align__(16) char smem[SM_TILE > SM_OUT ? SM_TILE : SM_OUT];
    bf16_t* gs = reinterpret_cast<bf16_t*>(smem);
    bf16_t* xs = gs + ROWS * TW * CO;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nci = Cin / CI;
    const int co0 = (int)(blockIdx.y / nci) * CO, ci0 = (int)(blockIdx.y % nci) * CI;
    const int ntx = (W + TW - 1) / TW, nty = (H + ROWS - 1) / ROWS, ntiles = ntx * nty * N;
    Stage<CO, ROWS, 1, false> sg_;
    Stage<CI, ROWS, 1, true> sx_;
    sg_.init(sg, W, 16u * (threadIdx.x % (CO / 8)));
    {   // a channel tile may span the halves of a concatenation
        const int xch = ci0 + (int)(threadIdx.x % (CI / 8)) * 8;
        const int64_t hop = xch >= xsplit && ci0 < xsplit ? xhs - xsplit : 0;
        sx_.init(sx, W, 16u * (threadIdx.x % (CI / 8)) + 2u * (uint32_t)hop);
    }
    const bf16_t* Xc = X + ci0 + (ci0 >= xsplit ? xhs - xsplit : 0);
    TileWalk tw(blockIdx.x, gridDim.x, ntx, nty);
    auto fetch = [&](bool any) {
        sg_.load(GY + co0 + (int64_t)tw.n * H * W * sg, sg, H, W, tw.x * TW, tw.y * ROWS, any);
        sx_.load(Xc + (int64_t)tw.n * H * W * sx, sx, H, W, tw.x * TW, tw.y * ROWS, any);
    };
    f4 acc[9][CB][IB], bacc[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        bacc[c] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int b = 0; b < IB; ++b) acc[t][c][b] = f4{0.f, 0.f, 0.f, 0.f};
    }
    // this lane's pixel and channel quarter in a group of 16 pixels
    const int pl = 4 * (lane >> 4) + ((lane & 15) >> 2), cq = 4 * (lane & 3);
    fetch((int)blockIdx.x < ntiles);
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
        __syncthreads();   // every wave is done with the previous tile
        sg_.put(gs);
        sx_.put(xs);
        __syncthreads();
        tw.next();
        fetch(t + (int)gridDim.x < ntiles);
        __builtin_amdgcn_sched_barrier(0);   // issued here, not where registers are free
#pragma unroll
        for (int r0 = 0; r0 < ROWS; r0 += 4) {
            const int row = r0 + wave;
#pragma unroll
            for (int k0 = 0; k0 < TW; k0 += 32) {
                bf16x8 a[CB];
                const bf16_t* gp = gs + (row * TW + k0 + pl) * CO + cq;
#pragma unroll
                for (int c = 0; c < CB; ++c) {
                    a[c] = tr_operand(gp + 16 * c, gp + 16 * CO + 16 * c);
                    bacc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[c], bf_ones(), bacc[c], 0, 0, 0);
                }
#pragma unroll
                for (int tap = 0; tap < 9; ++tap) {
                    const bf16_t* xp = xs + ((row + tap / 3) * XW + k0 + pl + tap % 3) * CI + cq;
#pragma unroll
                    for (int b = 0; b < IB; ++b) {
                        const bf16x8 bv = tr_operand(xp + 16 * b, xp + 16 * CI + 16 * b);
#pragma unroll
                        for (int c = 0; c < CB; ++c)
                            acc[tap][c][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[c], bv, acc[tap][c][b], 0, 0, 0);
                    }
                }
            }
        }
    }
    const int64_t per = (int64_t)9 * Cout * Cin;
    wgrad_out<9, CB, IB>(acc, bacc, reinterpret_cast<float*>(smem), co0, ci0, Cout, Cin, part + blockIdx.x * per,
                         bpart + (int64_t)blockIdx.x * Cout);
}

// Sum the chunk partials [chunk][tap][co][ci] (and [chunk][nbias] of the bias) of
// a layer into its flat gradient: weights [co][ci][taps] (3x3 convolutions, ci <
// cin_real) or [ci][co][taps] (T: transposed ones), then the bias.  A workgroup
// takes 64 outputs, 16 threads each over every 16th chunk, in float64.
template <bool T>
__global__ __launch_bounds__(1024) void k_wgrad_reduce(const float* __restrict__ part, const float* __restrict__ bpart,
                                                       int nchunks, int taps, int Cout, int Cin, int cin_real,
                                                       int nbias, float* __restrict__ gflat) {
    __shared__ double sm[16][64];
    const int64_t per = (int64_t)taps * Cout * Cin;
    const int64_t i = blockIdx.x * (int64_t)64 + (threadIdx.x & 63);
    const int slice = threadIdx.x >> 6;
    double s = 0.0;
    if (i < per + nbias) {
        const float* p = i < per ? part + i : bpart + (i - per);
        const int64_t stride = i < per ? per : nbias;
#pragma unroll 4
        for (int c = slice; c < nchunks; c += 16) s += p[c * stride];
    }
    sm[slice][threadIdx.x & 63] = s;
    __syncthreads();
    if (slice || i >= per + nbias) return;
    s = 0.0;
#pragma unroll
    for (int k = 0; k < 16; ++k) s += sm[k][threadIdx.x];
    if (i >= per) {
        gflat[(int64_t)Cout * cin_real * taps + (i - per)] = (float)s;
        return;
    }
    const int ci = (int)(i % Cin), co = (int)((i / Cin) % Cout), tap = (int)(i / ((int64_t)Cin * Cout));
    if (T) gflat[((int64_t)ci * Cout + co) * taps + tap] = (float)s;
    else if (ci < cin_real) gflat[((int64_t)co * cin_real + ci) * taps + tap] = (float)s;
}

// Gradient into an encoder output: g[n][y][x][c] = bf16(gp[n][y/2][x/2][c] / 4
// + gskip[n][y][x][c]), then the ReLU mask of that output.  One thread per 8
// channels of a pixel (16-byte loads and store: 18 us a level on average on 16
// images of 208 x 408, two bytes at a time 51).
__global__ void k_pool_back(const bf16_t* __restrict__ GP, const bf16_t* GS, const bf16_t* __restrict__ Yact,
                            bf16_t* G, int C, int N, int H, int W) {   // GS may be G
    const int C8 = C / 8;
    const int64_t total = (int64_t)N * H * W * C8;
    for (int64_t i = blockIdx.x * (int64_t)NT + threadIdx.x; i < total; i += (int64_t)gridDim.x * NT) {
        const int c = (int)(i % C8) * 8;
        const int64_t pix = i / C8;
        const int x = (int)(pix % W), y = (int)((pix / W) % H), n = (int)(pix / ((int64_t)W * H));
        const int64_t pp = ((int64_t)n * (H / 2) + y / 2) * (W / 2) + x / 2;
        bf8u gp, gsk, ya, o;
        gp.u = *reinterpret_cast<const uint4*>(GP + pp * C + c);
        gsk.u = *reinterpret_cast<const uint4*>(GS + pix * C + c);
        ya.u = *reinterpret_cast<const uint4*>(Yact + pix * C + c);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float v = 0.25f * bf2f(gp.h[e]) + bf2f(gsk.h[e]);
            o.h[e] = bf2f(ya.h[e]) > 0.f ? f2bf(v) : (bf16_t)0;
        }
        *reinterpret_cast<uint4*>(G + pix * C + c) = o.u;
    }
}

// Transposed 2x2 convolution, stride 2, as a GEMM per input pixel on
// v_mfma_f32_16x16x32_bf16: D[(a d) Cout + co][pixel] = sum_ci W[ci][co][a][d]
// X[pixel][ci], stored with its bias at output pixel (2i + a, 2j + d).  A is
// packed by k_pack_frag_t in the instruction's operand order ([ci / 32][row
// block][lane][8]).  Workgroup: 4 waves, one input row each, 64 input pixels
// x 16 CB rows of D; every operand load of the launch (NKC = Cin / 32 blocks)
// is issued before the first MFMA.
template <int CB, int NKC>
__global__ __launch_bounds__(NT) void k_convT_mfma(const bf16_t* __restrict__ X, int sx,
                                                   const bf16_t* __restrict__ Af, const float* __restrict__ bias,
                                                   bf16_t* __restrict__ Y, int sy, int Cout, int Hi, int Wi) {
    static_assert(CB % 2 == 0, "blocks of 16 outputs are stored in pairs");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int jl = lane & 15, g = lane >> 4;
    const int M = 4 * Cout, nmb = M / 16;
    const int ncog = M / (16 * CB);
    const int n = blockIdx.z / ncog;
    const int mb0 = (blockIdx.z % ncog) * CB;
    const int y = blockIdx.y * 4 + wave;
    if (y >= Hi) return;
    const int x0 = blockIdx.x * 64;
    const __amdgpu_buffer_rsrc_t rx = rsrc(X + (((int64_t)n * Hi + y) * Wi + x0) * sx), ra = rsrc(Af);
    bf16x8 b[NKC][4], a[NKC][CB];
    auto load = [](__amdgpu_buffer_rsrc_t r, uint32_t v, int o) {
        union { u32x4 u; bf16x8 h; } q;
        q.u = __builtin_amdgcn_raw_buffer_load_b128(r, (int)v, o, 0);
        return q.h;
    };
    uint32_t po[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const bool in = x0 + p * 16 + jl < Wi;
        const uint32_t vo = in ? 2 * ((p * 16 + jl) * sx + 8 * g) : OOB;
#pragma unroll
        for (int kc = 0; kc < NKC; ++kc) b[kc][p] = load(rx, vo, kc * 64);
        // 8 outputs of a pair of blocks: two neighbouring outputs pixels are 2 Cout
        // consecutive channels
        po[p] = in ? 2 * (2 * (p * 16 + jl) * sy + 16 * (g & 1) + 8 * (g >> 1)) : OOB;
    }
    f4 bs[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) {
#pragma unroll
        for (int kc = 0; kc < NKC; ++kc) a[kc][c] = load(ra, lane * 16, (kc * nmb + mb0 + c) * 1024);
#pragma unroll
        for (int e = 0; e < 4; ++e) bs[c][e] = bias[((mb0 + c) * 16) % Cout + 4 * g + e];
    }
    f4 acc[4][CB];
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            acc[p][c] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kc = 0; kc < NKC; ++kc)
                acc[p][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[kc][c], b[kc][p], acc[p][c], 0, 0, 0);
        }
    const int Wo = 2 * Wi;
#pragma unroll
    for (int c = 0; c < CB; c += 2) {
        const int m = (mb0 + c) * 16, ra2 = m / (2 * Cout);   // output row of the pair's four, and the channel in it
        const __amdgpu_buffer_rsrc_t ry = rsrc(Y + (((int64_t)n * 2 * Hi + 2 * y + ra2) * Wo + 2 * x0) * sy);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            u32x2 o[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                f4 v = acc[p][c + h];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] += bs[c + h][e];
                o[h] = u32x2{pk_bf16(v[0], v[1]), pk_bf16(v[2], v[3])};
            }
            store16(merge_blocks(o[0], o[1]), ry, po[p] + 2 * (m - ra2 * 2 * Cout));
        }
    }
}

// Data gradient of the transposed convolution: D[ci][pixel] = sum over
// (a d, co) of WT[ci][(a d) Cout + co] GY[(2i + a, 2j + d)][co]; WT is
// [Cin][4 Cout] bf16.  Outputs where the activation `act` (laid out as GX) is
// not positive are 0.  Same workgroup shape as k_convT_mfma.
template <int CB>
__global__ __launch_bounds__(NT) void k_convT_dgrad_mfma(const bf16_t* __restrict__ GY, int sg, int Cout,
                                                         const bf16_t* __restrict__ WT, bf16_t* __restrict__ GX,
                                                         int sx, int Cin, int Hi, int Wi,
                                                         const bf16_t* __restrict__ act) {
    static_assert(CB % 2 == 0, "blocks of 16 outputs are stored in pairs");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ncog = Cin / (16 * CB);
    const int n = blockIdx.z / ncog;
    const int c0 = (blockIdx.z % ncog) * 16 * CB;
    const int y = blockIdx.y * 4 + wave;
    if (y >= Hi) return;
    const int x0 = blockIdx.x * 64;
    const int jl = lane & 15, g = lane >> 4;
    const int K = 4 * Cout, Wo = 2 * Wi;
    auto load8 = [](__amdgpu_buffer_rsrc_t r, uint32_t v, int o) {
        union { u32x2 u; s4 h; } q;
        q.u = __builtin_amdgcn_raw_buffer_load_b64(r, (int)v, o, 0);
        return q.h;
    };
    const __amdgpu_buffer_rsrc_t rg = rsrc(GY + (((int64_t)n * 2 * Hi + 2 * y) * Wo + 2 * x0) * sg), rw = rsrc(WT);
    const int64_t row = (((int64_t)n * Hi + y) * Wi + x0) * sx + c0;
    const __amdgpu_buffer_rsrc_t rx = rsrc(GX + row), rm = rsrc(act + row);
    uint32_t bo[4], po[4], wo[CB];   // byte offsets: gradient, outputs (as stored), weights
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const int px = p * 16 + jl;
        bo[p] = x0 + px < Wi ? 2 * (2 * px * sg + 4 * g) : OOB;
        po[p] = x0 + px < Wi ? 2 * (px * sx + 16 * (g & 1) + 8 * (g >> 1)) : OOB;
    }
#pragma unroll
    for (int c = 0; c < CB; ++c) wo[c] = 2 * ((c0 + c * 16 + jl) * K + 4 * g);
    f4 acc[4][CB];
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int c = 0; c < CB; ++c) acc[p][c] = f4{0.f, 0.f, 0.f, 0.f};
    // four blocks of 16 contraction indices at a time (K is a multiple of 64):
    // their loads fly together
    for (int k0 = 0; k0 < K; k0 += 64) {
        s4 b[4][4], av[4][CB];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = k0 + 16 * u, ad = k / Cout, co = k - ad * Cout;
#pragma unroll
            for (int p = 0; p < 4; ++p) b[u][p] = load8(rg, bo[p], 2 * (((ad >> 1) * Wo + (ad & 1)) * sg + co));
#pragma unroll
            for (int c = 0; c < CB; ++c) av[u][c] = load8(rw, wo[c], 2 * k);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int c = 0; c < CB; ++c)
#pragma unroll
                for (int p = 0; p < 4; ++p)
                    acc[p][c] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(av[u][c], b[u][p], acc[p][c], 0, 0, 0);
    }
    u32x4 on[4][CB / 2];
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int c = 0; c < CB; c += 2) on[p][c / 2] = __builtin_amdgcn_raw_buffer_load_b128(rm, (int)po[p], 32 * c, 0);
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int c = 0; c < CB; c += 2) {
            u32x2 m[2], o[2];
            split_blocks(on[p][c / 2], m[0], m[1]);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const f4 v = acc[p][c + h];
                o[h] = u32x2{pk_bf16(bf_lo(m[h].x) > 0.f ? v[0] : 0.f, bf_hi(m[h].x) > 0.f ? v[1] : 0.f),
                             pk_bf16(bf_lo(m[h].y) > 0.f ? v[2] : 0.f, bf_hi(m[h].y) > 0.f ? v[3] : 0.f)};
            }
            store16(merge_blocks(o[0], o[1]), rx, po[p] + 32 * c);
        }
}

// Weight gradient of the transposed convolution: part[chunk][ad][co][ci] = sum
// over the chunk's input pixels of GY[(2i + a, 2j + d)][co] X[(i, j)][ci], and
// the bias partials sum GY.  As k_conv3_wgrad, on tiles of 2 x 64 input pixels
// (4 x 128 of GY, whose pixels a tap reads at a stride of two); wave w takes
// row w / 2, columns 32 (w % 2) on.
template <int CB, int IB>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2))) void k_convT_wgrad(
    const bf16_t* __restrict__ X, int sx, int Cin, const bf16_t* __restrict__ GY, int sg, int Cout, int Hi, int Wi,
    int N, float* __restrict__ part, float* __restrict__ bpart) {
    constexpr int CO = 16 * CB, CI = 16 * IB, TW = 64, ROWS = 2;
    constexpr int SM_TILE = (4 * ROWS * TW * CO + ROWS * TW * CI) * 2, SM_OUT = (4 * CO * CI + CO) * 4;
    __shared__ __align__(16) char smem[SM_TILE > SM_OUT ? SM_TILE : SM_OUT];
    bf16_t* gs = reinterpret_cast<bf16_t*>(smem);
    bf16_t* xs = gs + 4 * ROWS * TW * CO;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nci = Cin / CI;
    const int co0 = (int)(blockIdx.y / nci) * CO, ci0 = (int)(blockIdx.y % nci) * CI;
    const int ntx = (Wi + TW - 1) / TW, nty = (Hi + ROWS - 1) / ROWS, ntiles = ntx * nty * N;
    const int Wo = 2 * Wi, Ho = 2 * Hi;
    Stage<CO, 2 * ROWS, 2, false> sg_;
    Stage<CI, ROWS, 1, false> sx_;
    sg_.init(sg, Wo, 16u * (threadIdx.x % (CO / 8)));
    sx_.init(sx, Wi, 16u * (threadIdx.x % (CI / 8)));
    TileWalk tw(blockIdx.x, gridDim.x, ntx, nty);
    auto fetch = [&](bool any) {
        sg_.load(GY + co0 + (int64_t)tw.n * Ho * Wo * sg, sg, Ho, Wo, 2 * tw.x * TW, 2 * tw.y * ROWS, any);
        sx_.load(X + ci0 + (int64_t)tw.n * Hi * Wi * sx, sx, Hi, Wi, tw.x * TW, tw.y * ROWS, any);
    };
    f4 acc[4][CB][IB], bacc[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        bacc[c] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int b = 0; b < IB; ++b) acc[t][c][b] = f4{0.f, 0.f, 0.f, 0.f};
    }
    const int pl = 4 * (lane >> 4) + ((lane & 15) >> 2), cq = 4 * (lane & 3);
    const int row = wave >> 1, k0 = 32 * (wave & 1);
    fetch((int)blockIdx.x < ntiles);
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
        __syncthreads();   // every wave is done with the previous tile
        sg_.put(gs);
        sx_.put(xs);
        __syncthreads();
        tw.next();
        fetch(t + (int)gridDim.x < ntiles);
        __builtin_amdgcn_sched_barrier(0);   // issued here, not where registers are free
        bf16x8 bv[IB];
        const bf16_t* xp = xs + (row * TW + k0 + pl) * CI + cq;
#pragma unroll
        for (int b = 0; b < IB; ++b) bv[b] = tr_operand(xp + 16 * b, xp + 16 * CI + 16 * b);
#pragma unroll
        for (int ad = 0; ad < 4; ++ad) {
            const bf16_t* gp = gs + ((2 * row + (ad >> 1)) * 2 * TW + 2 * (k0 + pl) + (ad & 1)) * CO + cq;
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                const bf16x8 a = tr_operand(gp + 16 * c, gp + 32 * CO + 16 * c);
                bacc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bf_ones(), bacc[c], 0, 0, 0);
#pragma unroll
                for (int b = 0; b < IB; ++b)
                    acc[ad][c][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bv[b], acc[ad][c][b], 0, 0, 0);
            }
        }
    }
    const int64_t per = (int64_t)4 * Cout * Cin;
    wgrad_out<4, CB, IB>(acc, bacc, reinterpret_cast<float*>(smem), co0, ci0, Cout, Cin, part + blockIdx.x * per,
                         bpart + (int64_t)blockIdx.x * Cout);
}

// Back through the output layer: g[p][c] = bf16(w[c] go[p]) masked by the
// ReLU of its input x; weight and bias partials per chunk: part[chunk][17].
__global__ void k_out_back(const float* __restrict__ go, const bf16_t* __restrict__ X, int sx,
                           const bf16_t* __restrict__ w, bf16_t* __restrict__ G, int sg, int64_t npix,
                           int64_t pix_per_chunk, float* __restrict__ part) {
    __shared__ float red[17][NT / 64];
    const int chunk = blockIdx.x;
    const int64_t p0 = chunk * pix_per_chunk, p1 = min(npix, p0 + pix_per_chunk);
    float acc[17];
#pragma unroll
    for (int c = 0; c < 17; ++c) acc[c] = 0.f;
    for (int64_t p = p0 + threadIdx.x; p < p1; p += NT) {
        const float g = go[p];
        bf8u xv[2], gv[2];
        xv[0].u = *reinterpret_cast<const uint4*>(X + p * sx);
        xv[1].u = *reinterpret_cast<const uint4*>(X + p * sx + 8);
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            const float xc = bf2f(xv[c >> 3].h[c & 7]);
            acc[c] += g * xc;
            gv[c >> 3].h[c & 7] = xc > 0.f ? f2bf(bf2f(w[c]) * g) : (bf16_t)0;
        }
        *reinterpret_cast<uint4*>(G + p * sg) = gv[0].u;
        *reinterpret_cast<uint4*>(G + p * sg + 8) = gv[1].u;
        acc[16] += g;
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int c = 0; c < 17; ++c) {
        float v = acc[c];
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if (lane == 0) red[c][wv] = v;
    }
    __syncthreads();
    if (threadIdx.x < 17) {
        float s = 0.f;
        for (int k = 0; k < NT / 64; ++k) s += red[threadIdx.x][k];
        part[(int64_t)chunk * 17 + threadIdx.x] = s;
    }
}

// Default per-sample loss weight sum_x a / (sum_x c)^2 (0 when sum_x c <= 0).
// One workgroup per sample.
__global__ __launch_bounds__(NT) void k_loss_weights(const float* __restrict__ a, const float* __restrict__ c,
                                                     int64_t npix, float* __restrict__ w) {
    __shared__ double red[2][NT / 64];
    const int s = blockIdx.x;
    double sa = 0.0, sc = 0.0;
    for (int64_t p = threadIdx.x; p < npix; p += NT) {
        sa += a[(int64_t)s * npix + p];
        sc += c[(int64_t)s * npix + p];
    }
    for (int k = 32; k > 0; k >>= 1) {
        sa += __shfl_xor(sa, k, 64);
        sc += __shfl_xor(sc, k, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = sa;
        red[1][threadIdx.x >> 6] = sc;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double ta = 0.0, tc = 0.0;
        for (int k = 0; k < NT / 64; ++k) { ta += red[0][k]; tc += red[1][k]; }
        w[s] = (tc > 0.0 && ta > 0.0) ? (float)(ta / (tc * tc)) : 0.f;
    }
}

// Scaling loss per sample s: L_s = w_s sum_x (a e^{2o} - 2 c e^{o}) and
// go = w_s (2 a e^{2o} - 2 c e^{o}) / nbatch, with w from `weight` or the
// default sum_x a / (sum_x c)^2 of the image.  LOSS_BLOCKS workgroups per sample
// (grid LOSS_BLOCKS x nbatch) leave float64 partials, summed in a fixed order:
// k_loss_sums those of a and c, k_scaling_loss the loss's, k_loss_finish adds
// them up.  (One workgroup per sample took 266 us for 16 images of 208 x 408.)
constexpr int LOSS_BLOCKS = 32;

__device__ __forceinline__ double nt_block_sum(double v, double* red) {   // valid in every thread
    for (int k = 32; k > 0; k >>= 1) v += __shfl_xor(v, k, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
    for (int k = 0; k < NT / 64; ++k) t += red[k];
    return t;
}

// part[s][b][2]: partial sums of a and c
__global__ __launch_bounds__(NT) void k_loss_sums(const float* __restrict__ a, const float* __restrict__ c,
                                                  int64_t npix, double* __restrict__ part) {
    __shared__ double red[NT / 64];
    const int s = blockIdx.y;
    double suma = 0.0, sumc = 0.0;
    for (int64_t p = blockIdx.x * (int64_t)NT + threadIdx.x; p < npix; p += (int64_t)LOSS_BLOCKS * NT) {
        suma += a[(int64_t)s * npix + p];
        sumc += c[(int64_t)s * npix + p];
    }
    suma = nt_block_sum(suma, red);
    sumc = nt_block_sum(sumc, red);
    if (threadIdx.x == 0) {
        part[((int64_t)s * LOSS_BLOCKS + blockIdx.x) * 2] = suma;
        part[((int64_t)s * LOSS_BLOCKS + blockIdx.x) * 2 + 1] = sumc;
    }
}

// sums: k_loss_sums' partials (weight null); lpart[s][b]: partial of the weighted loss
__global__ __launch_bounds__(NT) void k_scaling_loss(const float* __restrict__ o, const float* __restrict__ a,
                                                     const float* __restrict__ c, const float* __restrict__ weight,
                                                     const double* __restrict__ sums, int64_t npix, int nbatch,
                                                     float* __restrict__ go, double* __restrict__ lpart) {
    __shared__ double red[NT / 64];
    const int s = blockIdx.y;
    const float* os = o + (int64_t)s * npix;
    const float* as = a + (int64_t)s * npix;
    const float* cs = c + (int64_t)s * npix;
    double wt;
    if (weight) {
        wt = weight[s];
    } else {
        double suma = 0.0, sumc = 0.0;
        for (int b = 0; b < LOSS_BLOCKS; ++b) {
            suma += sums[((int64_t)s * LOSS_BLOCKS + b) * 2];
            sumc += sums[((int64_t)s * LOSS_BLOCKS + b) * 2 + 1];
        }
        wt = (sumc > 0.0 && suma > 0.0) ? (double)(float)(suma / (sumc * sumc)) : 0.0;
    }
    const float inv = (float)wt;
    double sl = 0.0;
    for (int64_t p = blockIdx.x * (int64_t)NT + threadIdx.x; p < npix; p += (int64_t)LOSS_BLOCKS * NT) {
        const float e = expf(os[p]);
        const float ae = as[p] * e, ce = cs[p];
        sl += (double)(ae * e - 2.f * ce * e);
        go[(int64_t)s * npix + p] = (2.f * ae * e - 2.f * ce * e) * inv / (float)nbatch;
    }
    sl = nt_block_sum(sl, red);
    if (threadIdx.x == 0) lpart[(int64_t)s * LOSS_BLOCKS + blockIdx.x] = sl * wt;
}

__global__ void k_loss_finish(const double* __restrict__ lpart, int nbatch, double* __restrict__ loss) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= nbatch) return;
    double t = 0.0;
    for (int b = 0; b < LOSS_BLOCKS; ++b) t += lpart[(int64_t)s * LOSS_BLOCKS + b];
    loss[s] = t;
}

// Squared gradient norm: partials per block, summed by k_norm_finish.
__global__ __launch_bounds__(NT) void k_sqnorm(const float* __restrict__ g, int64_t n, double* __restrict__ part) {
    __shared__ double red[NT / 64];
    double acc = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)NT + threadIdx.x; i < n; i += (int64_t)gridDim.x * NT)
        acc += (double)g[i] * (double)g[i];
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int k = 0; k < NT / 64; ++k) t += red[k];
        part[blockIdx.x] = t;
    }
}

// factor[0] = min(1, clip / ||g||) from the block partials (one thread).
__global__ void k_clip_factor(const double* __restrict__ part, int nb, float clip, float* __restrict__ factor) {
    if (threadIdx.x != 0) return;
    double t = 0.0;
    for (int k = 0; k < nb; ++k) t += part[k];
    const double nrm = sqrt(t);
    factor[0] = (clip > 0.f && nrm > clip) ? (float)(clip / nrm) : 1.f;
}

// Adam (Kingma & Ba 2015) on the float32 master parameters, the gradient
// scaled by factor[0] (gradient-norm clipping) when factor is given.
__global__ void k_adam(float* __restrict__ th, float* __restrict__ m, float* __restrict__ v,
                       const float* __restrict__ g, int64_t n, float lr, float b1, float b2, float eps,
                       float bc1, float bc2, const float* __restrict__ factor) {
    const float f = factor ? factor[0] : 1.f;
    for (int64_t i = blockIdx.x * (int64_t)NT + threadIdx.x; i < n; i += (int64_t)gridDim.x * NT) {
        const float gi = g[i] * f;
        const float mi = b1 * m[i] + (1.f - b1) * gi;
        const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        th[i] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
    }
}

// bf16 weights of a 3x3 layer in the operand order of k_conv3, from the
// master weights w[co][ci][3][3] (cin real input channels): forward (bwd = 0)
// A[tap][m = co][k = ci], the data gradient (bwd = 1) A[tap][m = ci][k = co]
// with the taps reversed.  Element (chunk, kb, cb, lane, e) is A at
// m = 16 cb + lane % 16 and the lane's tap and channel k of block kb
// (k_conv3's contraction order); zero beyond M, K, cin or the ninth tap.
__global__ void k_pack_frag(const float* __restrict__ w, int cout, int cin, int M, int K, int bwd,
                            bf16_t* __restrict__ af, int64_t n) {
    const int ck = frag_ck(K), nkb = frag_nkb(ck), ncb = (M + 15) / 16;
    for (int64_t i = blockIdx.x * (int64_t)NT + threadIdx.x; i < n; i += (int64_t)gridDim.x * NT) {
        const int e = (int)(i & 7), lane = (int)((i >> 3) & 63);
        const int64_t rest = i >> 9;
        const int cb = (int)(rest % ncb), kb = (int)((rest / ncb) % nkb), chunk = (int)(rest / ((int64_t)ncb * nkb));
        const int g = lane >> 4, m = cb * 16 + (lane & 15);
        const int tap = ck == 32 ? kb : 2 * kb + (g >> 1);
        const int k = chunk * ck + (ck == 32 ? 8 * g : 8 * (g & 1)) + e;
        float v = 0.f;
        if (tap < 9 && m < M && k < K) {
            const int co = bwd ? k : m, ci = bwd ? m : k;
            if (ci < cin) v = w[((int64_t)co * cin + ci) * 9 + (bwd ? 8 - tap : tap)];
        }
        af[i] = f2bf(v);
    }
}

int64_t convT_frag_elems(int Cin, int Cout) { return (int64_t)((Cin + 31) / 32) * (4 * Cout / 16) * 512; }

int64_t frag_elems(int M, int K) {
    const int ck = frag_ck(K);
    return (int64_t)(K / ck) * frag_nkb(ck) * ((M + 15) / 16) * 512;
}

// bf16 data-gradient copy of transposed-convolution weights from
// [ci][co][a][d]: WT[ci][(a d) Cout + co].
__global__ void k_pack_convT(const float* __restrict__ w, int Cin, int Cout, bf16_t* __restrict__ wt) {
    const int64_t n = (int64_t)4 * Cin * Cout;
    for (int64_t i = blockIdx.x * (int64_t)NT + threadIdx.x; i < n; i += (int64_t)gridDim.x * NT) {
        const int ad = (int)(i % 4), co = (int)((i / 4) % Cout), ci = (int)(i / (4 * Cout));
        wt[(int64_t)ci * 4 * Cout + ad * Cout + co] = f2bf(w[i]);
    }
}

// Transposed-convolution weights w[ci][co][a][d] in k_convT_mfma's operand
// order: element (kc, mb, lane, e) is W at row m = 16 mb + lane % 16 =
// (a d) Cout + co and ci = 32 kc + 8 (lane / 16) + e.
__global__ void k_pack_frag_t(const float* __restrict__ w, int Cin, int Cout, bf16_t* __restrict__ af, int64_t n) {
    const int nmb = 4 * Cout / 16;
    for (int64_t i = blockIdx.x * (int64_t)NT + threadIdx.x; i < n; i += (int64_t)gridDim.x * NT) {
        const int e = (int)(i & 7), lane = (int)((i >> 3) & 63);
        const int64_t rest = i >> 9;
        const int mb = (int)(rest % nmb), kc = (int)(rest / nmb);
        const int m = mb * 16 + (lane & 15), ci = kc * 32 + 8 * (lane >> 4) + e;
        const int ad = m / Cout, co = m % Cout;
        af[i] = f2bf(ci < Cin ? w[((int64_t)ci * Cout + co) * 4 + ad] : 0.f);
    }
}

__global__ void k_to_bf16(const float* __restrict__ w, bf16_t* __restrict__ o, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)NT + threadIdx.x; i < n; i += (int64_t)gridDim.x * NT) o[i] = f2bf(w[i]);
}

// Network input: NCHW float32 [n][3][H][W] to NHWC bf16 with 16 channels
// (channels 3..15 zero), one thread per pixel.
__global__ void k_input(const float* __restrict__ x, bf16_t* __restrict__ X, int N, int64_t HW) {
    const int64_t total = (int64_t)N * HW;
    for (int64_t pix = blockIdx.x * (int64_t)NT + threadIdx.x; pix < total; pix += (int64_t)gridDim.x * NT) {
        const int64_t n = pix / HW, p = pix % HW;
        bf8u lo;
        lo.u = uint4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int c = 0; c < 3; ++c) lo.h[c] = f2bf(x[(n * 3 + c) * HW + p]);
        *reinterpret_cast<uint4*>(X + pix * 16) = lo.u;
        *reinterpret_cast<uint4*>(X + pix * 16 + 8) = uint4{0u, 0u, 0u, 0u};
    }
}

int grid_for(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>((n + NT - 1) / NT, 8192)); }

}  // namespace

// ---------------------------------------------------------------------------
// Network state and the layer sequence.
struct Layer {
    int kind;            // 0 conv3x3, 1 convT 2x2, 2 conv1x1
    int cin, cout;       // real channel counts
    int64_t off;         // offset of the weights in the flat vector (bias follows)
    int64_t nw;          // weight count
    bf16_t *wf = nullptr, *wb = nullptr;   // packed bf16 weights
};

struct Unet {
    int H = 0, W = 0, maxb = 0;
    hipStream_t stream = nullptr;
    std::vector<Layer> L;
    int64_t P = 0;
    float *theta = nullptr, *m = nullptr, *v = nullptr;
    bf16_t* act = nullptr;       // all activation buffers
    bf16_t* grad = nullptr;      // all gradient buffers
    float* go = nullptr;         // dL/do [maxb][H][W]
    float* part = nullptr;       // reduction partials
    int64_t part_cap = 0;
    double* dloss = nullptr;     // per-sample loss [maxb], then partials [maxb][LOSS_BLOCKS] x 3
    // activation views (element offsets into act / grad, per-image strides)
    // C channels per pixel at pixel stride `stride`; a concatenation buffer
    // holds its two halves of C / 2 channels as planar tensors hs apart
    struct View { int64_t off; int stride; int C; int lvl; int64_t hs; };
    std::vector<View> av;        // named below
};

enum {
    A_X, A_A1, A_CAT1, A_D1A, A_D1B,
    A_P1, A_A2, A_CAT2, A_D2A, A_D2B,
    A_P2, A_A3, A_CAT3, A_D3A, A_D3B,
    A_P3, A_A4, A_B4, A_COUNT
};

// layer indices in flat order
enum { C1A, C1B, C2A, C2B, C3A, C3B, C4A, C4B, U3, D3A, D3B, U2, D2A, D2B, U1, D1A, D1B, OUT, NLAYERS };

}  // namespace esi

using namespace esi;

namespace {

const int kLayerDef[NLAYERS][3] = {
    {0, 3, 16}, {0, 16, 16}, {0, 16, 32}, {0, 32, 32}, {0, 32, 64}, {0, 64, 64},
    {0, 64, 128}, {0, 128, 128}, {1, 128, 64}, {0, 128, 64}, {0, 64, 64},
    {1, 64, 32}, {0, 64, 32}, {0, 32, 32}, {1, 32, 16}, {0, 32, 16}, {0, 16, 16}, {2, 16, 1}};

int64_t layer_weights(int kind, int ci, int co) { return kind == 0 ? (int64_t)9 * ci * co : kind == 1 ? (int64_t)4 * ci * co : ci * co; }

// A tensor view handed to the convolution launchers: pointer, pixel stride and,
// for a concatenation buffer, the distance to the second half and the first
// channel that lives there (no split: hs = 0, split beyond every channel).
struct Tv {
    bf16_t* p;
    int s;
    int64_t hs = 0;
    int split = 1 << 30;
};

struct Ctx {
    Unet* U;
    int N;
    int64_t pix(int lvl) const { return (int64_t)N * (U->H >> lvl) * (U->W >> lvl); }
    bf16_t* a(int id) const { return U->act + U->av[id].off; }
    bf16_t* g(int id) const { return U->grad + U->av[id].off; }
    // half h (0: upsampled decoder input, 1: encoder skip) of a concatenation buffer
    bf16_t* ah(int id, int h) const { return U->act + U->av[id].off + h * U->av[id].hs; }
    bf16_t* gh(int id, int h) const { return U->grad + U->av[id].off + h * U->av[id].hs; }
    Tv at(int id) const { return view(U->act, id); }
    Tv gt(int id) const { return view(U->grad, id); }
    Tv view(bf16_t* base, int id) const {
        const Unet::View& v = U->av[id];
        Tv t{base + v.off, v.stride};
        if (v.hs) { t.hs = v.hs; t.split = v.C / 2; }
        return t;
    }
    int h(int lvl) const { return U->H >> lvl; }
    int w(int lvl) const { return U->W >> lvl; }
};

template <int CB, int CK, int EPI, bool RES, bool IN>
void launch_conv3(const Ctx& c, const ConvArgs& A, int M) {
    // Waves of all 64 pixels, so that a weight operand serves 8 sums; with 64 outputs
    // the sums of half a row fill the registers.
    constexpr int PG = CB == 4 ? 2 : 4;
    using T = Conv3Tile<CB, CK, PG>;
    // persistent grid: as many workgroups as the device holds at once
    static int resident = 0;
    if (!resident) {
        int per_cu = 0, cus = 0, dev = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_conv3<CB, CK, PG, EPI, RES, IN>, T::NTW, 0) != hipSuccess)
            per_cu = 1, cus = 256;
        resident = std::max(1, per_cu) * std::max(1, cus);
    }
    const int ncog = M / (16 * CB);
    const int ntiles = ((A.W + 63) / 64) * ((A.H + T::ROWS - 1) / T::ROWS) * A.N;
    const int grid = std::min(ntiles, std::max(1, resident / ncog));
    hipLaunchKernelGGL((k_conv3<CB, CK, PG, EPI, RES, IN>), dim3(grid, ncog), dim3(T::NTW), 0, c.U->stream, A);
}

// K input channels (Cin, or Cout for a data gradient) to M outputs at level
// lvl; A brings what the epilogue needs.
template <int EPI, bool IN = false>
esi_status_t conv3(const Ctx& c, const Tv& X, int K, int layer, const Tv& Y, int M, int lvl, ConvArgs A = {}) {
    constexpr bool BWD = EPI == E_GRAD || EPI == E_MASK;
    Unet* U = c.U;
    const Layer& Ly = U->L[layer];
    A.X = X.p; A.sx = X.s; A.xhs = X.hs; A.xsplit = X.split; A.K = K;
    A.Af = BWD ? Ly.wb : Ly.wf;
    A.ncb = (M + 15) / 16;
    A.bias = BWD ? nullptr : U->theta + Ly.off + Ly.nw;
    A.Y = Y.p; A.sy = Y.s; A.yhs = Y.hs; A.ysplit = Y.split;
    A.H = c.h(lvl); A.W = c.w(lvl); A.N = c.N;
    const int ck = frag_ck(K);
    if (K % 16 || M % 16 || (K > 16 && K % 32) || (M > 32 && M % 64))
        return fail(ESI_ERR_SHAPE, "3x3 convolution channels outside the supported set");
    if (X.split < K && X.split % ck && K != ck) return fail(ESI_ERR_SHAPE, "a chunk of channels spans two tensors");
    // weights in registers: one chunk and at most 20 blocks of 4 registers
    if constexpr (EPI == E_OUT || IN) {
        if (K != 16 || M != 16) return fail(ESI_ERR_SHAPE, "fused first and last convolutions have 16 channels");
        launch_conv3<1, 16, EPI, true, IN>(c, A, M);
    } else if constexpr (EPI == E_POOL) {
        if (K != M || M > 64) return fail(ESI_ERR_SHAPE, "pooled convolutions have 16, 32 or 64 channels");
        if (M == 16) launch_conv3<1, 16, EPI, true, false>(c, A, M);
        else if (M == 32) launch_conv3<2, 32, EPI, true, false>(c, A, M);
        else launch_conv3<4, 32, EPI, false, false>(c, A, M);
    } else if (ck == 16) {
        if (M == 16) launch_conv3<1, 16, EPI, true, false>(c, A, M);
        else launch_conv3<2, 16, EPI, true, false>(c, A, M);
    } else if (M >= 64) {
        launch_conv3<4, 32, EPI, false, false>(c, A, M);
    } else if (M == 32) {
        if (K == 32) launch_conv3<2, 32, EPI, true, false>(c, A, M);
        else launch_conv3<2, 32, EPI, false, false>(c, A, M);
    } else {
        if (K != 32) return fail(ESI_ERR_SHAPE, "16 outputs are those of at most 32 channels");
        launch_conv3<1, 32, EPI, true, false>(c, A, M);
    }
    ESI_HIP_TRY(hipGetLastError());
    return ESI_OK;
}

esi_status_t need_part(Unet* U, int64_t n) {
    return grow_t(&U->part, &U->part_cap, n, U->stream);
}

// Chunks of a weight gradient: as many workgroups as two per CU over the
// channel tiles, each with the same number of pixel tiles (but the last).
int wgrad_chunks(int ntiles, int channel_tiles) {
    const int want = std::max(1, std::min(ntiles, 512 / channel_tiles));
    const int each = (ntiles + want - 1) / want;
    return (ntiles + each - 1) / each;
}

template <int CB, int IB, int ROWS>
esi_status_t launch_conv3_wgrad(const Ctx& c, const Tv& GY, int Cout, const Tv& X, int Cin, int cin_real, int H, int W,
                                float* gflat) {
    Unet* U = c.U;
    const int ct = (Cout / (16 * CB)) * (Cin / (16 * IB));
    const int nchunks = wgrad_chunks(((W + 63) / 64) * ((H + ROWS - 1) / ROWS) * c.N, ct);
    const int64_t per = (int64_t)9 * Cout * Cin;
    ESI_TRY(need_part(U, nchunks * (per + Cout)));
    float* part = U->part;
    float* bpart = U->part + nchunks * per;
    hipLaunchKernelGGL((k_conv3_wgrad<CB, IB, ROWS>), dim3(nchunks, ct), dim3(NT), 0, U->stream, GY.p, GY.s, Cout, X.p,
                       X.s, X.hs, X.split, Cin, H, W, c.N, part, bpart);
    hipLaunchKernelGGL(k_wgrad_reduce<false>, dim3((int)((per + Cout + 63) / 64)), dim3(1024), 0, U->stream, part,
                       bpart, nchunks, 9, Cout, Cin, cin_real, Cout, gflat);
    ESI_HIP_TRY(hipGetLastError());
    return ESI_OK;
}

// weight + bias gradient of a 3x3 layer into gflat: channel tiles of 32 x 32,
// or 16 where a side has no more (16 x 16 is bound by memory: taller tiles
// stage less halo)
esi_status_t conv3_wgrad(const Ctx& c, const Tv& GY, int Cout, const Tv& X, int Cin, int cin_real, int lvl,
                         float* gflat) {
    const int H = c.h(lvl), W = c.w(lvl);
    if (Cout % 16 || Cin % 16 || (Cout > 16 && Cout % 32) || (Cin > 16 && Cin % 32) || X.split % 8)
        return fail(ESI_ERR_SHAPE, "weight-gradient channels outside the supported set");
    if (Cout == 16 && Cin == 16) return launch_conv3_wgrad<1, 1, 8>(c, GY, Cout, X, Cin, cin_real, H, W, gflat);
    if (Cout == 16) return launch_conv3_wgrad<1, 2, 4>(c, GY, Cout, X, Cin, cin_real, H, W, gflat);
    if (Cin == 16) return launch_conv3_wgrad<2, 1, 4>(c, GY, Cout, X, Cin, cin_real, H, W, gflat);
    return launch_conv3_wgrad<2, 2, 4>(c, GY, Cout, X, Cin, cin_real, H, W, gflat);
}

template <int CB, int NKC>
void launch_convT(const Ctx& c, const Layer& Ly, const bf16_t* X, int sx, const float* bias, bf16_t* Y, int sy,
                  int Hi, int Wi) {
    dim3 grid((Wi + 63) / 64, (Hi + 3) / 4, c.N * (4 * Ly.cout / (16 * CB)));
    hipLaunchKernelGGL((k_convT_mfma<CB, NKC>), grid, dim3(NT), 0, c.U->stream, X, sx, Ly.wf, bias, Y, sy, Ly.cout,
                       Hi, Wi);
}

esi_status_t convT_fwd(const Ctx& c, int layer, const bf16_t* X, int sx, bf16_t* Y, int sy, int lvl_in) {
    Unet* U = c.U;
    const Layer& Ly = U->L[layer];
    const int Hi = c.h(lvl_in), Wi = c.w(lvl_in);
    const float* bias = U->theta + Ly.off + Ly.nw;
    // 4 Cout rows of D in blocks of 64; Cin in blocks of 32 (32, 64 or 128)
    if (Ly.cout % 16 || sy != Ly.cout || (Ly.cin != 32 && Ly.cin != 64 && Ly.cin != 128))
        return fail(ESI_ERR_SHAPE, "transposed convolution channels outside the supported set");
    if (Ly.cin == 32) launch_convT<4, 1>(c, Ly, X, sx, bias, Y, sy, Hi, Wi);
    else if (Ly.cin == 64) launch_convT<4, 2>(c, Ly, X, sx, bias, Y, sy, Hi, Wi);
    else launch_convT<4, 4>(c, Ly, X, sx, bias, Y, sy, Hi, Wi);
    ESI_HIP_TRY(hipGetLastError());
    return ESI_OK;
}

template <int CB, int IB>
esi_status_t launch_convT_wgrad(const Ctx& c, const Layer& Ly, const bf16_t* X, int sx, const bf16_t* GY, int sg,
                                int Hi, int Wi, float* gflat) {
    Unet* U = c.U;
    const int ct = (Ly.cout / (16 * CB)) * (Ly.cin / (16 * IB));
    const int nchunks = wgrad_chunks(((Wi + 63) / 64) * ((Hi + 1) / 2) * c.N, ct);
    const int64_t per = (int64_t)4 * Ly.cout * Ly.cin;
    ESI_TRY(need_part(U, nchunks * (per + Ly.cout)));
    float* part = U->part;
    float* bpart = U->part + nchunks * per;
    hipLaunchKernelGGL((k_convT_wgrad<CB, IB>), dim3(nchunks, ct), dim3(NT), 0, U->stream, X, sx, Ly.cin, GY, sg,
                       Ly.cout, Hi, Wi, c.N, part, bpart);
    hipLaunchKernelGGL(k_wgrad_reduce<true>, dim3((int)((per + Ly.cout + 63) / 64)), dim3(1024), 0, U->stream, part,
                       bpart, nchunks, 4, Ly.cout, Ly.cin, Ly.cin, Ly.cout, gflat);
    ESI_HIP_TRY(hipGetLastError());
    return ESI_OK;
}

// weight + bias gradient of a transposed convolution and the gradient of its
// input, masked by that activation's ReLU (act)
esi_status_t convT_back(const Ctx& c, int layer, const bf16_t* X, int sx, const bf16_t* GY, int sg,
                        bf16_t* GX, int sgx, int lvl_in, const bf16_t* act, float* gflat) {
    Unet* U = c.U;
    const Layer& Ly = U->L[layer];
    const int Hi = c.h(lvl_in), Wi = c.w(lvl_in);
    {
        const int cb = Ly.cin >= 64 ? 4 : Ly.cin / 16;
        dim3 grid((Wi + 63) / 64, (Hi + 3) / 4, c.N * (Ly.cin / (16 * cb)));
        if (cb == 4)
            hipLaunchKernelGGL(k_convT_dgrad_mfma<4>, grid, dim3(NT), 0, U->stream, GY, sg, Ly.cout, Ly.wb, GX,
                               sgx, Ly.cin, Hi, Wi, act);
        else
            hipLaunchKernelGGL(k_convT_dgrad_mfma<2>, grid, dim3(NT), 0, U->stream, GY, sg, Ly.cout, Ly.wb, GX,
                               sgx, Ly.cin, Hi, Wi, act);
    }
    if (Ly.cin % 32 || Ly.cout % 16 || (Ly.cout > 16 && Ly.cout % 32))
        return fail(ESI_ERR_SHAPE, "transposed convolution channels outside the supported set");
    if (Ly.cout == 16) return launch_convT_wgrad<1, 2>(c, Ly, X, sx, GY, sg, Hi, Wi, gflat + Ly.off);
    return launch_convT_wgrad<2, 2>(c, Ly, X, sx, GY, sg, Hi, Wi, gflat + Ly.off);
}

// Forward pass.  Activations of every layer are left for a backward pass if
// `train`; else the padded input and the last convolution's output are not
// formed (168 MB of 8 images of 408 x 808 written and read).
esi_status_t forward(const Ctx& c, const float* x, float* o, bool train) {
    Unet* U = c.U;
    const int64_t HW = (int64_t)U->H * U->W;
    auto T = [](bf16_t* p, int s) { return Tv{p, s}; };
    // encoder: each level's second convolution writes the skip half of the
    // decoder's concatenation buffer and the next level's pooled input
    auto pooled = [](bf16_t* p) { ConvArgs A = {}; A.pool = p; return A; };
    if (train) {
        hipLaunchKernelGGL(k_input, dim3(grid_for(c.N * HW)), dim3(NT), 0, U->stream, x, c.a(A_X), c.N, HW);
        ESI_TRY(conv3<E_FWD>(c, c.at(A_X), 16, C1A, c.at(A_A1), 16, 0));
    } else {
        ConvArgs A = {};
        A.xin = x;
        ESI_TRY((conv3<E_FWD, true>(c, c.at(A_X), 16, C1A, c.at(A_A1), 16, 0, A)));
    }
    ESI_TRY(conv3<E_POOL>(c, c.at(A_A1), 16, C1B, T(c.ah(A_CAT1, 1), 16), 16, 0, pooled(c.a(A_P1))));
    ESI_TRY(conv3<E_FWD>(c, c.at(A_P1), 16, C2A, c.at(A_A2), 32, 1));
    ESI_TRY(conv3<E_POOL>(c, c.at(A_A2), 32, C2B, T(c.ah(A_CAT2, 1), 32), 32, 1, pooled(c.a(A_P2))));
    ESI_TRY(conv3<E_FWD>(c, c.at(A_P2), 32, C3A, c.at(A_A3), 64, 2));
    ESI_TRY(conv3<E_POOL>(c, c.at(A_A3), 64, C3B, T(c.ah(A_CAT3, 1), 64), 64, 2, pooled(c.a(A_P3))));
    ESI_TRY(conv3<E_FWD>(c, c.at(A_P3), 64, C4A, c.at(A_A4), 128, 3));
    ESI_TRY(conv3<E_FWD>(c, c.at(A_A4), 128, C4B, c.at(A_B4), 128, 3));
    // decoder: the transposed convolution writes the first half
    ESI_TRY(convT_fwd(c, U3, c.a(A_B4), 128, c.ah(A_CAT3, 0), 64, 3));
    ESI_TRY(conv3<E_FWD>(c, c.at(A_CAT3), 128, D3A, c.at(A_D3A), 64, 2));
    ESI_TRY(conv3<E_FWD>(c, c.at(A_D3A), 64, D3B, c.at(A_D3B), 64, 2));
    ESI_TRY(convT_fwd(c, U2, c.a(A_D3B), 64, c.ah(A_CAT2, 0), 32, 2));
    ESI_TRY(conv3<E_FWD>(c, c.at(A_CAT2), 64, D2A, c.at(A_D2A), 32, 1));
    ESI_TRY(conv3<E_FWD>(c, c.at(A_D2A), 32, D2B, c.at(A_D2B), 32, 1));
    ESI_TRY(convT_fwd(c, U1, c.a(A_D2B), 32, c.ah(A_CAT1, 0), 16, 1));
    ESI_TRY(conv3<E_FWD>(c, c.at(A_CAT1), 32, D1A, c.at(A_D1A), 16, 0));
    const Layer& Lo = U->L[OUT];
    ConvArgs A = {};
    A.wo = Lo.wf;
    A.bo = U->theta + Lo.off + Lo.nw;
    A.o = o;
    return conv3<E_OUT>(c, c.at(A_D1A), 16, D1B, train ? c.at(A_D1B) : T(nullptr, 16), 16, 0, A);
}

// Backward pass from U->go into the flat gradient gflat (after forward()).
esi_status_t backward(const Ctx& c, float* gflat) {
    Unet* U = c.U;
    auto T = [](bf16_t* p, int s) { return Tv{p, s}; };
    // output layer: g_d1b = bf16(w go) masked by d1b > 0; weight / bias sums
    {
        const int64_t npx = c.pix(0);
        const int nchunks = (int)std::max<int64_t>(1, std::min<int64_t>(1024, npx / 1024));
        const int64_t ppc = (npx + nchunks - 1) / nchunks;
        ESI_TRY(need_part(U, (int64_t)nchunks * 17));
        const Layer& Lo = U->L[OUT];
        hipLaunchKernelGGL(k_out_back, dim3(nchunks), dim3(NT), 0, U->stream, U->go, c.a(A_D1B), 16, Lo.wf,
                           c.g(A_D1B), 16, npx, ppc, U->part);
        // 16 weights and the bias: as a 1-tap layer of 17 input channels
        hipLaunchKernelGGL(k_wgrad_reduce<true>, dim3(1), dim3(1024), 0, U->stream, U->part, U->part, nchunks, 1, 1, 17,
                           17, 0, gflat + Lo.off);
        ESI_HIP_TRY(hipGetLastError());
    }
    // weight gradient of a 3x3 layer from its output gradient GY and input X,
    // then (GX.p non-null) the gradient of its input, masked by the ReLU of act
    // (the input itself, when that is another layer's output)
    auto conv_back = [&](int layer, const Tv& GY, int Cout, const Tv& X, int Cin, int lvl, const Tv& GX,
                         const bf16_t* act = nullptr) -> esi_status_t {
        const Layer& Ly = U->L[layer];
        ESI_TRY(conv3_wgrad(c, GY, Cout, X, Cin, Ly.cin, lvl, gflat + Ly.off));
        if (!GX.p) return ESI_OK;
        ConvArgs A = {};
        A.act = act;
        return act ? conv3<E_MASK>(c, GY, Cout, layer, GX, Cin, lvl, A) : conv3<E_GRAD>(c, GY, Cout, layer, GX, Cin, lvl);
    };
    // level 1 decoder: d1b, d1a (d1b's gradient is already masked)
    ESI_TRY(conv_back(D1B, c.gt(A_D1B), 16, c.at(A_D1A), 16, 0, c.gt(A_D1A), c.a(A_D1A)));
    ESI_TRY(conv_back(D1A, c.gt(A_D1A), 16, c.at(A_CAT1), 32, 0, c.gt(A_CAT1)));
    ESI_TRY(convT_back(c, U1, c.a(A_D2B), 32, c.gh(A_CAT1, 0), 16, c.g(A_D2B), 32, 1, c.a(A_D2B), gflat));
    // level 2 decoder
    ESI_TRY(conv_back(D2B, c.gt(A_D2B), 32, c.at(A_D2A), 32, 1, c.gt(A_D2A), c.a(A_D2A)));
    ESI_TRY(conv_back(D2A, c.gt(A_D2A), 32, c.at(A_CAT2), 64, 1, c.gt(A_CAT2)));
    ESI_TRY(convT_back(c, U2, c.a(A_D3B), 64, c.gh(A_CAT2, 0), 32, c.g(A_D3B), 64, 2, c.a(A_D3B), gflat));
    // level 3 decoder
    ESI_TRY(conv_back(D3B, c.gt(A_D3B), 64, c.at(A_D3A), 64, 2, c.gt(A_D3A), c.a(A_D3A)));
    ESI_TRY(conv_back(D3A, c.gt(A_D3A), 64, c.at(A_CAT3), 128, 2, c.gt(A_CAT3)));
    ESI_TRY(convT_back(c, U3, c.a(A_B4), 128, c.gh(A_CAT3, 0), 64, c.g(A_B4), 128, 3, c.a(A_B4), gflat));
    // bottleneck
    ESI_TRY(conv_back(C4B, c.gt(A_B4), 128, c.at(A_A4), 128, 3, c.gt(A_A4), c.a(A_A4)));
    ESI_TRY(conv_back(C4A, c.gt(A_A4), 128, c.at(A_P3), 64, 3, c.gt(A_P3)));
    // encoder levels: gradient into e_l = pool path + skip, masked by e_l > 0;
    // the e_l gradient goes into the skip half of the concat gradient buffer
    struct Enc { int lvl, ch, cat, p, a, cb, ca, pin; };
    const Enc enc[3] = {{2, 64, A_CAT3, A_P3, A_A3, C3B, C3A, A_P2},
                        {1, 32, A_CAT2, A_P2, A_A2, C2B, C2A, A_P1},
                        {0, 16, A_CAT1, A_P1, A_A1, C1B, C1A, A_X}};
    for (const Enc& e : enc) {
        const int64_t n = c.pix(e.lvl) * (e.ch / 8);
        hipLaunchKernelGGL(k_pool_back, dim3(grid_for(n)), dim3(NT), 0, U->stream, c.g(e.p), c.gh(e.cat, 1),
                           c.ah(e.cat, 1), c.gh(e.cat, 1), e.ch, c.N, c.h(e.lvl), c.w(e.lvl));
        ESI_HIP_TRY(hipGetLastError());
        const int cin_a = e.lvl == 0 ? 16 : e.ch / 2;
        ESI_TRY(conv_back(e.cb, T(c.gh(e.cat, 1), e.ch), e.ch, c.at(e.a), e.ch, e.lvl, c.gt(e.a), c.a(e.a)));
        ESI_TRY(conv_back(e.ca, c.gt(e.a), e.ch, c.at(e.pin), cin_a, e.lvl,
                          e.lvl == 0 ? Tv{nullptr, 0} : c.gt(e.pin)));
    }
    return ESI_OK;
}

esi_status_t pack(Unet* U) {
    for (Layer& Ly : U->L) {
        const float* w = U->theta + Ly.off;
        if (Ly.kind == 0) {
            const int cpad = Ly.cin < 16 ? 16 : Ly.cin;
            const int64_t nf = frag_elems(Ly.cout, cpad), nb = frag_elems(cpad, Ly.cout);
            hipLaunchKernelGGL(k_pack_frag, dim3(grid_for(nf)), dim3(NT), 0, U->stream, w, Ly.cout, Ly.cin, Ly.cout,
                               cpad, 0, Ly.wf, nf);
            hipLaunchKernelGGL(k_pack_frag, dim3(grid_for(nb)), dim3(NT), 0, U->stream, w, Ly.cout, Ly.cin, Ly.cin,
                               Ly.cout, 1, Ly.wb, nb);
        } else if (Ly.kind == 1) {
            const int64_t nf = convT_frag_elems(Ly.cin, Ly.cout);
            hipLaunchKernelGGL(k_pack_frag_t, dim3(grid_for(nf)), dim3(NT), 0, U->stream, w, Ly.cin, Ly.cout,
                               Ly.wf, nf);
            hipLaunchKernelGGL(k_pack_convT, dim3(grid_for(Ly.nw)), dim3(NT), 0, U->stream, w, Ly.cin, Ly.cout,
                               Ly.wb);
        } else {
            hipLaunchKernelGGL(k_to_bf16, dim3(grid_for(Ly.nw)), dim3(NT), 0, U->stream, w, Ly.wf, Ly.nw);
        }
    }
    ESI_HIP_TRY(hipGetLastError());
    return ESI_OK;
}

void free_unet(Unet* U) {
    for (Layer& Ly : U->L) {
        if (Ly.wf) hipFree(Ly.wf);
        if (Ly.wb) hipFree(Ly.wb);
    }
    void* b[] = {U->theta, U->m, U->v, U->act, U->grad, U->go, U->part, U->dloss};
    for (void* p : b)
        if (p) hipFree(p);
    delete U;
}

Unet* as_unet(esi_unet_t u) { return reinterpret_cast<Unet*>(u); }

}  // namespace

extern "C" int64_t esi_unet_num_params(void) {
    int64_t P = 0;
    for (int l = 0; l < NLAYERS; ++l)
        P += layer_weights(kLayerDef[l][0], kLayerDef[l][1], kLayerDef[l][2]) + kLayerDef[l][2];
    return P;
}

extern "C" esi_status_t esi_unet_create(esi_unet_t* out, int32_t H, int32_t W, int32_t max_batch,
                                        void* stream) {
    set_error("");
    if (!out) return fail(ESI_ERR_ARG, "null output");
    *out = nullptr;
    if (H < 8 || W < 8 || H % 8 || W % 8) return fail(ESI_ERR_SHAPE, "H and W must be positive multiples of 8");
    if (max_batch < 1) return fail(ESI_ERR_ARG, "max_batch must be >= 1");
    if ((int64_t)H * W * max_batch > ((int64_t)1 << 31) / 128)
        return fail(ESI_ERR_SHAPE, "batch of images too large for one network buffer");
    Unet* U = new Unet;
    U->H = H; U->W = W; U->maxb = max_batch;
    U->stream = (hipStream_t)stream;
    int64_t off = 0;
    for (int l = 0; l < NLAYERS; ++l) {
        Layer Ly;
        Ly.kind = kLayerDef[l][0]; Ly.cin = kLayerDef[l][1]; Ly.cout = kLayerDef[l][2];
        Ly.off = off;
        Ly.nw = layer_weights(Ly.kind, Ly.cin, Ly.cout);
        off += Ly.nw + Ly.cout;
        U->L.push_back(Ly);
    }
    U->P = off;
    // activation views: offset, channels per pixel, level
    const int defs[A_COUNT][2] = {{16, 0}, {16, 0}, {32, 0}, {16, 0}, {16, 0},
                                  {16, 1}, {32, 1}, {64, 1}, {32, 1}, {32, 1},
                                  {32, 2}, {64, 2}, {128, 2}, {64, 2}, {64, 2},
                                  {64, 3}, {128, 3}, {128, 3}};
    int64_t aoff = 0;
    for (int i = 0; i < A_COUNT; ++i) {
        Unet::View vw;
        const bool cat = i == A_CAT1 || i == A_CAT2 || i == A_CAT3;
        vw.off = aoff; vw.C = defs[i][0]; vw.lvl = defs[i][1];
        vw.stride = cat ? vw.C / 2 : vw.C;
        vw.hs = cat ? (int64_t)max_batch * (H >> vw.lvl) * (W >> vw.lvl) * (vw.C / 2) : 0;
        aoff += (int64_t)max_batch * (H >> vw.lvl) * (W >> vw.lvl) * vw.C;
        aoff = (aoff + 63) / 64 * 64;
        U->av.push_back(vw);
    }
    auto fail_oom = [&]() { free_unet(U); return fail(ESI_ERR_OOM, "network allocation failed"); };
    if (hipMalloc(&U->theta, U->P * 4) != hipSuccess || hipMalloc(&U->m, U->P * 4) != hipSuccess ||
        hipMalloc(&U->v, U->P * 4) != hipSuccess || hipMalloc(&U->act, aoff * 2) != hipSuccess ||
        hipMalloc(&U->grad, aoff * 2) != hipSuccess ||
        hipMalloc(&U->go, (int64_t)max_batch * H * W * 4) != hipSuccess ||
        hipMalloc(&U->dloss, (int64_t)max_batch * (1 + 3 * LOSS_BLOCKS) * 8) != hipSuccess)
        return fail_oom();
    for (Layer& Ly : U->L) {
        const int cpad = Ly.cin < 16 ? 16 : Ly.cin;
        const int64_t nf = Ly.kind == 0 ? frag_elems(Ly.cout, cpad) : Ly.kind == 1 ? convT_frag_elems(Ly.cin, Ly.cout)
                                                                            : Ly.nw;
        if (hipMalloc(&Ly.wf, nf * 2) != hipSuccess) return fail_oom();
        if (Ly.kind == 0 && hipMalloc(&Ly.wb, frag_elems(cpad, Ly.cout) * 2) != hipSuccess) return fail_oom();
        if (Ly.kind == 1 && hipMalloc(&Ly.wb, Ly.nw * 2) != hipSuccess) return fail_oom();
    }
    // zero everything so unused padding channels never hold garbage
    if (hipMemsetAsync(U->act, 0, aoff * 2, U->stream) != hipSuccess ||
        hipMemsetAsync(U->grad, 0, aoff * 2, U->stream) != hipSuccess ||
        hipMemsetAsync(U->theta, 0, U->P * 4, U->stream) != hipSuccess ||
        hipMemsetAsync(U->m, 0, U->P * 4, U->stream) != hipSuccess ||
        hipMemsetAsync(U->v, 0, U->P * 4, U->stream) != hipSuccess ||
        hipStreamSynchronize(U->stream) != hipSuccess) {
        free_unet(U);
        return fail(ESI_ERR_HIP, "network initialisation failed");
    }
    *out = reinterpret_cast<esi_unet_t>(U);
    return ESI_OK;
}

extern "C" esi_status_t esi_unet_destroy(esi_unet_t u) {
    set_error("");
    if (!u) return ESI_OK;
    Unet* U = as_unet(u);
    hipStreamSynchronize(U->stream);
    free_unet(U);
    return ESI_OK;
}

extern "C" esi_status_t esi_unet_set_params(esi_unet_t u, const float* theta) {
    set_error("");
    if (!u || !theta) return fail(ESI_ERR_ARG, "null argument");
    Unet* U = as_unet(u);
    ESI_HIP_TRY(hipMemcpyAsync(U->theta, theta, U->P * 4, hipMemcpyDefault, U->stream));
    ESI_HIP_TRY(hipMemsetAsync(U->m, 0, U->P * 4, U->stream));
    ESI_HIP_TRY(hipMemsetAsync(U->v, 0, U->P * 4, U->stream));
    ESI_TRY(pack(U));
    ESI_HIP_TRY(hipStreamSynchronize(U->stream));
    return ESI_OK;
}

extern "C" esi_status_t esi_unet_get_params(esi_unet_t u, float* theta) {
    set_error("");
    if (!u || !theta) return fail(ESI_ERR_ARG, "null argument");
    Unet* U = as_unet(u);
    ESI_HIP_TRY(hipMemcpyAsync(theta, U->theta, U->P * 4, hipMemcpyDefault, U->stream));
    ESI_HIP_TRY(hipStreamSynchronize(U->stream));
    return ESI_OK;
}

extern "C" esi_status_t esi_unet_forward(esi_unet_t u, const float* x, float* o, int32_t batch) {
    set_error("");
    if (!u || !x || !o) return fail(ESI_ERR_ARG, "null argument");
    Unet* U = as_unet(u);
    if (batch < 1 || batch > U->maxb) return fail(ESI_ERR_ARG, "batch outside [1, max_batch]");
    Ctx c{U, batch};
    return forward(c, x, o, false);
}

extern "C" esi_status_t esi_unet_loss_weights(const float* a, const float* c, int32_t batch, int64_t npix,
                                              float* w, void* stream) {
    set_error("");
    if (!a || !c || !w) return fail(ESI_ERR_ARG, "null argument");
    if (batch < 1 || npix < 1) return fail(ESI_ERR_ARG, "empty batch");
    hipLaunchKernelGGL(k_loss_weights, dim3(batch), dim3(NT), 0, (hipStream_t)stream, a, c, npix, w);
    ESI_HIP_TRY(hipGetLastError());
    return ESI_OK;
}

extern "C" esi_status_t esi_unet_loss_grad(esi_unet_t u, const float* x, const float* a, const float* cc,
                                           const float* weight, int32_t batch, float* grad, double* loss) {
    set_error("");
    if (!u || !x || !a || !cc || !grad) return fail(ESI_ERR_ARG, "null argument");
    Unet* U = as_unet(u);
    if (batch < 1 || batch > U->maxb) return fail(ESI_ERR_ARG, "batch outside [1, max_batch]");
    Ctx c{U, batch};
    const int64_t npix = (int64_t)U->H * U->W;
    ESI_TRY(grow_t(&U->part, &U->part_cap, (int64_t)batch * npix, U->stream));   // o scratch
    float* o = U->part;
    ESI_TRY(forward(c, x, o, true));
    double* sums = U->dloss + U->maxb;                     // [batch][LOSS_BLOCKS][2], then the loss partials
    double* lpart = sums + (int64_t)U->maxb * LOSS_BLOCKS * 2;
    if (!weight)
        hipLaunchKernelGGL(k_loss_sums, dim3(LOSS_BLOCKS, batch), dim3(NT), 0, U->stream, a, cc, npix, sums);
    hipLaunchKernelGGL(k_scaling_loss, dim3(LOSS_BLOCKS, batch), dim3(NT), 0, U->stream, o, a, cc, weight, sums, npix,
                       batch, U->go, lpart);
    hipLaunchKernelGGL(k_loss_finish, dim3((batch + 63) / 64), dim3(64), 0, U->stream, lpart, batch, U->dloss);
    ESI_HIP_TRY(hipGetLastError());
    ESI_TRY(backward(c, grad));
    if (loss) {
        std::vector<double> h(batch);
        ESI_HIP_TRY(hipMemcpyAsync(h.data(), U->dloss, batch * 8, hipMemcpyDeviceToHost, U->stream));
        ESI_HIP_TRY(hipStreamSynchronize(U->stream));
        double s = 0.0;
        for (double v : h) s += v;
        *loss = s / batch;
    }
    return ESI_OK;
}

extern "C" esi_status_t esi_unet_adam(esi_unet_t u, const float* grad, float lr, float beta1, float beta2,
                                      float eps, int32_t step, float clip_norm) {
    set_error("");
    if (!u || !grad) return fail(ESI_ERR_ARG, "null argument");
    if (step < 1) return fail(ESI_ERR_ARG, "Adam step counts from 1");
    Unet* U = as_unet(u);
    const float bc1 = (float)(1.0 - std::pow((double)beta1, step));
    const float bc2 = (float)(1.0 - std::pow((double)beta2, step));
    float* factor = nullptr;
    if (clip_norm > 0.f) {
        const int nb = 256;
        ESI_TRY(grow_t(&U->part, &U->part_cap, (int64_t)2 * nb + 2, U->stream));
        double* part = reinterpret_cast<double*>(U->part);
        factor = U->part + 2 * nb;
        hipLaunchKernelGGL(k_sqnorm, dim3(nb), dim3(NT), 0, U->stream, grad, U->P, part);
        hipLaunchKernelGGL(k_clip_factor, dim3(1), dim3(64), 0, U->stream, part, nb, clip_norm, factor);
    }
    hipLaunchKernelGGL(k_adam, dim3(grid_for(U->P)), dim3(NT), 0, U->stream, U->theta, U->m, U->v, grad, U->P,
                       lr, beta1, beta2, eps, bc1, bc2, factor);
    ESI_HIP_TRY(hipGetLastError());
    return pack(U);
}

namespace esi {

esi_status_t unet_dims(esi_unet_t u, int* H, int* W, int* maxb) {
    if (!u) return fail(ESI_ERR_ARG, "null network");
    Unet* U = as_unet(u);
    *H = U->H; *W = U->W; *maxb = U->maxb;
    return ESI_OK;
}

// Forward pass queued on `stream` (the caller's) instead of the network's own.
esi_status_t unet_forward_on(esi_unet_t u, hipStream_t stream, const float* x, float* o, int batch) {
    Unet* U = as_unet(u);
    if (batch < 1 || batch > U->maxb) return fail(ESI_ERR_ARG, "batch outside [1, max_batch]");
    hipStream_t own = U->stream;
    U->stream = stream;
    Ctx c{U, batch};
    esi_status_t st = forward(c, x, o, false);
    U->stream = own;
    return st;
}

}  // namespace esi
