// surrogate.hip -- gfx950 kernels of the learned surrogate (include/lbcg_surrogate.h):
// 3D convolutions as implicit GEMMs on the CDNA4 matrix cores
// (v_mfma_f32_16x16x32_bf16: BF16 operands, FP32 accumulation), their data and
// weight gradients, and the element-wise layers, loss and optimiser of a U-Net.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <mutex>

#include "lbcg_surrogate.h"

namespace sg {

typedef __bf16 bf16;
typedef bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// One MFMA 16x16x32 step.  Lane l (0..63) supplies A[l % 16][8 (l / 16) + j]
// and B[8 (l / 16) + j][l % 16] for j = 0..7, and receives
// D[4 (l / 16) + j][l % 16] for j = 0..3.
__device__ inline f32x4 mfma(const bf16x8 &a, const bf16x8 &b, const f32x4 &c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ inline int64_t npos(const sg_view &v) { return (int64_t)v.n * v.d * v.h * v.w; }

struct Pos { int n, z, y, x; };

__device__ inline Pos decode(const sg_view &v, int64_t p)
{
    Pos q;
    q.x = (int)(p % v.w);
    p /= v.w;
    q.y = (int)(p % v.h);
    p /= v.h;
    q.z = (int)(p % v.d);
    q.n = (int)(p / v.d);
    return q;
}

// Neighbour at offset (dz, dy, dx): flat position, or -1 where zero padding applies.
__device__ inline int64_t shifted(const sg_view &v, const Pos &q, int dz, int dy, int dx, int pmask)
{
    int z = q.z + dz, y = q.y + dy, x = q.x + dx;
    if (x < 0 || x >= v.w) {
        if (!(pmask & 1)) return -1;
        x = x < 0 ? x + v.w : x - v.w;
    }
    if (y < 0 || y >= v.h) {
        if (!(pmask & 2)) return -1;
        y = y < 0 ? y + v.h : y - v.h;
    }
    if (z < 0 || z >= v.d) {
        if (!(pmask & 4)) return -1;
        z = z < 0 ? z + v.d : z - v.d;
    }
    return (((int64_t)q.n * v.d + z) * v.h + y) * v.w + x;
}

__device__ inline void tap_offset(int tap, int k, int &dz, int &dy, int &dx)
{
    if (k == 1) {
        dz = dy = dx = 0;
        return;
    }
    dz = tap / 9 - 1;
    dy = (tap / 3) % 3 - 1;
    dx = tap % 3 - 1;
}

// ------------------------------------------------------------- forward
// Workgroup: 4 wavefronts; each wave owns a register tile of NO blocks of 16
// output channels x FP blocks of 16 positions (64 consecutive positions), so
// one weight fragment feeds FP MFMAs and one input fragment feeds NO of them.
// blockIdx.y selects the 16 NO output channels.  The K loop walks taps x
// input channels in groups of 8 (one 16-byte load per lane and operand).
constexpr int FP = 4;

template <int NO>
__global__ __launch_bounds__(256) void k_conv_fwd(sg_view x, const bf16 *__restrict__ W,
                                                  const float *__restrict__ bias, int k, int pmask, int relu,
                                                  sg_view y, sg_view y32, int accumulate)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 15, grp = lane >> 4;
    const int64_t P = npos(x);
    const int64_t p0 = ((int64_t)blockIdx.x * 4 + wave) * (16 * FP);
    const int co0 = blockIdx.y * 16 * NO;
    const int ci = x.c, g8 = ci >> 3, taps = k * k * k;
    const int K8 = taps * g8, K = taps * ci;
    Pos q[FP];
    bool pv[FP];
    #pragma unroll
    for (int i = 0; i < FP; ++i) {
        const int64_t pb = p0 + 16 * i + col;
        pv[i] = pb < P;
        q[i] = decode(x, pv[i] ? pb : 0);
    }
    const bf16 *xp = reinterpret_cast<const bf16 *>(x.p) + x.coff;
    const bf16 *wrow = W + (int64_t)(co0 + col) * K;
    f32x4 acc[NO][FP];
    #pragma unroll
    for (int o = 0; o < NO; ++o)
        #pragma unroll
        for (int i = 0; i < FP; ++i) acc[o][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bf16x8 zero = {};
    int last_tap = -1;
    int64_t src[FP];
    #pragma unroll
    for (int i = 0; i < FP; ++i) src[i] = -1;
    for (int kb = 0; kb < (K8 + 3) >> 2; ++kb) {
        const int g = (kb << 2) + grp;
        bf16x8 a[NO], b[FP];
        #pragma unroll
        for (int o = 0; o < NO; ++o) a[o] = zero;
        #pragma unroll
        for (int i = 0; i < FP; ++i) b[i] = zero;
        if (g < K8) {
            const int tap = g / g8, c8 = g - tap * g8;
            #pragma unroll
            for (int o = 0; o < NO; ++o) a[o] = *reinterpret_cast<const bf16x8 *>(wrow + (int64_t)16 * o * K + (g << 3));
            if (tap != last_tap) {
                int dz, dy, dx;
                tap_offset(tap, k, dz, dy, dx);
                #pragma unroll
                for (int i = 0; i < FP; ++i) src[i] = pv[i] ? shifted(x, q[i], dz, dy, dx, pmask) : -1;
                last_tap = tap;
            }
            #pragma unroll
            for (int i = 0; i < FP; ++i)
                if (src[i] >= 0) b[i] = *reinterpret_cast<const bf16x8 *>(xp + src[i] * x.ctot + (c8 << 3));
        }
        #pragma unroll
        for (int o = 0; o < NO; ++o)
            #pragma unroll
            for (int i = 0; i < FP; ++i) acc[o][i] = mfma(a[o], b[i], acc[o][i]);
    }
    #pragma unroll
    for (int o = 0; o < NO; ++o)
        #pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int oc = co0 + 16 * o + (grp << 2) + j;
            const bool sy = y.p && oc < y.c, s32 = y32.p && oc < y32.c;
            if (!sy && !s32) continue;                 // padded output rows
            const float bo = bias ? bias[oc] : 0.f;
            #pragma unroll
            for (int i = 0; i < FP; ++i) {
                if (!pv[i]) continue;
                const int64_t pb = p0 + 16 * i + col;
                float v = acc[o][i][j] + bo;
                if (relu) v = fmaxf(v, 0.f);
                if (sy) reinterpret_cast<bf16 *>(y.p)[pb * y.ctot + y.coff + oc] = (bf16)v;
                if (s32) {
                    float *out = reinterpret_cast<float *>(y32.p) + pb * y32.ctot + y32.coff + oc;
                    *out = accumulate ? *out + v : v;
                }
            }
        }
}

// 3x3x3 convolution on a brick of 16 (x) x 4 (y) x BZ (z) output positions of
// one batch item, for tensors whose extents are multiples of 16, 4 and 4.  The
// brick's input halo is staged in LDS one chunk of CT input channels at a time,
// so each input value is fetched from memory once per chunk instead of once per
// tap; the 27 taps then read their B fragments (a row of 16 positions) from LDS.
// Wave w owns ZW = BZ / 4 z-planes of the brick and NO blocks of 16 output
// channels.  A staged position holds CT/8 16-byte chunks, XOR-swizzled with the
// position's x against bank conflicts.
// DYR: the order in which a chunk's products are summed.  true: K blocks of four
// (dz, dx, channel group) combinations, each block's three dy taps in turn; a
// lane then loads the 6 halo rows its 4 output rows need once and feeds them to
// three K blocks, half the LDS reads.  false: K blocks of four consecutive (tap,
// channel group) pairs.  sg_conv3d_fwd chooses chunk length and order.
// WLDS: the chunk's weights are staged in LDS too, and the next chunk's loads
// fly during the K loop.  For launches that leave CUs idle or with one workgroup:
// there every K block would otherwise wait for its weights from L2.

// Workgroups are dealt to the 8 XCDs in turn by their linear id (x
// fastest).  This bijection on 0 .. n-1 maps the linear id to a position in
// the work order such that each XCD gets a contiguous run of it, so that
// neighbouring bricks, whose halos overlap, share an L2.
__device__ inline unsigned xcd_contiguous(unsigned lin, unsigned n)
{
    const unsigned x = lin & 7u, l = lin >> 3, q = n >> 3, r = n & 7u;
    return x * q + min(x, r) + l;
}

// Coordinate g in -1 .. n of an axis of n positions: wrapped when periodic, -1
// where the input is zero.
__device__ inline int edge(int g, int n, bool periodic)
{
    if (g < 0) return periodic ? n - 1 : -1;
    if (g < n) return g;
    return periodic ? 0 : -1;
}

// A lane's 4 consecutive output channels oc0 .. of position pb, stored as one
// 8-byte (BF16) or 16-byte (FP32) access when the slice allows it.
__device__ inline void store_out(const sg_view &y, const sg_view &y32, int64_t pb, int oc0, f32x4 v, int relu,
                                 int accumulate)
{
    if (relu)
        #pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = fmaxf(v[j], 0.f);
    if (y.p) {
        bf16 *out = reinterpret_cast<bf16 *>(y.p) + pb * y.ctot + y.coff + oc0;
        if (((y.ctot | y.coff) & 3) == 0 && ((uintptr_t)y.p & 7) == 0 && oc0 + 3 < y.c) {
            *reinterpret_cast<bf16x4 *>(out) = bf16x4{(bf16)v[0], (bf16)v[1], (bf16)v[2], (bf16)v[3]};
        } else {
            #pragma unroll
            for (int j = 0; j < 4; ++j)
                if (oc0 + j < y.c) out[j] = (bf16)v[j];
        }
    }
    if (y32.p) {
        float *out = reinterpret_cast<float *>(y32.p) + pb * y32.ctot + y32.coff + oc0;
        if (((y32.ctot | y32.coff) & 3) == 0 && ((uintptr_t)y32.p & 15) == 0 && oc0 + 3 < y32.c) {
            f32x4 *o4 = reinterpret_cast<f32x4 *>(out);
            *o4 = accumulate ? *o4 + v : v;
        } else {
            #pragma unroll
            for (int j = 0; j < 4; ++j)
                if (oc0 + j < y32.c) out[j] = accumulate ? out[j] + v[j] : v[j];
        }
    }
}

// The biases of output channels oc0 .. oc0 + 3 (zero past the views' channels).
__device__ inline f32x4 bias4(const float *bias, int oc0, const sg_view &y, const sg_view &y32)
{
    const int nb = max(y.p ? y.c : 0, y32.p ? y32.c : 0);
    f32x4 b;
    #pragma unroll
    for (int j = 0; j < 4; ++j) b[j] = bias && oc0 + j < nb ? bias[oc0 + j] : 0.f;
    return b;
}

// Three workgroups per CU for two output blocks of 16-channel chunks: left to
// itself the compiler took 173 registers, five too many for three (16 -> 32
// channels on 128^3 positions 93 us, 79 so; no spills).
template <int NO, int BZ, int CT, bool DYR, bool WLDS>
__global__ __launch_bounds__(256, NO == 2 && BZ == 8 && CT == 16 ? 3 : 1) void k_conv3(sg_view x, const bf16 *__restrict__ W, const float *__restrict__ bias,
                                               int pmask, int relu, sg_view y, sg_view y32, int accumulate, int nbx,
                                               int nby, int nbz)
{
    constexpr int BX = 16, BY = 4, HX = BX + 2, HY = BY + 2, HZ = BZ + 2, ROWS = HY * HZ, HP = HX * ROWS;
    constexpr int NC = CT / 8, XSPAN = 16 / NC;           // chunks per position; positions per 256 bytes
    constexpr int ZW = BZ / 4, NF = ZW * BY, NR = BY + 2;
    static_assert(BZ % 4 == 0 && ZW <= 2, "brick shape");
    // staging: rows of BX interior positions, RPW rows per wave and load, then
    // the two side columns of every row
    constexpr int LR = BX * NC, RPW = 64 / LR, NL = (ROWS + 4 * RPW - 1) / (4 * RPW);
    constexpr int SIDE = 2 * NC * ROWS, NS = (SIDE + 255) / 256;
    constexpr int WE = WLDS ? 27 * 16 * NO * NC : 0, NW = (WE + 255) / 256;
    __shared__ __attribute__((aligned(16))) bf16 halo[HP * CT];
    __shared__ __attribute__((aligned(16))) bf16 wl[WLDS ? WE * 8 : 8];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int col = lane & 15, grp = lane >> 4;
    auto swz = [](int hx, int c8) { return c8 ^ ((hx / XSPAN) & (NC - 1)); };
    // work order: output-channel blocks of a brick adjacent, then bricks x-fastest
    const unsigned ncb = gridDim.y;
    const unsigned v = xcd_contiguous(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * ncb);
    int bi = (int)(v / ncb);
    const int X0 = bi % nbx * BX;
    bi /= nbx;
    const int Y0 = bi % nby * BY;
    bi /= nby;
    const int Z0 = bi % nbz * BZ;
    const int n = bi / nbz;
    const int co0 = (int)(v % ncb) * 16 * NO;
    const int ci = x.c, K = 27 * ci;
    // offsets of the input in 16-byte chunks, 32 bits per batch item (host-checked)
    const int ct8 = x.ctot >> 3;
    const bf16x8 *xp = reinterpret_cast<const bf16x8 *>(reinterpret_cast<const bf16 *>(x.p) + x.coff) +
                       (int64_t)n * x.d * x.h * x.w * ct8;
    const bf16x8 zero = {};

    // this lane's part of a row: interior position xl, chunk rc8, sub-row
    const int xl = (lane % LR) / NC, rc8 = lane % NC, sub = lane / LR;
    const int offx = (X0 + xl) * ct8 + rc8;
    const int rdst = ((wave * RPW + sub) * HX + 1 + xl) * CT + 8 * swz(1 + xl, rc8);
    auto row_off = [&](int row) {                         // chunk offset of a halo row, -1: zero
        const int gy = edge(Y0 - 1 + row % HY, x.h, pmask & 2), gz = edge(Z0 - 1 + row / HY, x.d, pmask & 4);
        return row < ROWS && gy >= 0 && gz >= 0 ? (gz * x.h + gy) * x.w * ct8 : -1;
    };
    bf16x8 hv[NL + NS], wv[WLDS ? NW : 1];
    // every load of this thread is issued before the first LDS store, so a
    // chunk costs one memory latency, not one per element
    auto load = [&](int c0) {
        const int gpt = (ci - c0) >> 3;                   // channel groups left (chunks past it are zero)
        const bf16x8 *xc = xp + (c0 >> 3);
        #pragma unroll
        for (int k = 0; k < NL; ++k) {
            int ro = row_off((k * 4 + wave) * RPW);
            #pragma unroll
            for (int r = 1; r < RPW; ++r) {
                const int o = row_off((k * 4 + wave) * RPW + r);
                ro = sub == r ? o : ro;
            }
            hv[k] = zero;
            if (ro >= 0 && rc8 < gpt) hv[k] = xc[(unsigned)(ro + offx)];
        }
        #pragma unroll
        for (int k = 0; k < NS; ++k) {
            const int e = (int)threadIdx.x + 256 * k, row = e / (2 * NC), j = e % (2 * NC);
            const int ro = row_off(row), gx = edge(j / NC ? X0 + BX : X0 - 1, x.w, pmask & 1);
            hv[NL + k] = zero;
            if (ro >= 0 && gx >= 0 && j % NC < gpt) hv[NL + k] = xc[(unsigned)(ro + gx * ct8 + j % NC)];
        }
        if constexpr (WLDS) {
            #pragma unroll
            for (int k = 0; k < NW; ++k) {
                const int e = (int)threadIdx.x + 256 * k, c8 = e % NC, o = e / NC % (16 * NO), t = e / (16 * NO * NC);
                wv[k] = zero;
                if (e < WE && c8 < gpt)
                    wv[k] = *reinterpret_cast<const bf16x8 *>(W + (int64_t)(co0 + o) * K + t * ci + c0 + 8 * c8);
            }
        }
    };
    auto store = [&]() {
        #pragma unroll
        for (int k = 0; k < NL; ++k)
            if ((k * 4 + wave) * RPW + sub < ROWS)
                *reinterpret_cast<bf16x8 *>(&halo[rdst + k * 4 * RPW * HX * CT]) = hv[k];
        #pragma unroll
        for (int k = 0; k < NS; ++k) {
            const int e = (int)threadIdx.x + 256 * k, row = e / (2 * NC), j = e % (2 * NC);
            const int hx = j / NC ? HX - 1 : 0;
            if (e < SIDE) *reinterpret_cast<bf16x8 *>(&halo[(row * HX + hx) * CT + 8 * swz(hx, j % NC)]) = hv[NL + k];
        }
        if constexpr (WLDS)
            #pragma unroll
            for (int k = 0; k < NW; ++k) {
                const int e = (int)threadIdx.x + 256 * k, c8 = e % NC, oc = e / NC;
                if (e < WE) *reinterpret_cast<bf16x8 *>(&wl[(oc * NC + swz(oc & 15, c8)) * 8]) = wv[k];
            }
    };

    f32x4 acc[NO][NF];
    #pragma unroll
    for (int o = 0; o < NO; ++o)
        #pragma unroll
        for (int i = 0; i < NF; ++i) acc[o][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bf16 *wrow = W + (int64_t)(co0 + col) * K;

    if (WLDS) load(0);
    for (int c0 = 0; c0 < ci; c0 += CT) {
        if (!WLDS) load(c0);
        __syncthreads();                                  // previous chunk's fragment reads are done
        store();
        __syncthreads();
        if (WLDS && c0 + CT < ci) load(c0 + CT);
        const int g = min(CT, ci - c0) >> 3, lg = g == 1 ? 0 : (g == 2 ? 1 : 2), gpt = 1 << lg;
        // weights of tap t, channel group c8 of this chunk, output block o
        auto weight = [&](int t, int c8, int o) {
            if constexpr (WLDS)
                return *reinterpret_cast<const bf16x8 *>(&wl[((t * 16 * NO + 16 * o + col) * NC + swz(col, c8)) * 8]);
            else return *reinterpret_cast<const bf16x8 *>(wrow + (int64_t)16 * o * K + t * ci + c0 + 8 * c8);
        };
        if constexpr (DYR) {
            // Super-block s gives lane group grp the combination q = 4 s + grp of
            // (dz, dx, c8); combinations past the last get zero weights.
            const int Q9 = 9 * gpt, nsb = (Q9 + 3) >> 2;
            auto rows = [&](int s, int z, bf16x8 (&R)[NR]) {
                const int q = min(4 * s + grp, Q9 - 1);
                const int c8 = q & (gpt - 1), dzx = q >> lg;
                const int dz = dzx / 3, hx = col + dzx % 3;                 // offsets + 1
                const bf16 *p = &halo[((wave * ZW + z + dz) * HY * HX + hx) * CT + 8 * swz(hx, c8)];
                #pragma unroll
                for (int r = 0; r < NR; ++r) R[r] = *reinterpret_cast<const bf16x8 *>(p + r * HX * CT);
            };
            auto wts = [&](int s, bf16x8 (&A)[3][NO]) {
                const int q4 = 4 * s + grp, q = min(q4, Q9 - 1);
                const int c8 = q & (gpt - 1), dzx = q >> lg;
                const int tap0 = dzx / 3 * 9 + dzx % 3;
                #pragma unroll
                for (int d = 0; d < 3; ++d)
                    #pragma unroll
                    for (int o = 0; o < NO; ++o) {
                        const bf16x8 a = weight(tap0 + 3 * d, c8, o);
                        A[d][o] = q4 < Q9 ? a : zero;
                    }
            };
            auto mma = [&](int z, const bf16x8 (&R)[NR], const bf16x8 (&A)[3][NO]) {
                #pragma unroll
                for (int d = 0; d < 3; ++d)
                    #pragma unroll
                    for (int o = 0; o < NO; ++o)
                        #pragma unroll
                        for (int f = 0; f < BY; ++f) acc[o][z * BY + f] = mfma(A[d][o], R[f + d], acc[o][z * BY + f]);
            };
            // register sets in turn, so a plane's MFMAs never wait for the fetch
            // issued after them; the fetch past the end re-reads a valid block.
            // 8- and 16-channel chunks fetch their weights at use: the registers
            // saved let one more workgroup stay on the CU, which hides more (on the
            // 128 x 128 x 512 box 16 -> 16 channels 266 -> 254 us, 8 -> 16 177 -> 166).
            constexpr bool AHEAD = CT == 32;
            bf16x8 R0[NR], R1[NR], A0[3][NO], A1[3][NO];
            auto step = [&](int s, bf16x8 (&Rc)[NR], bf16x8 (&Rn)[NR], bf16x8 (&Ac)[3][NO], bf16x8 (&An)[3][NO]) {
                const int sn = min(s + 1, nsb - 1);
                if constexpr (AHEAD) wts(sn, An);
                else wts(s, Ac);
                if constexpr (ZW == 2) {
                    rows(s, 1, Rn);
                    mma(0, Rc, Ac);
                    rows(sn, 0, Rc);
                    mma(1, Rn, Ac);
                } else {
                    rows(sn, 0, Rn);
                    mma(0, Rc, Ac);
                }
            };
            rows(0, 0, R0);
            if constexpr (AHEAD) wts(0, A0);
            int s = 0;
            for (; s + 2 <= nsb; s += 2) {
                step(s, R0, R1, A0, A1);
                if constexpr (ZW == 2) step(s + 1, R0, R1, A1, A0);
                else step(s + 1, R1, R0, A1, A0);
            }
            if (s < nsb) step(s, R0, R1, A0, A1);
        } else {
            // K blocks of 4 (tap, 8-channel group) pairs.  The full blocks run
            // unmasked; a last partial block (27 gpt not a multiple of 4) zeroes
            // the weights of its idle lanes.
            const int G = 27 * gpt, nfull = G >> 2, rem = G & 3;
            auto fetch = [&](int q, bf16x8 (&a)[NO], bf16x8 (&b)[NF]) {
                const int tap = q >> lg, c8 = q & (gpt - 1);
                const int dz = tap / 9, dy = (tap / 3) % 3, hx = col + tap % 3;
                #pragma unroll
                for (int o = 0; o < NO; ++o) a[o] = weight(tap, c8, o);
                #pragma unroll
                for (int i = 0; i < NF; ++i)
                    b[i] = *reinterpret_cast<const bf16x8 *>(
                        &halo[(((wave * ZW + i / BY + dz) * HY + i % BY + dy) * HX + hx) * CT + 8 * swz(hx, c8)]);
            };
            auto mma = [&](const bf16x8 (&a)[NO], const bf16x8 (&b)[NF]) {
                #pragma unroll
                for (int o = 0; o < NO; ++o)
                    #pragma unroll
                    for (int i = 0; i < NF; ++i) acc[o][i] = mfma(a[o], b[i], acc[o][i]);
            };
            bf16x8 a[NO], b[NF], a1[NO], b1[NF];
            fetch(grp, a, b);
            int kb = 0;
            for (; kb + 2 <= nfull; kb += 2) {
                fetch(((kb + 1) << 2) + grp, a1, b1);
                mma(a, b);
                fetch((min(kb + 2, nfull - 1) << 2) + grp, a, b);
                mma(a1, b1);
            }
            if (kb < nfull) mma(a, b);
            if (rem) {
                const bool valid = grp < rem;
                fetch(valid ? (nfull << 2) + grp : G - 1, a, b);
                #pragma unroll
                for (int o = 0; o < NO; ++o)
                    if (!valid) a[o] = zero;
                mma(a, b);
            }
        }
    }
    #pragma unroll
    for (int o = 0; o < NO; ++o) {
        const int oc0 = co0 + 16 * o + (grp << 2);
        const f32x4 bo = bias4(bias, oc0, y, y32);
        #pragma unroll
        for (int i = 0; i < NF; ++i) {
            const int64_t pb = (((int64_t)n * x.d + Z0 + wave * ZW + i / BY) * x.h + Y0 + i % BY) * x.w + X0 + col;
            store_out(y, y32, pb, oc0, acc[o][i] + bo, relu, accumulate);
        }
    }
}

// Convolution straight from memory, for extents without whole bricks and for
// 1x1x1 layers: every wave owns NO x 16 output channels x FP x 16 consecutive
// positions and walks the K blocks in order (4 consecutive 8-channel groups of the
// tap-major, channel-minor K axis).  Its operands come from L1 and L2 (16 bytes
// per lane and fragment), whose latency a ring of D blocks in flight covers; the
// offsets of a position's taps are computed once per workgroup into an LDS
// table, and taps outside the box read past the buffer's end, which gives zero.
// Deep layers of small boxes have few positions, so the host takes few per wave
// there: 64 -> 128 channels on 4 x 8^3 positions 66 us with one block ahead and
// 64 positions per wave, 21.5 now; 48 -> 16 on 200 x 104 x 104 633, 383.
template <int NO, int FP, int D>
__global__ __launch_bounds__(256) void k_conv_direct(sg_view x, const bf16 *__restrict__ W, int co_all,
                                                     const float *__restrict__ bias, int k, int pmask, int relu,
                                                     sg_view y, sg_view y32, int accumulate)
{
    constexpr int NP = 64 * FP;                            // positions of a workgroup
    __shared__ unsigned tab[27][NP];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 15, grp = lane >> 4;
    const int P = (int)npos(x), p0 = (int)blockIdx.x * NP;
    const int co0 = blockIdx.y * 16 * NO;
    const int ci = x.c, g8 = ci >> 3, taps = k * k * k, K8 = taps * g8, nkb = (K8 + 3) >> 2;
    constexpr unsigned OUT = 0xfffffff0u;                  // beyond any buffer
    for (int e = threadIdx.x; e < NP; e += 256) {
        const bool ok = p0 + e < P;
        const Pos q = decode(x, ok ? p0 + e : 0);
        for (int t = 0; t < taps; ++t) {
            int dz, dy, dx;
            tap_offset(t, k, dz, dy, dx);
            const int64_t src = ok ? shifted(x, q, dz, dy, dx, pmask) : -1;
            tab[t][e] = src < 0 ? OUT : (unsigned)((src * x.ctot + x.coff) * 2);
        }
    }
    __syncthreads();
    typedef int i32x4 __attribute__((ext_vector_type(4)));
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
        x.p, (short)0, (int)(unsigned)((int64_t)P * x.ctot * 2), 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16 *>(W), (short)0, (int)(unsigned)((int64_t)co_all * K8 * 16), 0x00020000);
    auto ld = [](__amdgpu_buffer_rsrc_t r, unsigned off) {
        return __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
    };
    f32x4 acc[NO][FP];
    #pragma unroll
    for (int o = 0; o < NO; ++o)
        #pragma unroll
        for (int i = 0; i < FP; ++i) acc[o][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    // this lane's group of the next block to load: g = 4 kb + grp = tap g8 + c8
    int gl = grp, tap = grp / g8, c8 = grp % g8;
    const int dt = 4 / g8, dc = 4 % g8;
    const int pl = wave * 16 * FP + col;
    const unsigned wrow = (unsigned)(co0 + col) * (unsigned)K8 * 16u;
    // the ring holds 32-bit words (16-bit elements carried around the loop cost
    // a copy, and with it a wait, per trip)
    i32x4 a[D][NO], b[D][FP];
    auto load = [&](i32x4 (&av)[NO], i32x4 (&bv)[FP]) {
        const bool in = gl < K8;
        #pragma unroll
        for (int o = 0; o < NO; ++o) av[o] = ld(rw, in ? wrow + (unsigned)(16 * o * K8 + gl) * 16u : OUT);
        const int t = min(tap, taps - 1);
        #pragma unroll
        for (int i = 0; i < FP; ++i) {
            const unsigned off = tab[t][pl + 16 * i];
            bv[i] = ld(rx, in && off != OUT ? off + 16u * (unsigned)c8 : OUT);
        }
        gl += 4;
        tap += dt;
        c8 += dc;
        if (c8 >= g8) {
            c8 -= g8;
            ++tap;
        }
    };
    #pragma unroll
    for (int j = 0; j < D; ++j) load(a[j], b[j]);
    for (int kb = 0; kb < nkb; kb += D) {
        #pragma unroll
        for (int j = 0; j < D; ++j) {
            // blocks past the last hold zeros
            #pragma unroll
            for (int o = 0; o < NO; ++o)
                #pragma unroll
                for (int i = 0; i < FP; ++i)
                    acc[o][i] = mfma(__builtin_bit_cast(bf16x8, a[j][o]), __builtin_bit_cast(bf16x8, b[j][i]), acc[o][i]);
            load(a[j], b[j]);
        }
    }
    #pragma unroll
    for (int o = 0; o < NO; ++o) {
        const int oc0 = co0 + 16 * o + (grp << 2);
        const f32x4 bo = bias4(bias, oc0, y, y32);
        #pragma unroll
        for (int i = 0; i < FP; ++i)
            if (p0 + pl + 16 * i < P) store_out(y, y32, p0 + pl + 16 * i, oc0, acc[o][i] + bo, relu, accumulate);
    }
}

struct ConvArgs {
    const sg_view *x;
    const void *w;
    const float *bias;
    int co, pmask, relu;
    sg_view y, y32;
    int accumulate;
    hipStream_t st;
};

template <int NO, int BZ, int CT, bool DYR, bool WLDS>
static void launch_conv3(const ConvArgs &a)
{
    const sg_view *x = a.x;
    const int nbx = x->w / 16, nby = x->h / 4, nbz = x->d / BZ;
    hipLaunchKernelGGL((k_conv3<NO, BZ, CT, DYR, WLDS>), dim3((unsigned)((int64_t)x->n * nbx * nby * nbz), a.co / (16 * NO)),
                       dim3(256), 0, a.st, *x, (const bf16 *)a.w, a.bias, a.pmask, a.relu, a.y, a.y32, a.accumulate,
                       nbx, nby, nbz);
}

template <int NO, int FP, int D>
static void launch_direct(const ConvArgs &a, int k)
{
    const int64_t P = (int64_t)a.x->n * a.x->d * a.x->h * a.x->w;
    hipLaunchKernelGGL((k_conv_direct<NO, FP, D>), dim3((unsigned)((P + 64 * FP - 1) / (64 * FP)), a.co / (16 * NO)),
                       dim3(256), 0, a.st, *a.x, (const bf16 *)a.w, a.co, a.bias, k, a.pmask, a.relu, a.y, a.y32,
                       a.accumulate);
}

// 1x1x1 convolution with few outputs (the network head): one position per
// lane, the weight rows read as wave-uniform vectors, FP32 dot products.  The
// layer moves ~3x more bytes than it computes, so it is written for HBM.
template <int NOUT>
__global__ __launch_bounds__(256) void k_conv1_small(sg_view x, const bf16 *__restrict__ W,
                                                     const float *__restrict__ bias, int relu, sg_view y, sg_view y32,
                                                     int accumulate)
{
    const int64_t P = npos(x);
    const int ci = x.c, g8 = ci >> 3;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < P; p += (int64_t)gridDim.x * blockDim.x) {
        float acc[NOUT];
        #pragma unroll
        for (int o = 0; o < NOUT; ++o) acc[o] = bias ? bias[o] : 0.f;
        const bf16 *xr = reinterpret_cast<const bf16 *>(x.p) + p * x.ctot + x.coff;
        for (int g = 0; g < g8; ++g) {
            const bf16x8 v = *reinterpret_cast<const bf16x8 *>(xr + 8 * g);
            #pragma unroll
            for (int o = 0; o < NOUT; ++o) {
                const bf16x8 w = *reinterpret_cast<const bf16x8 *>(W + (int64_t)o * ci + 8 * g);
                #pragma unroll
                for (int j = 0; j < 8; ++j) acc[o] = __builtin_fmaf((float)w[j], (float)v[j], acc[o]);
            }
        }
        #pragma unroll
        for (int o = 0; o < NOUT; ++o) {
            float v = relu ? fmaxf(acc[o], 0.f) : acc[o];
            if (y.p && o < y.c) reinterpret_cast<bf16 *>(y.p)[p * y.ctot + y.coff + o] = (bf16)v;
            if (y32.p && o < y32.c) {
                float *out = reinterpret_cast<float *>(y32.p) + p * y32.ctot + y32.coff + o;
                *out = accumulate ? *out + v : v;
            }
        }
    }
}

// Master weights -> BF16 [co_pad][K] and the flipped transpose
// Wt[ci][tap' co8 + c] = W[c][tap ci + ci] with tap' the mirrored tap.
__global__ void k_weight_prep(const float *w32, int co, int ci, int k, bf16 *wb, bf16 *wt, int co_pad, int ci_pad)
{
    const int taps = k * k * k, K = taps * ci, co8 = (co + 7) & ~7, Kt = taps * co8;
    const int64_t n1 = (int64_t)co_pad * K, n2 = (int64_t)ci_pad * Kt;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n1 + n2; e += (int64_t)gridDim.x * blockDim.x) {
        if (e < n1) {
            const int o = (int)(e / K);
            wb[e] = (bf16)(o < co ? w32[e] : 0.f);
        } else {
            const int64_t f = e - n1;
            const int i = (int)(f / Kt), r = (int)(f % Kt);
            const int tp = r / co8, c = r % co8;
            const int tap = taps - 1 - tp;     // (dz,dy,dx) -> (-dz,-dy,-dx)
            wt[f] = (bf16)((i < ci && c < co) ? w32[(int64_t)c * K + (int64_t)tap * ci + i] : 0.f);
        }
    }
}

// ------------------------------------------------------ weight gradient
// dW[co][tap ci + c] = sum_p dy[p][co] x[p + off(tap)][c].  The contraction
// runs over positions, so both MFMA operands need 8 positions of one channel
// per lane while the tensors are channels-last.  A workgroup stages a brick of
// 256 positions as it lies in memory (16 channels, 32 bytes, per position and
// channel block): dy, and x with its one-node halo.  Fragments are then read by
// ds_read_b64_tr_b16, which transposes 4 positions x 16 channels per 16 lanes,
// so a tap is only another LDS offset: x goes to LDS once instead of once per
// tap, and nothing is transposed by 2-byte stores.  (Before, staging wrote
// every tap's rows transposed, 55 KB of LDS stores per 64 positions: 16 -> 16
// channels on 4 x 64^3 positions 247 us with the reduction, 50 now; 48 -> 16 791,
// 164; 64 -> 64 on 4 x 16^3 65, 29.)  Within a K block of 32 positions lane group g and
// read r cover brick positions 16 r + 4 g .. + 3, the same for both operands.
// Wave w owns taps w, w + 4, ...; its accumulators stay in registers over all
// bricks of its group (a contiguous run), the next brick's loads are issued
// before the current brick's MFMAs, and each group writes one partial sum per
// weight to ws[group][co_pad][K].  Extents need not be multiples of the brick
// (RAG): planes beyond the box are skipped; positions beyond it in x or y carry
// dy = 0, and their x rows are read from a block of zeros, since a tap reaches
// back into the box from there and 0 x Inf would enter a sum that the value is
// no part of (16 -> 16 channels on 61 x 67 x 71 positions 22.9 us without, 25.2 so;
// clearing the fragments instead 25.0 there, but 64 -> 64 146 against 127).
constexpr int WP = 256;              // positions per brick
constexpr int WTAPS = 7;             // taps per wave (27 taps over 4 waves)

typedef short s16x4 __attribute__((ext_vector_type(4)));

// 8 positions of channel (lane & 15): two transposed reads of 4 positions
__device__ inline bf16x8 read_tr(const bf16 *r0, const bf16 *r1)
{
    typedef __attribute__((address_space(3))) s16x4 *lp;
    const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)r0);
    const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)r1);
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    const s16x8 v = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
}

// NOB x NCB blocks of 16 output x 16 input channels per workgroup; BX x BY x
// BZ = 256 positions per brick (27 taps); K1: a 1x1x1 layer, whose bricks are
// 256 consecutive positions and whose waves share the K blocks.
template <int NOB, int NCB, int BX, int BY, int BZ, bool K1, bool RAG>
__global__ __launch_bounds__(256, NOB * NCB == 1 ? 3 : 2) void k_conv_bwd_w(sg_view x, sg_view dy, int pmask, int co_pad, int nbx, int nby,
                                                    int nbz, int64_t nbricks, float *ws, float *wsb)
{
    static_assert(BX * BY * BZ == WP && 16 % BX == 0, "brick shape");
    constexpr int HXW = K1 ? BX : BX + 2, HYW = K1 ? BY : BY + 2, HZW = K1 ? BZ : BZ + 2, HPW = HXW * HYW * HZW;
    constexpr int XE = 2 * NCB * HPW, XN = (XE + 255) / 256;     // 16-byte chunks of x and their rounds
    constexpr int DE = 2 * NOB * WP, DN = DE / 256;
    constexpr int NT = K1 ? 1 : WTAPS;
    __shared__ __attribute__((aligned(16))) bf16 xs[NCB][HPW][16];
    __shared__ __attribute__((aligned(16))) bf16 dys[NOB][WP][16];
    static_assert(!RAG || !K1, "1x1x1 layers have no position beyond the last");
    constexpr int ZE = RAG ? 16 * (2 + HXW * (2 + HYW * 2)) + 8 : 8;     // a row of zeros at every tap's offset
    __shared__ __attribute__((aligned(16))) bf16 zeros[ZE];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 15, grp = lane >> 4;
    const int ci = x.c, taps = K1 ? 1 : 27, K = taps * ci;
    const int co0 = blockIdx.y * 16 * NOB, c0 = blockIdx.z * 16 * NCB;
    const bf16 *xp = reinterpret_cast<const bf16 *>(x.p) + x.coff + c0;
    const bf16 *dp = reinterpret_cast<const bf16 *>(dy.p) + dy.coff + co0;
    const bf16x8 zero = {};
    const int64_t P = npos(x);

    bf16x8 xv[XN], dv[DN];
    // position of brick b: origin, and (27 taps) its batch item
    auto load = [&](int64_t b) {
        int X0 = 0, Y0 = 0, Z0 = 0, n = 0;
        if constexpr (!K1) {
            int64_t q = b;
            X0 = (int)(q % nbx) * BX; q /= nbx;
            Y0 = (int)(q % nby) * BY; q /= nby;
            Z0 = (int)(q % nbz) * BZ;
            n = (int)(q / nbz);
        }
        #pragma unroll
        for (int k = 0; k < XN; ++k) {
            const int e = tid + 256 * k;
            const int hp = e / (2 * NCB), c8 = e % (2 * NCB);
            bool ok = e < XE && c0 + 8 * c8 < ci;
            int64_t src;
            if constexpr (K1) {
                src = b * WP + hp;
                ok = ok && src < P;
            } else {
                int gx = X0 - 1 + hp % HXW, gy = Y0 - 1 + (hp / HXW) % HYW, gz = Z0 - 1 + hp / (HXW * HYW);
                // one step beyond the box wraps or is zero, further is not read
                if (gx < 0 || gx >= x.w) { ok = ok && (pmask & 1) && gx <= x.w; gx = gx < 0 ? x.w - 1 : 0; }
                if (gy < 0 || gy >= x.h) { ok = ok && (pmask & 2) && gy <= x.h; gy = gy < 0 ? x.h - 1 : 0; }
                if (gz < 0 || gz >= x.d) { ok = ok && (pmask & 4) && gz <= x.d; gz = gz < 0 ? x.d - 1 : 0; }
                src = (((int64_t)n * x.d + gz) * x.h + gy) * x.w + gx;
            }
            xv[k] = zero;
            if (ok) xv[k] = *reinterpret_cast<const bf16x8 *>(xp + src * x.ctot + 8 * c8);
        }
        #pragma unroll
        for (int k = 0; k < DN; ++k) {
            const int e = tid + 256 * k;
            const int p = e / (2 * NOB), c8 = e % (2 * NOB);
            bool ok = co0 + 8 * c8 < dy.c;
            int64_t src;
            if constexpr (K1) {
                src = b * WP + p;
                ok = ok && src < P;
            } else {
                const int gx = X0 + p % BX, gy = Y0 + (p / BX) % BY, gz = Z0 + p / (BX * BY);
                ok = ok && gx < x.w && gy < x.h && gz < x.d;
                src = (((int64_t)n * x.d + gz) * x.h + gy) * x.w + gx;
            }
            dv[k] = zero;
            if (ok) {
                dv[k] = *reinterpret_cast<const bf16x8 *>(dp + src * dy.ctot + 8 * c8);
                #pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (co0 + 8 * c8 + j >= dy.c) dv[k][j] = (bf16)0.f;
            }
        }
    };
    auto store = [&]() {
        #pragma unroll
        for (int k = 0; k < XN; ++k) {
            const int e = tid + 256 * k, hp = e / (2 * NCB), c8 = e % (2 * NCB);
            if (e < XE) *reinterpret_cast<bf16x8 *>(&xs[c8 >> 1][hp][8 * (c8 & 1)]) = xv[k];
        }
        #pragma unroll
        for (int k = 0; k < DN; ++k) {
            const int e = tid + 256 * k, p = e / (2 * NOB), c8 = e % (2 * NOB);
            *reinterpret_cast<bf16x8 *>(&dys[c8 >> 1][p][8 * (c8 & 1)]) = dv[k];
        }
    };

    f32x4 acc[NT][NOB][NCB], accb[NOB];
    #pragma unroll
    for (int t = 0; t < NT; ++t)
        #pragma unroll
        for (int o = 0; o < NOB; ++o)
            #pragma unroll
            for (int c = 0; c < NCB; ++c) acc[t][o][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    #pragma unroll
    for (int o = 0; o < NOB; ++o) accb[o] = f32x4{0.f, 0.f, 0.f, 0.f};
    // the bias gradient is the weight gradient of an input channel of ones;
    // the wave with the fewest taps (K1: every wave, for its K blocks) computes
    // it in the first input-channel block
    const bool bias_wave = wsb && blockIdx.z == 0 && (K1 || wave == 3);
    bf16x8 ones;
    #pragma unroll
    for (int j = 0; j < 8; ++j) ones[j] = (bf16)1.f;
    // a lane's row of a transposed read: position 4 grp + (lane & 15) / 4, channels 4 (lane & 3) ..
    const int lp = 4 * grp + (col >> 2), lc = 4 * (col & 3);
    // LDS offset (elements) of this lane's row at K block 0 for read r, and per tap
    auto hidx = [](int p) { return p % BX + HXW * ((p / BX) % BY + HYW * (p / (BX * BY))); };
    const int xo0 = hidx(lp) * 16 + lc, xo1 = hidx(lp + 16) * 16 + lc;
    int to[NT];
    #pragma unroll
    for (int i = 0; i < NT; ++i) {
        const int t = min(wave + 4 * i, 26);
        to[i] = K1 ? 0 : 16 * (t % 3 + HXW * ((t / 3) % 3 + HYW * (t / 9)));
    }

    if constexpr (RAG)
        for (int e = 8 * tid; e < ZE; e += 8 * 256) *reinterpret_cast<bf16x8 *>(&zeros[e]) = zero;

    const int64_t b0 = nbricks * blockIdx.x / gridDim.x, b1 = nbricks * (blockIdx.x + 1) / gridDim.x;
    if (b0 < b1) load(b0);
    for (int64_t b = b0; b < b1; ++b) {
        __syncthreads();                                   // the previous brick's fragment reads are done
        store();
        __syncthreads();
        // planes of this brick inside the box (K blocks beyond it are skipped)
        const int nz = K1 ? BZ : min(BZ, x.d - (int)(b / ((int64_t)nbx * nby) % nbz) * BZ);
        // positions of this lane's rows inside the box in x; the row of its first position
        const bool in_x = (int)(b % nbx) * BX + lp % BX < x.w;
        const int Y0 = (int)(b / nbx % nby) * BY;
        if (b + 1 < b1) load(b + 1);
        #pragma unroll
        for (int ks = 0; ks < WP / 32; ++ks) {
            constexpr int KZP = BX * BY / 32;              // K blocks per plane
            if (K1 ? (ks & 3) != wave : ks / KZP >= nz) continue;
            const int hk = 16 * (K1 ? 32 * ks : BX == 16 ? HXW * ((2 * ks) % BY + HYW * (ks / KZP))
                                             : HXW * ((32 / BX * ks) % BY + HYW * (ks / KZP)));
            bf16x8 a[NOB];
            #pragma unroll
            for (int o = 0; o < NOB; ++o)
                a[o] = read_tr(&dys[o][32 * ks + lp][lc], &dys[o][32 * ks + 16 + lp][lc]);
            // the lane's rows (a position, 4 channels) at the first tap
            const bf16 *r0[NCB], *r1[NCB];
            #pragma unroll
            for (int c = 0; c < NCB; ++c) {
                r0[c] = &xs[c][0][0] + hk + xo0;
                r1[c] = &xs[c][0][0] + hk + xo1;
                if constexpr (RAG) {
                    if (!in_x || Y0 + (32 * ks + lp) / BX % BY >= x.h) r0[c] = zeros;
                    if (!in_x || Y0 + (32 * ks + 16 + lp) / BX % BY >= x.h) r1[c] = zeros;
                }
            }
            #pragma unroll
            for (int i = 0; i < NT; ++i) {
                if (!K1 && i == NT - 1 && wave == 3) continue;     // 27 taps: wave 3 has six
                #pragma unroll
                for (int c = 0; c < NCB; ++c) {
                    const bf16x8 bb = read_tr(r0[c] + to[i], r1[c] + to[i]);
                    #pragma unroll
                    for (int o = 0; o < NOB; ++o) acc[i][o][c] = mfma(a[o], bb, acc[i][o][c]);
                }
            }
            if (bias_wave)
                #pragma unroll
                for (int o = 0; o < NOB; ++o) accb[o] = mfma(a[o], ones, accb[o]);
        }
    }
    if constexpr (K1) {
        // the four waves' sums over their K blocks, added in order through LDS
        float *red = reinterpret_cast<float *>(&xs[0][0][0]);
        constexpr int PER = 4 * NOB * (NCB + 1);
        static_assert(sizeof(float) * 3 * 64 * PER <= sizeof(xs), "the waves' sums must fit the x stage");
        __syncthreads();
        if (wave > 0) {
            float *r = red + ((wave - 1) * 64 + lane) * PER;
            #pragma unroll
            for (int o = 0; o < NOB; ++o)
                #pragma unroll
                for (int j = 0; j < 4; ++j) {
                    #pragma unroll
                    for (int c = 0; c < NCB; ++c) r[(o * 4 + j) * (NCB + 1) + c] = acc[0][o][c][j];
                    r[(o * 4 + j) * (NCB + 1) + NCB] = accb[o][j];
                }
        }
        __syncthreads();
        if (wave > 0) return;
        for (int w = 0; w < 3; ++w) {
            const float *r = red + (w * 64 + lane) * PER;
            #pragma unroll
            for (int o = 0; o < NOB; ++o)
                #pragma unroll
                for (int j = 0; j < 4; ++j) {
                    #pragma unroll
                    for (int c = 0; c < NCB; ++c) acc[0][o][c][j] += r[(o * 4 + j) * (NCB + 1) + c];
                    accb[o][j] += r[(o * 4 + j) * (NCB + 1) + NCB];
                }
        }
    }
    if (bias_wave && col == 0)
        #pragma unroll
        for (int o = 0; o < NOB; ++o)
            #pragma unroll
            for (int j = 0; j < 4; ++j) wsb[(int64_t)blockIdx.x * co_pad + co0 + 16 * o + 4 * grp + j] = accb[o][j];
    // D[4 grp + j][col]: output channel co0 + 16 o + 4 grp + j, input channel c0 + 16 c + col
    #pragma unroll
    for (int i = 0; i < NT; ++i) {
        const int t = wave + 4 * i;
        if (t >= taps) continue;
        #pragma unroll
        for (int c = 0; c < NCB; ++c) {
            const int ic = c0 + 16 * c + col;
            if (ic >= ci) continue;
            #pragma unroll
            for (int o = 0; o < NOB; ++o)
                #pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int oc = co0 + 16 * o + 4 * grp + j;
                    ws[((int64_t)blockIdx.x * co_pad + oc) * K + (int64_t)t * ci + ic] = acc[i][o][c][j];
                }
        }
    }
}

// Fixed-order sum of the per-group partials of the weights (n values, group
// stride gs) and the bias (nb values, group stride gsb): 32 outputs x 8 slices of
// the groups per workgroup, the slices added in order through LDS.  A chain of
// load latencies: U of them in flight where a slice has that many groups (16 ->
// 16 channels on 4 x 64^3 positions, 768 groups: 15.6 -> 12 us).
__global__ __launch_bounds__(256) void k_reduce_groups(const float *__restrict__ ws, int64_t gs, int64_t n,
                                                       const float *__restrict__ wsb, int gsb, int nb, int groups,
                                                       float *dw, float *db)
{
    constexpr int U = 16;
    __shared__ float sh[8][32];
    const int l = threadIdx.x & 31, s = threadIdx.x >> 5;
    const int64_t e = (int64_t)blockIdx.x * 32 + l;
    const bool bias = e >= n;
    const float *src = bias ? wsb + (e - n) : ws + e;
    const int64_t st = bias ? gsb : gs;
    float acc = 0.f;
    if (e < n + nb) {
        int g = s;
        for (; g + 8 * (U - 1) < groups; g += 8 * U) {     // U loads in flight, added in order
            float v[U];
            #pragma unroll
            for (int u = 0; u < U; ++u) v[u] = src[(g + 8 * u) * st];
            __builtin_amdgcn_sched_barrier(0);
            #pragma unroll
            for (int u = 0; u < U; ++u) acc += v[u];
        }
        #pragma unroll 4
        for (; g < groups; g += 8) acc += src[g * st];
    }
    sh[s][l] = acc;
    __syncthreads();
    if (s == 0 && e < n + nb) {
        float v = sh[0][l];
        #pragma unroll
        for (int k = 1; k < 8; ++k) v += sh[k][l];
        if (bias) db[e - n] = v;
        else dw[e] = v;
    }
}

// ------------------------------------------------------- element-wise
__global__ void k_relu_bwd_cast(sg_view dx, sg_view y, sg_view dyb)
{
    const int64_t n = npos(dx) * dx.c;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t p = e / dx.c;
        const int c = (int)(e % dx.c);
        float g = reinterpret_cast<const float *>(dx.p)[p * dx.ctot + dx.coff + c];
        if (y.p && !((float)reinterpret_cast<const bf16 *>(y.p)[p * y.ctot + y.coff + c] > 0.f)) g = 0.f;
        reinterpret_cast<bf16 *>(dyb.p)[p * dyb.ctot + dyb.coff + c] = (bf16)g;
    }
}

// The same for channel-aligned views, V = 8 or 4 channels per thread and 32-bit
// indices (the host checks both).  Bound by its 8 bytes per value: a 64-bit
// division and accesses of 2 and 4 bytes per value took 44 us on 4 x 64^3 x 16
// values, where the traffic takes 26 at the copy rate.
template <int V>
__global__ void k_relu_bwd_castv(sg_view dx, sg_view y, sg_view dyb)
{
    typedef bf16 bv __attribute__((ext_vector_type(V)));
    const unsigned gv = (unsigned)dx.c / V, n = (unsigned)npos(dx) * gv;
    for (unsigned e = blockIdx.x * blockDim.x + threadIdx.x; e < n; e += gridDim.x * blockDim.x) {
        const unsigned p = e / gv, c = (e - p * gv) * V;
        const f32x4 *src = reinterpret_cast<const f32x4 *>(reinterpret_cast<const float *>(dx.p) + (int64_t)p * dx.ctot +
                                                           dx.coff + c);
        f32x4 g[V / 4];
        #pragma unroll
        for (int k = 0; k < V / 4; ++k) g[k] = src[k];
        if (y.p) {
            const bv v = *reinterpret_cast<const bv *>(reinterpret_cast<const bf16 *>(y.p) + (int64_t)p * y.ctot + y.coff + c);
            #pragma unroll
            for (int j = 0; j < V; ++j) g[j / 4][j % 4] = (float)v[j] > 0.f ? g[j / 4][j % 4] : 0.f;
        }
        bv o;
        #pragma unroll
        for (int j = 0; j < V; ++j) o[j] = (bf16)g[j / 4][j % 4];
        *reinterpret_cast<bv *>(reinterpret_cast<bf16 *>(dyb.p) + (int64_t)p * dyb.ctot + dyb.coff + c) = o;
    }
}

__device__ inline int64_t flat(const sg_view &v, int n, int z, int y, int x)
{
    return (((int64_t)n * v.d + z) * v.h + y) * v.w + x;
}

__global__ void k_pool2_fwd(sg_view x, sg_view y)
{
    const int64_t n = npos(y) * y.c;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t p = e / y.c;
        const int c = (int)(e % y.c);
        const Pos q = decode(y, p);
        float s = 0.f;
        for (int dz = 0; dz < 2; ++dz)
            for (int dy = 0; dy < 2; ++dy)
                for (int dx = 0; dx < 2; ++dx)
                    s += (float)reinterpret_cast<const bf16 *>(x.p)[flat(x, q.n, 2 * q.z + dz, 2 * q.y + dy, 2 * q.x + dx) * x.ctot + x.coff + c];
        reinterpret_cast<bf16 *>(y.p)[p * y.ctot + y.coff + c] = (bf16)(0.125f * s);
    }
}

__global__ void k_pool2_bwd(sg_view dy, sg_view dx, int accumulate)
{
    const int64_t n = npos(dx) * dx.c;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t p = e / dx.c;
        const int c = (int)(e % dx.c);
        const Pos q = decode(dx, p);
        const float g = 0.125f * reinterpret_cast<const float *>(dy.p)[flat(dy, q.n, q.z >> 1, q.y >> 1, q.x >> 1) * dy.ctot + dy.coff + c];
        float *o = reinterpret_cast<float *>(dx.p) + p * dx.ctot + dx.coff + c;
        *o = accumulate ? *o + g : g;
    }
}

__global__ void k_up2_fwd(sg_view x, sg_view y)
{
    const int64_t n = npos(y) * y.c;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t p = e / y.c;
        const int c = (int)(e % y.c);
        const Pos q = decode(y, p);
        reinterpret_cast<bf16 *>(y.p)[p * y.ctot + y.coff + c] =
            reinterpret_cast<const bf16 *>(x.p)[flat(x, q.n, q.z >> 1, q.y >> 1, q.x >> 1) * x.ctot + x.coff + c];
    }
}

// 8-channel (16-byte) forms of the two sampling layers for channel-aligned views.
// One thread per coarse position and 8-channel group: the coarse chunk is read
// once and written to the 8 fine positions it covers.  Indices are 32-bit
// (the host checks that the coarse element count fits).
__global__ void k_up2_fwd8(sg_view x, sg_view y)
{
    const unsigned g8 = (unsigned)y.c >> 3;
    const unsigned n = (unsigned)npos(x) * g8;
    for (unsigned e = blockIdx.x * blockDim.x + threadIdx.x; e < n; e += gridDim.x * blockDim.x) {
        const unsigned p = e / g8, c = (e - p * g8) << 3;
        const unsigned px = p % (unsigned)x.w, t1 = p / (unsigned)x.w;
        const unsigned py = t1 % (unsigned)x.h, t2 = t1 / (unsigned)x.h;
        const unsigned pz = t2 % (unsigned)x.d, nb = t2 / (unsigned)x.d;
        const bf16x8 v = *reinterpret_cast<const bf16x8 *>(reinterpret_cast<const bf16 *>(x.p) +
                                                           (int64_t)p * x.ctot + x.coff + c);
        bf16 *yb = reinterpret_cast<bf16 *>(y.p) + y.coff + c;
        #pragma unroll
        for (int dz = 0; dz < 2; ++dz)
            #pragma unroll
            for (int dy = 0; dy < 2; ++dy) {
                const int64_t row = (((int64_t)nb * y.d + 2 * pz + dz) * y.h + 2 * py + dy) * y.w + 2 * px;
                *reinterpret_cast<bf16x8 *>(yb + row * y.ctot) = v;
                *reinterpret_cast<bf16x8 *>(yb + (row + 1) * y.ctot) = v;
            }
    }
}

// Upsampling into a concatenation: y's first x.c channels are the nearest 2x
// upsampling of x, the remaining ones a copy of `skip` (same positions as y).
// One thread per fine position and 8-channel group of y, so that a position's
// whole row of y is written by adjacent lanes: full-line writes even where y
// interleaves the two parts per position.  32-bit indices (host-checked).
__global__ void k_up2_cat8(sg_view x, sg_view skip, sg_view y)
{
    const unsigned g8 = (unsigned)y.c >> 3, gx = (unsigned)x.c >> 3;
    const unsigned n = (unsigned)npos(y) * g8;
    for (unsigned e = blockIdx.x * blockDim.x + threadIdx.x; e < n; e += gridDim.x * blockDim.x) {
        const unsigned p = e / g8, g = e - p * g8;
        bf16x8 v;
        if (g < gx) {
            const unsigned fx = p % (unsigned)y.w, t1 = p / (unsigned)y.w;
            const unsigned fy = t1 % (unsigned)y.h, t2 = t1 / (unsigned)y.h;
            const unsigned fz = t2 % (unsigned)y.d, nb = t2 / (unsigned)y.d;
            const int64_t q = (((int64_t)nb * x.d + (fz >> 1)) * x.h + (fy >> 1)) * x.w + (fx >> 1);
            v = *reinterpret_cast<const bf16x8 *>(reinterpret_cast<const bf16 *>(x.p) + q * x.ctot + x.coff + 8 * g);
        } else {
            v = *reinterpret_cast<const bf16x8 *>(reinterpret_cast<const bf16 *>(skip.p) + (int64_t)p * skip.ctot +
                                                  skip.coff + 8 * (g - gx));
        }
        *reinterpret_cast<bf16x8 *>(reinterpret_cast<bf16 *>(y.p) + (int64_t)p * y.ctot + y.coff + 8 * g) = v;
    }
}

// One thread per coarse position and 8-channel group; 32-bit indices (the
// host checks that the coarse element count fits).
__global__ void k_pool2_fwd8(sg_view x, sg_view y)
{
    const unsigned g8 = (unsigned)y.c >> 3;
    const unsigned n = (unsigned)npos(y) * g8;
    for (unsigned e = blockIdx.x * blockDim.x + threadIdx.x; e < n; e += gridDim.x * blockDim.x) {
        const unsigned p = e / g8, c = (e - p * g8) << 3;
        const unsigned px = p % (unsigned)y.w, t1 = p / (unsigned)y.w;
        const unsigned py = t1 % (unsigned)y.h, t2 = t1 / (unsigned)y.h;
        const unsigned pz = t2 % (unsigned)y.d, nb = t2 / (unsigned)y.d;
        float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        #pragma unroll
        for (int dz = 0; dz < 2; ++dz)
            #pragma unroll
            for (int dy = 0; dy < 2; ++dy)
                #pragma unroll
                for (int dx = 0; dx < 2; ++dx) {
                    const int64_t q = (((int64_t)nb * x.d + 2 * pz + dz) * x.h + 2 * py + dy) * x.w + 2 * px + dx;
                    const bf16x8 v = *reinterpret_cast<const bf16x8 *>(reinterpret_cast<const bf16 *>(x.p) +
                                                                       q * x.ctot + x.coff + c);
                    #pragma unroll
                    for (int j = 0; j < 8; ++j) s[j] += (float)v[j];
                }
        bf16x8 o;
        #pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = (bf16)(0.125f * s[j]);
        *reinterpret_cast<bf16x8 *>(reinterpret_cast<bf16 *>(y.p) + (int64_t)p * y.ctot + y.coff + c) = o;
    }
}

__global__ void k_up2_bwd(sg_view dy, sg_view dx, int accumulate)
{
    const int64_t n = npos(dx) * dx.c;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t p = e / dx.c;
        const int c = (int)(e % dx.c);
        const Pos q = decode(dx, p);
        float s = 0.f;
        for (int dz = 0; dz < 2; ++dz)
            for (int dyy = 0; dyy < 2; ++dyy)
                for (int dxx = 0; dxx < 2; ++dxx)
                    s += reinterpret_cast<const float *>(dy.p)[flat(dy, q.n, 2 * q.z + dz, 2 * q.y + dyy, 2 * q.x + dxx) * dy.ctot + dy.coff + c];
        float *o = reinterpret_cast<float *>(dx.p) + p * dx.ctot + dx.coff + c;
        *o = accumulate ? *o + s : s;
    }
}

// 4-channel (16-byte) forms of the two adjoints for channel-aligned FP32 views:
// one thread per coarse position and 4-channel group reads (pooling) or writes
// (upsampling) its coarse value once; the fine values are summed in the same
// order.  Bound by their traffic.
__global__ void k_pool2_bwd4(sg_view dy, sg_view dx, int accumulate)
{
    const unsigned g4 = (unsigned)dy.c >> 2, n = (unsigned)npos(dy) * g4;
    for (unsigned e = blockIdx.x * blockDim.x + threadIdx.x; e < n; e += gridDim.x * blockDim.x) {
        const unsigned p = e / g4, c = (e - p * g4) << 2;
        const unsigned px = p % (unsigned)dy.w, t1 = p / (unsigned)dy.w;
        const unsigned py = t1 % (unsigned)dy.h, t2 = t1 / (unsigned)dy.h;
        const unsigned pz = t2 % (unsigned)dy.d, nb = t2 / (unsigned)dy.d;
        const f32x4 g = 0.125f * *reinterpret_cast<const f32x4 *>(reinterpret_cast<const float *>(dy.p) +
                                                                  (int64_t)p * dy.ctot + dy.coff + c);
        float *base = reinterpret_cast<float *>(dx.p) + dx.coff + c;
        f32x4 *o[8], old[8];
        #pragma unroll
        for (int k = 0; k < 8; ++k) {
            o[k] = reinterpret_cast<f32x4 *>(
                base + flat(dx, nb, 2 * pz + (k >> 2), 2 * py + ((k >> 1) & 1), 2 * px + (k & 1)) * dx.ctot);
            if (accumulate) old[k] = *o[k];
        }
        #pragma unroll
        for (int k = 0; k < 8; ++k) *o[k] = accumulate ? old[k] + g : g;
    }
}

__global__ void k_up2_bwd4(sg_view dy, sg_view dx, int accumulate)
{
    const unsigned g4 = (unsigned)dx.c >> 2, n = (unsigned)npos(dx) * g4;
    for (unsigned e = blockIdx.x * blockDim.x + threadIdx.x; e < n; e += gridDim.x * blockDim.x) {
        const unsigned p = e / g4, c = (e - p * g4) << 2;
        const unsigned px = p % (unsigned)dx.w, t1 = p / (unsigned)dx.w;
        const unsigned py = t1 % (unsigned)dx.h, t2 = t1 / (unsigned)dx.h;
        const unsigned pz = t2 % (unsigned)dx.d, nb = t2 / (unsigned)dx.d;
        const float *base = reinterpret_cast<const float *>(dy.p) + dy.coff + c;
        f32x4 v[8], s = {0.f, 0.f, 0.f, 0.f};
        #pragma unroll
        for (int k = 0; k < 8; ++k)
            v[k] = *reinterpret_cast<const f32x4 *>(
                base + flat(dy, nb, 2 * pz + (k >> 2), 2 * py + ((k >> 1) & 1), 2 * px + (k & 1)) * dy.ctot);
        #pragma unroll
        for (int k = 0; k < 8; ++k) s += v[k];
        f32x4 *o = reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(dx.p) + (int64_t)p * dx.ctot + dx.coff + c);
        *o = accumulate ? *o + s : s;
    }
}

// MSE: per-workgroup partial sums (fixed order) then one wavefront.  256
// workgroups (the caller's array holds 256 partial sums) of 1024 lanes, so that
// the memory latency is covered; V4: 4 contiguous, aligned channels per lane
// (4 x 64^3 x 4 values 40 us with 256 lanes and a 64-bit division per value).
template <bool V4>
__global__ __launch_bounds__(1024) void k_mse(sg_view out, sg_view tgt, sg_view grad, double *partial)
{
    __shared__ double sh[1024];
    const int64_t P = npos(out), n = P * out.c;
    const double inv = 1.0 / (double)n;
    double s = 0.0;
    if constexpr (V4) {
        for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < P; p += (int64_t)gridDim.x * blockDim.x) {
            auto at = [&](const sg_view &v) {
                return reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(v.p) + p * v.ctot + v.coff);
            };
            const f32x4 d = *at(out) - *at(tgt);
            f32x4 g;
            #pragma unroll
            for (int j = 0; j < 4; ++j) {
                g[j] = (float)(2.0 * d[j] * inv);
                s += (double)d[j] * d[j];
            }
            *at(grad) = g;
        }
    } else {
        for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
            const int64_t p = e / out.c;
            const int c = (int)(e % out.c);
            const float d = reinterpret_cast<const float *>(out.p)[p * out.ctot + out.coff + c] -
                            reinterpret_cast<const float *>(tgt.p)[p * tgt.ctot + tgt.coff + c];
            reinterpret_cast<float *>(grad.p)[p * grad.ctot + grad.coff + c] = (float)(2.0 * d * inv);
            s += (double)d * d;
        }
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int st = 512; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) sh[threadIdx.x] += sh[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = sh[0] * inv;
}

// Sum of n partial sums by one wavefront, in a fixed order.
__global__ __launch_bounds__(64) void k_sum_partials(const double *partial, int n, double *out)
{
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 64) s += partial[i];
    #pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
    if (threadIdx.x == 0) *out = s;
}

__global__ void k_adam(float *w, const float *g, float *m, float *v, int64_t n, float lr, float b1, float b2, float eps,
                       float c1, float c2)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const float gi = g[e];
        const float mi = b1 * m[e] + (1.f - b1) * gi;
        const float vi = b2 * v[e] + (1.f - b2) * gi * gi;
        m[e] = mi;
        v[e] = vi;
        w[e] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
    }
}

struct Scale { float s[8]; };

__global__ void k_pack(const float *f, int nf, int nx, int ny, int nz, int x0, int y0, int z0, sg_view y, sg_view y32, int b,
                       Scale sc)
{
    const int64_t per = (int64_t)y.d * y.h * y.w;
    const int64_t n = per * y.c;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t p = e / y.c;
        const int c = (int)(e % y.c);
        const int x = (int)(p % y.w), yy = (int)((p / y.w) % y.h), z = (int)(p / ((int64_t)y.w * y.h));
        float v = 0.f;
        if (c < nf) {
            const int gx = (x0 + x) % nx, gy = (y0 + yy) % ny, gz = (z0 + z) % nz;
            v = f[(int64_t)c * nx * ny * nz + gx + (int64_t)nx * (gy + (int64_t)ny * gz)] / sc.s[c];
        }
        const int64_t pp = (int64_t)b * per + p;
        reinterpret_cast<bf16 *>(y.p)[pp * y.ctot + y.coff + c] = (bf16)v;
        if (y32.p && c < y32.c) reinterpret_cast<float *>(y32.p)[pp * y32.ctot + y32.coff + c] = v;
    }
}

// Position-per-lane form of k_pack for an 8-channel BF16 view (the network
// input): the nf planar fields are read coalesced, one 16-byte BF16 row and
// (optionally) the FP32 row are written per position.
__global__ void k_pack8(const float *f, int nf, int nx, int ny, int nz, int x0, int y0, int z0, sg_view y, sg_view y32,
                        int b, Scale sc)
{
    const int64_t per = (int64_t)y.d * y.h * y.w;
    const int64_t nxyz = (int64_t)nx * ny * nz;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < per; p += (int64_t)gridDim.x * blockDim.x) {
        const int x = (int)(p % y.w), yy = (int)((p / y.w) % y.h), z = (int)(p / ((int64_t)y.w * y.h));
        const int gx = (x0 + x) % nx, gy = (y0 + yy) % ny, gz = (z0 + z) % nz;
        const int64_t src = gx + (int64_t)nx * (gy + (int64_t)ny * gz);
        float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int c = 0; c < nf; ++c) v[c] = f[(int64_t)c * nxyz + src] / sc.s[c];
        bf16x8 o;
        #pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = (bf16)v[j];
        const int64_t pp = (int64_t)b * per + p;
        *reinterpret_cast<bf16x8 *>(reinterpret_cast<bf16 *>(y.p) + pp * y.ctot + y.coff) = o;
        if (y32.p)
            for (int c = 0; c < y32.c; ++c) reinterpret_cast<float *>(y32.p)[pp * y32.ctot + y32.coff + c] = v[c];
    }
}

__global__ void k_unpack(sg_view x, int b, float *f, int nf, Scale sc)
{
    const int64_t per = (int64_t)x.d * x.h * x.w;
    const int64_t n = per * nf;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const int c = (int)(e / per);
        const int64_t p = e % per;
        f[e] = reinterpret_cast<const float *>(x.p)[((int64_t)b * per + p) * x.ctot + x.coff + c] * sc.s[c];
    }
}

__global__ void k_lift(const float *pred, int64_t n, const float *pR, const float *pB, float cs2R, float cs2B,
                       float p_in, double *out)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const float v = fminf(1.f, fmaxf(-1.f, pred[e]));
        const float p = pR ? pR[e] * cs2R + pB[e] * cs2B : p_in;
        out[e] = (double)(0.5f * p * (1.f + v) / cs2R);
        out[n + e] = (double)(0.5f * p * (1.f - v) / cs2B);
        out[2 * n + e] = (double)pred[n + e];
        out[3 * n + e] = (double)pred[2 * n + e];
        out[4 * n + e] = (double)pred[3 * n + e];
    }
}

inline unsigned grid_for(int64_t n, int block = 256)
{
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + block - 1) / block, 65536));
}

inline bool ok_view(const sg_view *v) { return v && v->p && v->n > 0 && v->d > 0 && v->h > 0 && v->w > 0 && v->c > 0 && v->coff >= 0 && v->coff + v->c <= v->ctot; }
inline bool mfma_view(const sg_view *v) { return ok_view(v) && v->c % 8 == 0 && v->ctot % 8 == 0 && v->coff % 8 == 0; }
// v's channel slice starts on a 16-byte boundary at every position and is a
// whole number of `per` channels (4 FP32 or 8 BF16 values: 16 bytes) long.
inline bool vec_view(const sg_view *v, int per)
{
    return v->c % per == 0 && v->ctot % per == 0 && v->coff % per == 0 && ((uintptr_t)v->p & 15) == 0;
}
inline bool same_pos(const sg_view *a, const sg_view *b) { return a->n == b->n && a->d == b->d && a->h == b->h && a->w == b->w; }

int status() { return hipGetLastError() == hipSuccess ? SG_OK : SG_EDEVICE; }

// Scratch of the no-allocation weight gradient: a file-scope device array,
// one copy per GPU, held until the process ends.  Host code never passes the
// array's name to a kernel (on the host it is only a stand-in for the
// symbol): the device address of each GPU's copy is looked up once, with
// that GPU current, and kept.
static __device__ __align__(256) float scratch[SG_NOALLOC_SCRATCH_BYTES / sizeof(float)];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float *g_scratch_ptr[kMaxDevices] = {};

int scratch_on_current_device(float **out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SG_EDEVICE;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return SG_EDEVICE;
        g_scratch_ptr[dev] = static_cast<float *>(p);
    }
    *out = g_scratch_ptr[dev];
    return SG_OK;
}

// Workspace of the weight gradient, as the interface states it (callers size
// their buffers by it, and sg_conv3d_bwd_weight_noalloc accepts what fits its
// scratch): partial sums of up to max_groups position groups and some slack.
struct BwdPlan { int max_groups, co_pad, K; int64_t ws_floats, bias_off; };

static BwdPlan bwd_plan(const sg_view *dy, int ci, int k)
{
    BwdPlan b;
    b.co_pad = (dy->c + 15) & ~15;
    b.K = k * k * k * ci;
    const int64_t P = (int64_t)dy->n * dy->d * dy->h * dy->w;
    const int64_t nchunks = (P + 63) / 64;
    const int64_t yz = (int64_t)(b.co_pad / (b.co_pad % 32 == 0 ? 32 : 16)) * ((ci + 15) / 16);
    int64_t g = std::max<int64_t>(1, std::min<int64_t>(nchunks, (1024 + yz - 1) / yz));
    // keep the partial sums within 64 Mi floats
    g = std::max<int64_t>(1, std::min<int64_t>(g, ((int64_t)1 << 26) / ((int64_t)b.co_pad * b.K)));
    b.max_groups = (int)g;
    b.bias_off = g * b.co_pad * b.K;
    b.ws_floats = b.bias_off + g * b.co_pad + std::min<int64_t>(16, g) * b.co_pad * ((int64_t)b.K + 1);
    return b;
}

template <int NOB, int NCB, int BX, int BY, int BZ, bool K1>
static void bwd_launch(const sg_view *x, const sg_view *dy, int pmask, float *dw, float *db, float *ws,
                       const BwdPlan &b, hipStream_t st)
{
    const int64_t P = (int64_t)x->n * x->d * x->h * x->w;
    const int nbx = (x->w + BX - 1) / BX, nby = (x->h + BY - 1) / BY, nbz = (x->d + BZ - 1) / BZ;
    const int64_t nb = K1 ? (P + WP - 1) / WP : (int64_t)x->n * nbx * nby * nbz;
    const int gy = b.co_pad / (16 * NOB), gz = (x->c + 16 * NCB - 1) / (16 * NCB);
    // position groups: as many workgroups as the GPU's 256 CUs hold at once
    // (registers: 3 per CU with one block pair, else 2), at least one brick each
    const int target = NOB * NCB == 1 ? 768 : 512;
    int64_t g = std::min<int64_t>(nb, std::max<int64_t>(1, target / ((int64_t)gy * gz)));
    g = std::min<int64_t>(g, b.max_groups);
    float *wsb = db ? ws + b.bias_off : nullptr;
    const dim3 grid((unsigned)g, gy, gz);
    if (!K1 && (x->w % BX || x->h % BY))
        hipLaunchKernelGGL((k_conv_bwd_w<NOB, NCB, BX, BY, BZ, K1, !K1>), grid, dim3(256), 0, st, *x, *dy, pmask,
                           b.co_pad, nbx, nby, nbz, nb, ws, wsb);
    else
        hipLaunchKernelGGL((k_conv_bwd_w<NOB, NCB, BX, BY, BZ, K1, false>), grid, dim3(256), 0, st, *x, *dy, pmask,
                           b.co_pad, nbx, nby, nbz, nb, ws, wsb);
    const int64_t n = (int64_t)dy->c * b.K;
    const int nbias = db ? dy->c : 0;
    hipLaunchKernelGGL(k_reduce_groups, dim3((unsigned)((n + nbias + 31) / 32)), dim3(256), 0, st, (const float *)ws,
                       (int64_t)b.co_pad * b.K, n, (const float *)wsb, b.co_pad, nbias, (int)g, dw, db);
}

template <int NOB, int NCB>
static void bwd_shape(const sg_view *x, const sg_view *dy, int pmask, float *dw, float *db, float *ws,
                      const BwdPlan &b, hipStream_t st)
{
    // the brick that pads the box least (16-wide rows on a tie)
    auto pad = [&](int bx, int by, int bz) {
        return (int64_t)((x->w + bx - 1) / bx * bx) * ((x->h + by - 1) / by * by) * ((x->d + bz - 1) / bz * bz);
    };
    const int64_t p16 = pad(16, 4, 4), p8 = pad(8, 8, 4), p4 = pad(4, 8, 8);
    if (p16 <= p8 && p16 <= p4) bwd_launch<NOB, NCB, 16, 4, 4, false>(x, dy, pmask, dw, db, ws, b, st);
    else if (p8 <= p4) bwd_launch<NOB, NCB, 8, 8, 4, false>(x, dy, pmask, dw, db, ws, b, st);
    else bwd_launch<NOB, NCB, 4, 8, 8, false>(x, dy, pmask, dw, db, ws, b, st);
}

// The weight-gradient kernels with the per-group partial sums in ws (at least
// b.ws_floats floats); shared by the workspace and the no-allocation entries.
static int bwd_weight_launch(const sg_view *x, const sg_view *dy, int32_t k, int32_t periodic_mask, float *dw,
                             float *db, float *ws, const BwdPlan &b, hipStream_t st)
{
    const int nci = (x->c + 15) / 16;
    const int64_t P = (int64_t)x->n * x->d * x->h * x->w;
    if (k == 1) {
        bwd_launch<1, 1, 16, 4, 4, true>(x, dy, periodic_mask, dw, db, ws, b, st);
    } else if (b.co_pad % 32 == 0 && nci % 2 == 0 && P / WP * (b.co_pad / 32) * (nci / 2) >= 256) {
        bwd_shape<2, 2>(x, dy, periodic_mask, dw, db, ws, b, st);
    } else if (b.co_pad % 32 == 0 && P / WP * (b.co_pad / 32) * nci >= 256) {
        bwd_shape<2, 1>(x, dy, periodic_mask, dw, db, ws, b, st);
    } else {
        bwd_shape<1, 1>(x, dy, periodic_mask, dw, db, ws, b, st);
    }
    return status();
}

}  // namespace sg

using namespace sg;

extern "C" {

int sg_conv3d_fwd(const sg_view *x, const void *w, const float *bias, int32_t co, int32_t k, int32_t periodic_mask,
                  int32_t relu, const sg_view *y, const sg_view *y32, int32_t accumulate, void *hip_stream)
{
    if (!mfma_view(x) || !w || co <= 0 || co % 16 || (k != 1 && k != 3)) return SG_EINVAL;
    if (!y && !y32) return SG_EINVAL;
    if (y && (!ok_view(y) || !same_pos(x, y) || y->c > co)) return SG_EINVAL;
    if (y32 && (!ok_view(y32) || !same_pos(x, y32) || y32->c > co)) return SG_EINVAL;
    const sg_view none = {};
    const int64_t P = (int64_t)x->n * x->d * x->h * x->w;
    const ConvArgs a{x, w, bias, co, periodic_mask, relu, y ? *y : none, y32 ? *y32 : none, accumulate,
                     (hipStream_t)hip_stream};
    const bool bricks = x->w % 16 == 0 && x->h % 4 == 0 && x->d % 4 == 0;
    if (k == 3 && bricks && (int64_t)x->d * x->h * x->w * (x->ctot / 8) < (int64_t)1 << 31) {
        // The order of a layer's sums (chunk length, DYR) follows from its channels
        // and extents, save that layers of a multiple of 32 outputs leave DYR at the
        // size `big` below, which counts the batch: a 32 -> 32 layer on 64 x 64 x 32
        // positions sums in another order for one item than for two.  Within an
        // order the launch shape goes by size and changes no bit.  Chunks: 16
        // channels where ci is no multiple of 32 and two planes per wave fit, or
        // where ci leaves 24 (an 8-channel layer's one chunk is 8 long); else 32.
        const bool two = x->d % 8 == 0, few = x->c % 32 != 0 && two, odd = x->c % 32 == 24;
        // large: two planes per wave for 32-channel chunks when that still leaves
        // at least 512 workgroups (less halo per output)
        const bool big = two && P / 512 * (co / 32) >= 512;
        // Below two workgroups of one output block per CU the weights go through
        // LDS: 192 -> 64 channels on 4 x 16^3 60 -> 26 us, 64 -> 64 there 22.7 ->
        // 12.7; above it the larger LDS use costs more (32 -> 64 on 128 x 32 x 32 25
        // us without, 43 with).  Not for the few input channels whose K loop is over
        // before the staging has paid (kernel us on 12 x 64 x 64, with / without: 8 ->
        // 16 7.7 / 5.7, 48 -> 16 11.3 / 9.8, 128 -> 16 17.3 / 19.9; 16 -> 32 9.9 / 8.8;
        // on 4 x 16^3 32 -> 32 8.8 / 10.2): up to 48 with one output block per
        // workgroup, up to 16 where the other form takes two.
        const bool small = P / 256 * (co / 16) <= 512 && x->c > (co % 32 ? 48 : 16);
        if (co % 32 == 0 && (few || odd)) {
            if (few) launch_conv3<2, 8, 16, false, false>(a);
            else launch_conv3<2, 4, 16, false, false>(a);
        } else if (co % 32 == 0 && big) {
            launch_conv3<2, 8, 32, false, false>(a);
        } else if (few || odd) {
            if (x->c == 8) launch_conv3<1, 8, 8, true, false>(a);
            else if (few) launch_conv3<1, 8, 16, true, false>(a);
            else launch_conv3<1, 4, 16, true, false>(a);
        } else {
            if (small) launch_conv3<1, 4, 32, true, true>(a);
            else if (co % 32 == 0) launch_conv3<2, 4, 32, true, false>(a);
            else launch_conv3<1, 4, 32, true, false>(a);
        }
        return status();
    }
    const int nout = std::max(y ? y->c : 0, y32 ? y32->c : 0);
    if (k == 1 && nout <= 4 && x->c <= 64) {
        hipLaunchKernelGGL(k_conv1_small<4>, dim3(grid_for(P)), dim3(256), 0, (hipStream_t)hip_stream, *x,
                           (const bf16 *)w, bias, relu, y ? *y : none, y32 ? *y32 : none, accumulate);
        return status();
    }
    // 32-bit byte offsets: tensors and weights below 2^31 bytes
    if (P * x->ctot * 2 < (int64_t)1 << 31 && (int64_t)co * k * k * k * x->c * 2 < (int64_t)1 << 31) {
        const int64_t waves = P / 64 * (co / 16);         // at 64 positions and one output block each
        // 64 positions per wave keep the reuse of four fragments per weight fragment
        // while there are waves enough; below that 16 positions per wave fill the
        // GPU (16 -> 16 on 72 x 40 x 40, 1800 waves: 17.6 us, 27 with 16; 64 -> 128 on
        // 4 x 8^3, 256 waves: 21.5, 40 with 64).  Two output blocks per wave once one
        // each would put a second wave on some of the 1024 SIMDs (192 -> 64 on 30 x 31
        // x 33, 1916 waves: 186 us with one, 117 with two; at 928 waves 99 with one).
        if (waves >= 1024 && co % 32 == 0) launch_direct<2, 4, 2>(a, k);
        else if (waves >= 512) launch_direct<1, 4, 3>(a, k);
        else launch_direct<1, 1, 8>(a, k);
        return status();
    }
    const unsigned gx = (unsigned)((P + 64 * FP - 1) / (64 * FP));
    if (co % 32 == 0)
        hipLaunchKernelGGL(k_conv_fwd<2>, dim3(gx, co / 32), dim3(256), 0, (hipStream_t)hip_stream, *x, (const bf16 *)w,
                           bias, k, periodic_mask, relu, y ? *y : none, y32 ? *y32 : none, accumulate);
    else
        hipLaunchKernelGGL(k_conv_fwd<1>, dim3(gx, co / 16), dim3(256), 0, (hipStream_t)hip_stream, *x, (const bf16 *)w,
                           bias, k, periodic_mask, relu, y ? *y : none, y32 ? *y32 : none, accumulate);
    return status();
}

int sg_weight_prep(const float *w32, int32_t co, int32_t ci, int32_t k, void *w_bf16, void *wt_bf16, int32_t co_pad,
                   int32_t ci_pad, void *hip_stream)
{
    if (!w32 || !w_bf16 || !wt_bf16 || co <= 0 || ci <= 0 || co_pad < co || ci_pad < ci || co_pad % 16 || ci_pad % 16 ||
        (k != 1 && k != 3))
        return SG_EINVAL;
    const int taps = k * k * k;
    const int64_t n = (int64_t)co_pad * taps * ci + (int64_t)ci_pad * taps * ((co + 7) & ~7);
    hipLaunchKernelGGL(k_weight_prep, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)hip_stream, w32, co, ci, k,
                       (bf16 *)w_bf16, (bf16 *)wt_bf16, co_pad, ci_pad);
    return status();
}

int64_t sg_conv3d_bwd_weight_ws(const sg_view *dy, int32_t ci, int32_t k)
{
    if (!ok_view(dy) || ci <= 0 || (k != 1 && k != 3)) return -1;
    return bwd_plan(dy, ci, k).ws_floats * (int64_t)sizeof(float);
}

static bool bwd_weight_args(const sg_view *x, const sg_view *dy, int32_t k, const float *dw)
{
    return mfma_view(x) && ok_view(dy) && dy->ctot % 8 == 0 && dy->coff % 8 == 0 && dy->c <= 256 && same_pos(x, dy) &&
           dw && (k == 1 || k == 3);
}

int sg_conv3d_bwd_weight(const sg_view *x, const sg_view *dy, int32_t k, int32_t periodic_mask, float *dw, float *db,
                         float *ws, int64_t ws_bytes, void *hip_stream)
{
    if (!bwd_weight_args(x, dy, k, dw) || !ws) return SG_EINVAL;
    const BwdPlan b = bwd_plan(dy, x->c, k);
    if (ws_bytes < b.ws_floats * (int64_t)sizeof(float)) return SG_EINVAL;
    return bwd_weight_launch(x, dy, k, periodic_mask, dw, db, ws, b, (hipStream_t)hip_stream);
}

int sg_conv3d_bwd_weight_noalloc(const sg_view *x, const sg_view *dy, int32_t k, int32_t periodic_mask, float *dw,
                                 float *db, void *hip_stream)
{
    if (!bwd_weight_args(x, dy, k, dw)) return SG_EINVAL;
    const BwdPlan b = bwd_plan(dy, x->c, k);
    if (b.ws_floats * (int64_t)sizeof(float) > SG_NOALLOC_SCRATCH_BYTES) return SG_EINVAL;
    float *ws = nullptr;
    const int rc = scratch_on_current_device(&ws);
    if (rc != SG_OK) return rc;
    return bwd_weight_launch(x, dy, k, periodic_mask, dw, db, ws, b, (hipStream_t)hip_stream);
}

int sg_relu_bwd_cast(const sg_view *dx, const sg_view *y, const sg_view *dyb, void *hip_stream)
{
    if (!ok_view(dx) || !ok_view(dyb) || !same_pos(dx, dyb) || dx->c != dyb->c) return SG_EINVAL;
    if (y && (!ok_view(y) || !same_pos(dx, y) || y->c != dx->c)) return SG_EINVAL;
    const sg_view none = {};
    const int64_t n = (int64_t)dx->n * dx->d * dx->h * dx->w * dx->c;
    if (dx->c % 8 == 0 && vec_view(dx, 4) && vec_view(dyb, 8) && (!y || vec_view(y, 8)) && n / 8 < (int64_t)1 << 31)
        hipLaunchKernelGGL(k_relu_bwd_castv<8>, dim3(grid_for(n / 8)), dim3(256), 0, (hipStream_t)hip_stream, *dx,
                           y ? *y : none, *dyb);
    else if (vec_view(dx, 4) && vec_view(dyb, 4) && (!y || vec_view(y, 4)) && n / 4 < (int64_t)1 << 31)
        hipLaunchKernelGGL(k_relu_bwd_castv<4>, dim3(grid_for(n / 4)), dim3(256), 0, (hipStream_t)hip_stream, *dx,
                           y ? *y : none, *dyb);
    else
        hipLaunchKernelGGL(k_relu_bwd_cast, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)hip_stream, *dx,
                           y ? *y : none, *dyb);
    return status();
}

static bool half_of(const sg_view *big, const sg_view *small)
{
    return big->n == small->n && big->d == 2 * small->d && big->h == 2 * small->h && big->w == 2 * small->w &&
           big->c == small->c;
}

int sg_pool2_fwd(const sg_view *x, const sg_view *y, void *hip_stream)
{
    if (!ok_view(x) || !ok_view(y) || !half_of(x, y)) return SG_EINVAL;
    const int64_t n = (int64_t)y->n * y->d * y->h * y->w * y->c;
    if (mfma_view(x) && mfma_view(y) && n / 8 < (int64_t)1 << 31)
        hipLaunchKernelGGL(k_pool2_fwd8, dim3(grid_for(n / 8)), dim3(256), 0, (hipStream_t)hip_stream, *x, *y);
    else
        hipLaunchKernelGGL(k_pool2_fwd, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)hip_stream, *x, *y);
    return status();
}

int sg_pool2_bwd(const sg_view *dy, const sg_view *dx, int32_t accumulate, void *hip_stream)
{
    if (!ok_view(dy) || !ok_view(dx) || !half_of(dx, dy)) return SG_EINVAL;
    const int64_t n = (int64_t)dx->n * dx->d * dx->h * dx->w * dx->c;
    if (vec_view(dy, 4) && vec_view(dx, 4) && n / 32 < (int64_t)1 << 31)
        hipLaunchKernelGGL(k_pool2_bwd4, dim3(grid_for(n / 32)), dim3(256), 0, (hipStream_t)hip_stream, *dy, *dx,
                           accumulate);
    else
        hipLaunchKernelGGL(k_pool2_bwd, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)hip_stream, *dy, *dx, accumulate);
    return status();
}

int sg_up2_cat_fwd(const sg_view *x, const sg_view *skip, const sg_view *y, void *hip_stream)
{
    if (!mfma_view(x) || !mfma_view(skip) || !mfma_view(y)) return SG_EINVAL;
    if (y->n != x->n || y->d != 2 * x->d || y->h != 2 * x->h || y->w != 2 * x->w) return SG_EINVAL;
    if (!same_pos(y, skip) || y->c != x->c + skip->c) return SG_EINVAL;
    const int64_t n = (int64_t)y->n * y->d * y->h * y->w * (y->c / 8);
    if (n >= (int64_t)1 << 31) return SG_EINVAL;
    hipLaunchKernelGGL(k_up2_cat8, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)hip_stream, *x, *skip, *y);
    return status();
}

int sg_up2_fwd(const sg_view *x, const sg_view *y, void *hip_stream)
{
    if (!ok_view(x) || !ok_view(y) || !half_of(y, x)) return SG_EINVAL;
    const int64_t n = (int64_t)y->n * y->d * y->h * y->w * y->c;
    if (mfma_view(x) && mfma_view(y) && n / 64 < (int64_t)1 << 31)
        hipLaunchKernelGGL(k_up2_fwd8, dim3(grid_for(n / 64)), dim3(256), 0, (hipStream_t)hip_stream, *x, *y);
    else
        hipLaunchKernelGGL(k_up2_fwd, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)hip_stream, *x, *y);
    return status();
}

int sg_up2_bwd(const sg_view *dy, const sg_view *dx, int32_t accumulate, void *hip_stream)
{
    if (!ok_view(dy) || !ok_view(dx) || !half_of(dy, dx)) return SG_EINVAL;
    const int64_t n = (int64_t)dx->n * dx->d * dx->h * dx->w * dx->c;
    if (vec_view(dy, 4) && vec_view(dx, 4) && n / 4 < (int64_t)1 << 31)
        hipLaunchKernelGGL(k_up2_bwd4, dim3(grid_for(n / 4)), dim3(256), 0, (hipStream_t)hip_stream, *dy, *dx,
                           accumulate);
    else
        hipLaunchKernelGGL(k_up2_bwd, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)hip_stream, *dy, *dx, accumulate);
    return status();
}

int sg_mse(const sg_view *out, const sg_view *target, const sg_view *grad, double *loss, void *hip_stream)
{
    if (!ok_view(out) || !ok_view(target) || !ok_view(grad) || !loss || !same_pos(out, target) ||
        !same_pos(out, grad) || out->c != target->c || out->c != grad->c)
        return SG_EINVAL;
    const int nb = 256;
    if (out->c == 4 && vec_view(out, 4) && vec_view(target, 4) && vec_view(grad, 4))
        hipLaunchKernelGGL(k_mse<true>, dim3(nb), dim3(1024), 0, (hipStream_t)hip_stream, *out, *target, *grad, loss + 1);
    else
        hipLaunchKernelGGL(k_mse<false>, dim3(nb), dim3(1024), 0, (hipStream_t)hip_stream, *out, *target, *grad, loss + 1);
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(64), 0, (hipStream_t)hip_stream, (const double *)(loss + 1), nb, loss);
    return status();
}

int sg_adam(float *w, const float *g, float *m, float *v, int64_t n, float lr, float beta1, float beta2, float eps,
            int64_t step, void *hip_stream)
{
    if (!w || !g || !m || !v || n <= 0 || step < 1) return SG_EINVAL;
    const float c1 = (float)(1.0 / (1.0 - std::pow((double)beta1, (double)step)));
    const float c2 = (float)(1.0 / (1.0 - std::pow((double)beta2, (double)step)));
    hipLaunchKernelGGL(k_adam, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)hip_stream, w, g, m, v, n, lr, beta1, beta2,
                       eps, c1, c2);
    return status();
}

static bool make_scale(const float *scale, int nf, Scale &sc)
{
    if (nf > 8) return false;
    for (int c = 0; c < 8; ++c) sc.s[c] = 1.0f;
    if (scale)
        for (int c = 0; c < nf; ++c) {
            if (!(scale[c] != 0.0f)) return false;
            sc.s[c] = scale[c];
        }
    return true;
}

int sg_pack(const float *f, int32_t nf, int32_t nx, int32_t ny, int32_t nz, int32_t x0, int32_t y0, int32_t z0,
            const float *scale, const sg_view *y, const sg_view *y32, int32_t b, void *hip_stream)
{
    Scale sc;
    if (!f || !ok_view(y) || nf <= 0 || nf > y->c || b < 0 || b >= y->n || x0 < 0 || y0 < 0 || z0 < 0 ||
        !make_scale(scale, nf, sc))
        return SG_EINVAL;
    if (y32 && (!ok_view(y32) || !same_pos(y, y32))) return SG_EINVAL;
    const sg_view none = {};
    if (y->c == 8 && mfma_view(y) && (!y32 || y32->c <= 8)) {
        const int64_t per = (int64_t)y->d * y->h * y->w;
        hipLaunchKernelGGL(k_pack8, dim3(grid_for(per)), dim3(256), 0, (hipStream_t)hip_stream, f, nf, nx, ny, nz, x0, y0,
                           z0, *y, y32 ? *y32 : none, b, sc);
        return status();
    }
    const int64_t n = (int64_t)y->d * y->h * y->w * y->c;
    hipLaunchKernelGGL(k_pack, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)hip_stream, f, nf, nx, ny, nz, x0, y0, z0,
                       *y, y32 ? *y32 : none, b, sc);
    return status();
}

int sg_unpack(const sg_view *x32, int32_t b, const float *scale, float *f, int32_t nf, void *hip_stream)
{
    Scale sc;
    if (!ok_view(x32) || !f || nf <= 0 || nf > x32->c || b < 0 || b >= x32->n || !make_scale(scale, nf, sc))
        return SG_EINVAL;
    const int64_t n = (int64_t)x32->d * x32->h * x32->w * nf;
    hipLaunchKernelGGL(k_unpack, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)hip_stream, *x32, b, f, nf, sc);
    return status();
}

int sg_lift(const float *pred, int64_t n, const float *rhoR_prev, const float *rhoB_prev, double cs2R, double cs2B,
            double p_in, double *out, void *hip_stream)
{
    if (!pred || !out || n <= 0 || !(cs2R > 0.0) || !(cs2B > 0.0) || (!rhoR_prev) != (!rhoB_prev) ||
        (!rhoR_prev && !(p_in > 0.0)))
        return SG_EINVAL;
    hipLaunchKernelGGL(k_lift, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)hip_stream, pred, n, rhoR_prev, rhoB_prev,
                       (float)cs2R, (float)cs2B, (float)p_in, out);
    return status();
}

}  // extern "C"
