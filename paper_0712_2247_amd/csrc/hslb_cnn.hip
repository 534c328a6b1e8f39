// Learned-force network on gfx950: 5x5x5 convolutions as implicit GEMMs on
// the BF16 matrix cores (v_mfma_f32_16x16x32_bf16, FP32 accumulation).
//
// MFMA operand layout (16x16x32): lane l holds A[m = l%16][k = 8(l/16) .. +8),
// B[k = 8(l/16) .. +8][n = l%16], and accumulates D[m = 4(l/16) + j][n = l%16],
// j = 0..3.  The 8 K-values of a lane are contiguous in K.
//
//  - Forward and input-gradient convolutions: M = 16 consecutive x-nodes of a
//    row, N = output channels, K = (tap, input channel).  The 8 K-values of a
//    lane are 8 channels of one node, a 16-byte load from channel-last bf16
//    activations.  A wave computes 4 rows (z) x 16 nodes against both 16-column
//    output halves; B comes pre-packed in lane order.  The forward layers with
//    32 input channels stage them in two halves of 16 (k_conv_fwd_split), which
//    halves the LDS per block and doubles the resident waves.
//  - Weight gradients: K = nodes, so a lane's 8 K-values are 8 consecutive
//    x-nodes of one channel (channel-major copies).  The x-shift of a tap is
//    taken from aligned 16-byte chunks with 16-bit funnel shifts, wrapping at
//    row ends (nx % 8 == 0 makes the chunks row-aligned).  Per-wave partial
//    sums go to scratch and a second kernel reduces them in a fixed order.
#include "hslb_cnn.hpp"
#include "hslb_internal.hpp"

#include <algorithm>
#include <cmath>

namespace hslb {
namespace cnn {
namespace {

typedef __bf16 bf16x8 __attribute__((__vector_size__(16)));
typedef float f32x4 __attribute__((__vector_size__(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// FP32 -> bf16, round to nearest, ties to even (finite inputs).
__device__ __forceinline__ uint32_t f2bf(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return u >> 16;
}

// FP64 -> bf16 directly: keep 8 significant bits of m in d = m 2^e, ties to even.
__device__ __forceinline__ uint32_t d2bf(double d)
{
    int e;
    const double m = frexp(d, &e);
    const double r = rint(m * 256.0) * (1.0 / 256.0);
    return __float_as_uint((float)ldexp(r, e)) >> 16;
}

__device__ __forceinline__ float bf2f(uint32_t h) { return __uint_as_float(h << 16); }

// The standard normal distribution function Phi(z) in FP32, with the Gaussian
// g = exp(-z^2/2) it is built from.  For t = |z|,
//   Phi(-t) = g E(t) / 2,  E(t) = exp(t^2/2) erfc(t / sqrt 2),
// and E = u P(u) with u = 1/(1 + 0.3 t) and P the degree-9 polynomial of
// gen_phi_poly.py (relative error of the fit 3.5e-9 on [0, 16]);
// Phi(z) = 1 - Phi(-z) for z > 0.  z^2 is split exactly (FMA), so that g keeps
// its relative accuracy far in the tail, and the Gaussian is the hardware
// base-2 exponential of c z^2 with the product's rounding carried to first
// order: the result is good to about 6e-7 relative also for z << 0 (where
// 1 + erf(z / sqrt 2) would cancel), with well under half the instructions of
// erfcf.  For z < -13 the Gaussian leaves the normal range (the caller takes
// the reference form there).
__device__ __forceinline__ float phi_cdf_fast(float z, float &g)
{
    const float t = fabsf(z);
    const float q = z * z;
    // g = 2^(c z^2), c = -log2(e) / 2 = CH + CL, z^2 = q + ql: x = q CH rounded, the
    // rest xl = c z^2 - x goes in to first order, g = 2^x (1 + ln2 xl)
    constexpr float CH = -0.7213475108146667f, CL = -9.629815167500055e-09f;
    const float ql = fmaf(z, z, -q);
    const float x = q * CH;
    const float xl = fmaf(q, CH, -x) + fmaf(q, CL, ql * CH);
    g = __builtin_amdgcn_exp2f(x) * fmaf(xl, 0.69314718055994531f, 1.0f);
    const float u = __builtin_amdgcn_rcpf(fmaf(0.3f, t, 1.0f));
    float p = -0.04126075655221939f;
    p = fmaf(p, u, 0.22495317459106445f);
    p = fmaf(p, u, -0.4566359519958496f);
    p = fmaf(p, u, 0.3838684558868408f);
    p = fmaf(p, u, -0.15911298990249634f);
    p = fmaf(p, u, 0.19246527552604675f);
    p = fmaf(p, u, 0.1567239612340927f);
    p = fmaf(p, u, 0.22048330307006836f);
    p = fmaf(p, u, 0.2391420602798462f);
    p = fmaf(p, u, 0.23937346041202545f);
    const float tail = 0.5f * g * (u * p);  // Phi(-t)
    return z < 0.f ? tail : 1.0f - tail;
}

// The reference evaluation, Phi(z) = erfc(-z / sqrt 2) / 2 (a few ulp).
__device__ __forceinline__ float phi_cdf_ref(float z) { return 0.5f * erfcf(-z * 0.70710678118654752f); }

// The forward activations are stored as bf16.  The fast form decides the
// rounding wherever it lies more than 32 FP32 ulps (at least 1.9e-6 relative,
// three times its distance from the reference form) from a bf16 rounding tie;
// the few values nearer a tie (about 1 in 1000) are evaluated again with
// erfcf.  The stored bits are therefore those of the reference form
// z * phi_cdf_ref(z), for a small share of its cost.
__device__ __forceinline__ bool near_bf16_tie(float v)
{
    const uint32_t lo = __float_as_uint(v) & 0xFFFFu;
    return lo - 0x7FE0u < 0x40u;  // lo within 0x8000 - 32 .. 0x8000 + 31
}

// GELU in the reference form, out of line: it runs for about one value in a
// thousand and would otherwise double the epilogue's code.
__device__ __attribute__((noinline)) float gelu_ref(float z) { return z * phi_cdf_ref(z); }

// bf16(GELU(z)), GELU(z) = z Phi(z)
__device__ __forceinline__ uint32_t gelu_bf16(float z)
{
    float g;
    float v = z * phi_cdf_fast(z, g);
    if (near_bf16_tie(v) || z < -13.0f) v = gelu_ref(z);
    return f2bf(v);
}

// bf16(d GELU'(z)), GELU'(z) = Phi(z) + z phi(z), in the reference form on every
// value: the two terms cancel near z = -0.75, where the fast form's absolute error
// (9e-8 in GELU', the reference form's 5e-8; 2.1e-7 against 1.2e-7 over all z) is no
// multiple of the small value's last place, so that no window around the rounding
// ties can hold it.  Nor is it faster: with such a window the input gradients of
// layers 2 and 3 take 106.8 + 45.8 us on 64 x 64 x 88, so 102.6 + 47.5 us.
__device__ __forceinline__ uint32_t dgelu_bf16(float d, float z)
{
    return f2bf(d * (phi_cdf_ref(z) + z * expf(-0.5f * z * z) * 0.39894228040143268f));
}

__device__ __forceinline__ bf16x8 as_bf(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

__device__ __forceinline__ int wrapi(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

// z of a tap read: -1 when it falls beyond a walled array.
__device__ __forceinline__ int zsrc(const Geo &g, int z)
{
    if (g.zper) return wrapi(z, g.nz);
    return (z < 0 || z >= g.nz) ? -1 : z;
}

// ------------------------------------------------------------- forward

// A block of 4 waves computes a 16 (x) x 4 (y) x 4 (z) tile of output nodes:
// wave w takes y0 + w, its 4 rows the layers z0 .. z0 + 3.  The input nodes
// the tile reads, 20 x 8 x 8 with the halo of 2, are staged in LDS once (x
// and y wrapped, z wrapped or zero beyond walls); every tap's A operand then
// comes from LDS.  32 input channels are staged as two halves of 32 B per node
// (40 KB each, k_conv_fwd_split); cin = 4: 8 B per node; cin = 1: 2 B.
#ifndef HSLB_CNN_TZ
#define HSLB_CNN_TZ 4
#endif
constexpr int TX = 16, TY = 4, TZ = HSLB_CNN_TZ;
constexpr int KQ = (NT + 1) / 2;  // two-tap K-steps per channel half (k_conv_fwd_split)
constexpr int HX = TX + 4, HY = TY + 4, HZ = TZ + 4, HNODES = HX * HY * HZ;
constexpr int ROWS = TZ;

// v mod n in [0, n) for v within a few periods of the range (halo indices of
// small lattices): adds and subtracts instead of two integer divisions.
__device__ __forceinline__ int mod_pos(int v, int n)
{
    while (v < 0) v += n;
    while (v >= n) v -= n;
    return v;
}

__host__ __device__ __forceinline__ constexpr int lnode(int hx, int hy, int hz) { return (hz * HY + hy) * HX + hx; }

// LDS byte offsets of the tap pairs of the split-channel convolution relative
// to the output node (16-byte parts): v[2q] is the offset of tap 2q, v[2q + 1]
// that of tap 2q + 1 minus it.  A block reads them as scalar loads; the pad
// tap t = NT reads the node itself (its weights are 0).
struct TapOffsets {
    uint32_t v[2 * KQ];
};
constexpr uint32_t tap_lds_offset(int t) { return t < NT ? (uint32_t)lnode(t % 5, (t / 5) % 5, t / 25) * 16u : 0u; }
constexpr TapOffsets make_tap_offsets()
{
    TapOffsets o{};
    for (int q = 0; q < KQ; ++q) {
        o.v[2 * q] = tap_lds_offset(2 * q);
        o.v[2 * q + 1] = tap_lds_offset(2 * q + 1) - tap_lds_offset(2 * q);
    }
    return o;
}
__constant__ TapOffsets c_tap_offsets = make_tap_offsets();

// Stages channel half hc (16 channels, two 16-byte parts per node, stored
// planar by part) of the block's input halo.  Wave w copies the halo rows
// (hz, hy) = w, w + 4, ...: their source y and z are uniform, and lanes
// 0 .. 2 HX - 1 take the row's HX nodes x 2 parts.
__device__ __forceinline__ void stage_half(const Geo &g, const uint16_t *__restrict__ in, uint16_t *tile, int x0,
                                           int y0, int z0, int hc, int lane)
{
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int hx = lane >> 1, pt = lane & 1;
    const bool act = lane < 2 * HX;
    const size_t col = (size_t)(act ? wrapi(x0 - 2 + hx, g.nx) : 0) * 32 + 16 * hc + 8 * pt;
    for (int row = w; row < HY * HZ; row += 4) {
        const int hy = row % HY, hz = row / HY;
        const int zr = z0 - 2 + hz;
        const int zs = g.zper ? mod_pos(zr, g.nz) : ((zr < 0 || zr >= g.nz) ? -1 : zr);
        const size_t rbase = (size_t)g.nx * (mod_pos(y0 - 2 + hy, g.ny) + (size_t)g.ny * (zs < 0 ? 0 : zs)) * 32;
        if (act) {
            u32x4 v = {0u, 0u, 0u, 0u};
            if (zs >= 0) v = *(const u32x4 *)(in + rbase + col);
            ((u32x4 *)tile)[pt * HNODES + row * HX + hx] = v;
        }
    }
}


template <int CIN>
__device__ __forceinline__ void stage_tile(const Geo &g, const uint16_t *__restrict__ in, uint16_t *tile, int x0,
                                           int y0, int z0)
{
    static_assert(CIN == 1 || CIN == 4, "32-channel inputs are staged by halves (stage_half)");
    for (int node = threadIdx.x; node < HNODES; node += 256) {
        const int hx = node % HX, hy = (node / HX) % HY, hz = node / (HX * HY);
        const int zr = z0 - 2 + hz;
        const int zs = g.zper ? mod_pos(zr, g.nz) : ((zr < 0 || zr >= g.nz) ? -1 : zr);
        size_t src = 0;
        if (zs >= 0) src = (size_t)wrapi(x0 - 2 + hx, g.nx) + (size_t)g.nx * (mod_pos(y0 - 2 + hy, g.ny) + (size_t)g.ny * zs);
        if constexpr (CIN == 4) {
            u32x2 v = {0u, 0u};
            if (zs >= 0) v = *(const u32x2 *)(in + src * 4);
            ((u32x2 *)tile)[node] = v;
        } else {
            tile[node] = zs >= 0 ? in[src] : (uint16_t)0;
        }
    }
}

// Tap offsets of the A operands of k_conv_fwd, in tile nodes relative to the
// lane's node, per K-step s and lane group lg: CIN 1, taps 32 s + 8 lg + e
// (e = 0..7); CIN 4, taps 8 s + 2 lg + q (q = 0, 1).  Taps past the last read
// the node itself against zero weights.  A lane reads its step's offsets with
// one or two 16-byte loads instead of dividing each tap index by 5 and 25.
struct FwdTapOffsets {
    uint32_t c1[4][4][8];
    uint32_t c4[16][4][4];  // q = 0, 1 used; padded to 16 bytes
};
constexpr uint32_t tap_node(int t) { return t < NT ? (uint32_t)lnode(t % 5, (t / 5) % 5, t / 25) : 0u; }
constexpr FwdTapOffsets make_fwd_tap_offsets()
{
    FwdTapOffsets o{};
    for (int s = 0; s < 4; ++s)
        for (int lg = 0; lg < 4; ++lg)
            for (int e = 0; e < 8; ++e) o.c1[s][lg][e] = tap_node(32 * s + 8 * lg + e);
    for (int s = 0; s < 16; ++s)
        for (int lg = 0; lg < 4; ++lg)
            for (int q = 0; q < 2; ++q) o.c4[s][lg][q] = tap_node(8 * s + 2 * lg + q);
    return o;
}
__constant__ FwdTapOffsets c_fwd_taps = make_fwd_tap_offsets();

// A operand of K-step s for the lane's node `node` (tile index of row r) from
// the step's tap offsets.
template <int CIN>
__device__ __forceinline__ u32x4 lds_a(const uint16_t *tile, int node, const uint32_t (&off)[8])
{
    u32x4 v = {0u, 0u, 0u, 0u};
    if constexpr (CIN == 4) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const u32x2 w2 = ((const u32x2 *)tile)[node + off[q]];
            v[2 * q] = w2[0];
            v[2 * q + 1] = w2[1];
        }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e >> 1] |= (uint32_t)tile[node + off[e]] << (16 * (e & 1));
    }
    return v;
}

// Where the four pre-activations a lane holds of row r, half h lie in zfrag: in
// the order in which the lanes hold them, so that a wave reads and writes whole
// kilobytes.  The forward layers and the input gradients use the same tiles;
// the rows of a partial z tile are packed, so that the array has N x 32 values.
__device__ __forceinline__ size_t zfrag_at(const Geo &g, int x0, int y0, int z0, int rows, int w, int r, int h, int lane)
{
    const int tile = x0 / TX + (g.nx / TX) * (y0 / TY);
    return (size_t)g.nx * g.ny * z0 * 32 + (((size_t)tile * 4 + w) * rows + r) * 512 + h * 256 + lane * 4;
}

// The channel-last copy of a block's 32-channel bf16 results, from ot.
__device__ __forceinline__ void store_cl(const FwdArgs &a, const Geo &g, const uint16_t *ot, int x0, int y0, int z0,
                                         int rows)
{
    constexpr int TN = TX * TY * TZ;
    for (int q = threadIdx.x; q < TN * 4; q += 256) {
        const int l = q >> 2, pt = q & 3;
        const int x = l % TX, y = (l / TX) % TY, r = l / (TX * TY);
        if (r < rows) {
            const size_t node = (size_t)(x0 + x) + (size_t)g.nx * ((y0 + y) + (size_t)g.ny * (z0 + r));
            *(u32x4 *)(a.out_cl + node * 32 + 8 * pt) = *(const u32x4 *)(ot + l * 32 + 8 * pt);
        }
    }
}

// Stores a block's 32-channel bf16 results: lane (li, lg) holds v[r][h][j] of
// node (x0 + 4 lg + j, y0 + w, z0 + r), channel 16 h + li.  The channel-last
// copy goes through LDS and leaves as whole 16-byte node parts; of the
// channel-major copy a lane has four consecutive nodes, 8 bytes.  `ot` holds
// TX * TY * TZ * 32 bf16 (16 KB) of LDS that no wave reads any more; tile-local
// node l = (r TY + y) TX + x.
__device__ __forceinline__ void store_bf16(const FwdArgs &a, const Geo &g, uint16_t *ot, const uint32_t (&v)[ROWS][2][4],
                                           int x0, int y0, int z0, int rows, int w, int li, int lg)
{
    if (a.out_cm) {
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            if (r >= rows) continue;
            const size_t node = (size_t)(x0 + 4 * lg) + (size_t)g.nx * ((y0 + w) + (size_t)g.ny * (z0 + r));
#pragma unroll
            for (int h = 0; h < 2; ++h)
                *(u32x2 *)(a.out_cm + (size_t)(16 * h + li) * g.N + node) =
                    (u32x2){v[r][h][0] | v[r][h][1] << 16, v[r][h][2] | v[r][h][3] << 16};
        }
    }
    if (!a.out_cl) return;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int j = 0; j < 4; ++j) ot[((r * TY + w) * TX + 4 * lg + j) * 32 + 16 * h + li] = (uint16_t)v[r][h][j];
    __syncthreads();
    store_cl(a, g, ot, x0, y0, z0, rows);
}

// GELU epilogue of a forward layer with 32 output channels outside training: only
// the channel-last activations are wanted, and each goes to LDS as it is formed.
// The training epilogue holds all 32 of a lane and tests its optional outputs: on
// 64 x 64 x 136 layers 1 and 2 take 34.4 + 124.9 us with it, 31.5 + 121.8 us so.
__device__ __forceinline__ void gelu_epilogue_cl(const FwdArgs &a, const Geo &g, uint16_t *ot,
                                                 const f32x4 (&acc)[ROWS][2], int x0, int y0, int z0, int rows, int w,
                                                 int li, int lg)
{
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                ot[((r * TY + w) * TX + 4 * lg + j) * 32 + 16 * h + li] =
                    (uint16_t)gelu_bf16(acc[r][h][j] + a.bias[16 * h + li]);
    __syncthreads();
    store_cl(a, g, ot, x0, y0, z0, rows);
}

// GELU epilogue of a forward layer with 32 output channels, and the GELU'
// epilogue of an input gradient, on the sums acc[r][h][j] held as v above.
// 64 x 64 x 88 in training, where the pre-activations are kept and both copies
// written: layer 1 44 -> 36 us, layer 2 104 -> 101 us, input gradients of layer 2
// 120 -> 103 us and of layer 3 62 -> 48 us (before, the pre-activations moved as
// single words and the copies as single bf16 values).
__device__ __forceinline__ void gelu_epilogue(const FwdArgs &a, const Geo &g, uint16_t *ot, const f32x4 (&acc)[ROWS][2],
                                              int x0, int y0, int z0, int rows, int w, int li, int lg)
{
    uint32_t v[ROWS][2][4];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const int rowbase = g.nx * ((y0 + w) + g.ny * (z0 + r));
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int c = 16 * h + li;
            f32x4 zz;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                zz[j] = acc[r][h][j] + a.bias[c];
                v[r][h][j] = gelu_bf16(zz[j]);
                if (a.out_f32 && r < rows) a.out_f32[(size_t)(rowbase + x0 + 4 * lg + j) * 32 + c] = zz[j];
            }
            if (a.zfrag && r < rows) *(f32x4 *)(a.zfrag + zfrag_at(g, x0, y0, z0, rows, w, r, h, 16 * lg + li)) = zz;
        }
    }
    store_bf16(a, g, ot, v, x0, y0, z0, rows, w, li, lg);
}

__device__ __forceinline__ void dgelu_epilogue(const FwdArgs &a, const Geo &g, uint16_t *ot, const f32x4 (&acc)[ROWS][2],
                                               int x0, int y0, int z0, int rows, int w, int li, int lg)
{
    uint32_t v[ROWS][2][4];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const int rowbase = g.nx * ((y0 + w) + g.ny * (z0 + min(r, rows - 1)));
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int c = 16 * h + li;
            f32x4 zz;
            if (a.zfrag)
                zz = *(const f32x4 *)(a.zfrag + zfrag_at(g, x0, y0, z0, rows, w, min(r, rows - 1), h, 16 * lg + li));
            else
#pragma unroll
                for (int j = 0; j < 4; ++j) zz[j] = a.zsave[(size_t)(rowbase + x0 + 4 * lg + j) * 32 + c];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[r][h][j] = dgelu_bf16(acc[r][h][j], zz[j]);
                if (a.out_f32 && r < rows) a.out_f32[(size_t)(rowbase + x0 + 4 * lg + j) * 32 + c] = acc[r][h][j];
            }
        }
    }
    store_bf16(a, g, ot, v, x0, y0, z0, rows, w, li, lg);
}

// Layer 1 forward (1 -> 32 channels, GELU epilogue) and the input gradient of
// layer 3 (its 3 output-gradient channels padded to 4 -> 32, GELU' epilogue):
// the block's whole input halo fits LDS (2 or 8 bytes per node).  The B
// operands (the same for every block, so cache hits) are loaded PD K-steps
// ahead into a register ring; rows past the end of a partial z tile are
// computed on the staged zeros or wrapped layers and not stored, which keeps
// the loop free of branches.
template <int CIN, int EPI, bool TRAIN>
__global__ __launch_bounds__(256) void k_conv_fwd(FwdArgs a)
{
    static_assert((CIN == 1 && EPI == EPI_GELU) || (CIN == 4 && EPI == EPI_DGELU),
                  "layer 1 forward, layer 3 input gradient");
    constexpr int NH = 2;
    constexpr int KS = CIN == 4 ? 16 : 4;
    __shared__ __attribute__((aligned(16))) uint16_t tile[HNODES * CIN];
    const Geo g = a.g;
    const int nxb = g.nx / TX, nyb = g.ny / TY;
    const int b = xcd_block((int)blockIdx.x, (int)gridDim.x);
    const int zb = b / (nxb * nyb);
    const int rem = b - zb * nxb * nyb;
    const int yb = rem / nxb;
    const int x0 = (rem - yb * nxb) * TX, y0 = yb * TY, z0 = zb * TZ;
    stage_tile<CIN>(g, a.in, tile, x0, y0, z0);
    __syncthreads();

    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int li = lane & 15, lg = lane >> 4;
    const int rows = min(ROWS, g.nz - z0);  // the last z tile may be partial
    f32x4 acc[ROWS][NH];
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int h = 0; h < NH; ++h) acc[r][h] = (f32x4){0.f, 0.f, 0.f, 0.f};

    constexpr int PD = 8;
    auto load_b = [&](int s, int h) { return *(const u32x4 *)(a.wp + ((size_t)(s * NH + h) * 64 + lane) * 8); };
    u32x4 bq[PD][NH];
#pragma unroll
    for (int q = 0; q < PD; ++q)
#pragma unroll
        for (int h = 0; h < NH; ++h) bq[q][h] = q < KS ? load_b(q, h) : (u32x4){0u, 0u, 0u, 0u};
    for (int s0 = 0; s0 < KS; s0 += PD) {
#pragma unroll
        for (int q = 0; q < PD; ++q) {
            const int s = s0 + q;
            if (s < KS) {
                uint32_t off[8];
                if constexpr (CIN == 1) {
                    const u32x4 o0 = *(const u32x4 *)&c_fwd_taps.c1[s][lg][0];
                    const u32x4 o1 = *(const u32x4 *)&c_fwd_taps.c1[s][lg][4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        off[e] = o0[e];
                        off[4 + e] = o1[e];
                    }
                } else {
                    const u32x4 o0 = *(const u32x4 *)&c_fwd_taps.c4[s][lg][0];
#pragma unroll
                    for (int e = 0; e < 4; ++e) off[e] = o0[e];
                    off[4] = off[5] = off[6] = off[7] = 0u;
                }
                bf16x8 av[ROWS], bw[NH];
#pragma unroll
                for (int r = 0; r < ROWS; ++r) av[r] = as_bf(lds_a<CIN>(tile, lnode(li, w, r), off));
#pragma unroll
                for (int h = 0; h < NH; ++h) {
                    bw[h] = as_bf(bq[q][h]);
                    if (s + PD < KS) bq[q][h] = load_b(s + PD, h);
                }
#pragma unroll
                for (int r = 0; r < ROWS; ++r)
#pragma unroll
                    for (int h = 0; h < NH; ++h)
                        acc[r][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[r], bw[h], acc[r][h], 0, 0, 0);
            }
        }
    }

    __shared__ __attribute__((aligned(16))) uint16_t ot[TX * TY * TZ * 32];
    if constexpr (EPI == EPI_GELU && TRAIN)
        gelu_epilogue(a, g, ot, acc, x0, y0, z0, rows, w, li, lg);
    else if constexpr (EPI == EPI_GELU)
        gelu_epilogue_cl(a, g, ot, acc, x0, y0, z0, rows, w, li, lg);
    else
        dgelu_epilogue(a, g, ot, acc, x0, y0, z0, rows, w, li, lg);
}

// Forward layer 2 (32 -> 32 channels, GELU) and its input gradient
// (transposed weights, GELU' epilogue), with the input channels in two halves
// of 16.  The staged halo then holds 32 B per node (40 KB instead of
// 80 KB), so four blocks share a compute unit, twice the resident waves of the
// 64-byte halo, which hides the latencies of the LDS and weight reads.  A K-step
// of 32 covers two taps x 16 channels: lane group lg takes tap 2q + lg/2 and
// channels 8 (lg % 2) .. + 8 of the half; the weights come packed in that order
// (PK_F2, PK_D2).  Output layout and epilogues as k_conv_fwd.  The K-loop
// carries no branch and no per-lane index arithmetic: the tap offsets come
// from a constant table through scalar loads, the B ring runs on over the
// zero-padded end of the pack, and a ring slot is refilled after its products
// are issued (no register copies, no wait on a load just issued).  On the
// 64x64x136 slit layer 2 takes 141 us (40 % of the BF16 peak; 188 us with
// per-lane tap division and guarded loads, 249 us with the 64-byte halo).
template <int NH, int EPI, bool TRAIN>
__global__ __launch_bounds__(256, 4) void k_conv_fwd_split(FwdArgs a)
{
    static_assert(NH == 2 && (EPI == EPI_GELU || EPI == EPI_DGELU), "layer 2 forward and input gradient");
    __shared__ __attribute__((aligned(16))) uint16_t tile[HNODES * 16];
    const Geo g = a.g;
    const int nxb = g.nx / TX, nyb = g.ny / TY;
    const int b = xcd_block((int)blockIdx.x, (int)gridDim.x);
    const int zb = b / (nxb * nyb);
    const int rem = b - zb * nxb * nyb;
    const int yb = rem / nxb;
    const int x0 = (rem - yb * nxb) * TX, y0 = yb * TY, z0 = zb * TZ;

    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int li = lane & 15, lg = lane >> 4;
    const int part = lg & 1, second = lg >> 1;
    const int rows = min(ROWS, g.nz - z0);
    f32x4 acc[ROWS][NH];
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int h = 0; h < NH; ++h) acc[r][h] = (f32x4){0.f, 0.f, 0.f, 0.f};

    // B operands: a ring of PD K-steps loaded ahead, over the steps of both
    // channel halves in a row (the packs end in PACK_PAD zero steps).
    constexpr int PD = 3;
    static_assert(KQ % PD == 0 && PD <= PACK_PAD, "the prefetch ring runs on across the halves");
    auto load_b = [&](int sq, int h) { return *(const u32x4 *)(a.wp + ((size_t)(sq * NH + h) * 64 + lane) * 8); };
    u32x4 bq[PD][NH];
#pragma unroll
    for (int q = 0; q < PD; ++q)
#pragma unroll
        for (int h = 0; h < NH; ++h) bq[q][h] = load_b(q, h);
    // A operands: the LDS byte offset of a lane's node (x0 + li, y0 + w, z0)
    // of its 16-byte part, plus the offset of its tap of the pair.
    const uint32_t lane_base = (uint32_t)(part * HNODES + lnode(li, w, 0)) * 16u;
    const uint32_t second_mask = second ? ~0u : 0u;
    constexpr uint32_t ROW_BYTES = HX * HY * 16;
    for (int hc = 0; hc < 2; ++hc) {
        if (hc) __syncthreads();  // every wave is done with the first half
        stage_half(g, a.in, tile, x0, y0, z0, hc, lane);
        __syncthreads();
#pragma unroll 1
        for (int q0 = 0; q0 < KQ; q0 += PD) {
#pragma unroll
            for (int qq = 0; qq < PD; ++qq) {
                const int q = q0 + qq;
                const uint32_t t0 = __builtin_amdgcn_readfirstlane(c_tap_offsets.v[2 * q]);
                const uint32_t dt = __builtin_amdgcn_readfirstlane(c_tap_offsets.v[2 * q + 1]);
                const uint32_t off = lane_base + t0 + (dt & second_mask);
                bf16x8 av[ROWS];
#pragma unroll
                for (int r = 0; r < ROWS; ++r)
                    av[r] = as_bf(*(const u32x4 *)((const char *)tile + off + r * ROW_BYTES));
#pragma unroll
                for (int r = 0; r < ROWS; ++r)
#pragma unroll
                    for (int h = 0; h < NH; ++h)
                        acc[r][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[r], as_bf(bq[qq][h]), acc[r][h], 0, 0, 0);
                // refill the ring slot once its products are issued, so that
                // the load lands in the same registers
#pragma unroll
                for (int h = 0; h < NH; ++h) bq[qq][h] = load_b(hc * KQ + q + PD, h);
            }
        }
    }

    static_assert(TX * TY * TZ * 32 <= HNODES * 16, "the block's activations fit the halo buffer");
    if constexpr (EPI == EPI_GELU && TRAIN)
        gelu_epilogue(a, g, tile, acc, x0, y0, z0, rows, w, li, lg);
    else if constexpr (EPI == EPI_GELU)
        gelu_epilogue_cl(a, g, tile, acc, x0, y0, z0, rows, w, li, lg);
    else
        dgelu_epilogue(a, g, tile, acc, x0, y0, z0, rows, w, li, lg);
}

// Layer 3 forward (32 -> 3 channels) with (output channel, dx) on the M
// dimension of the products instead of the 16 x-nodes: M = 15 used of 16
// rows (c, dx), N = 16 input columns x', K = 16 channels x two (dy, dz) taps.
// The partial sums P[(c, dx)][x'] of a row then give
//   out[c][x] = b[c] + sum_dx P[(c, dx)][x + dx]
// through LDS.  A wave covers the 20 input columns of its 16 output nodes with
// two N-tiles (32 columns, 20 used) and 4 z-rows, so a K-step is 8 products
// against 1 weight fragment, where the node-major form (3 of 16 output
// columns used) needs 2.4 times the products and LDS reads.  Halo staging and
// the block's tile as in k_conv_fwd_split.  Weights packed as PK_F3.  On the
// 64x64x136 slit: 61 us, against 91 us for the node-major form in the
// split-channel kernel (69 us with the K loop rolled).
constexpr int KD = 13;  // (dy, dz) pair steps per channel half: 25 taps + 1 pad

struct DyDzOffsets {
    uint32_t v[2 * KD];
};
constexpr DyDzOffsets make_dydz_offsets()
{
    DyDzOffsets o{};
    for (int q = 0; q < KD; ++q)
        for (int p = 0; p < 2; ++p) {
            const int i = 2 * q + p;
            o.v[i] = i < 25 ? (uint32_t)lnode(0, i % 5, i / 5) * 16u : 0u;
        }
    return o;
}
__constant__ DyDzOffsets c_dydz_offsets = make_dydz_offsets();

__global__ __launch_bounds__(256, 4) void k_conv_out(FwdArgs a)
{
    __shared__ __attribute__((aligned(16))) uint16_t tile[HNODES * 16];
    const Geo g = a.g;
    const int nxb = g.nx / TX, nyb = g.ny / TY;
    const int b = xcd_block((int)blockIdx.x, (int)gridDim.x);
    const int zb = b / (nxb * nyb);
    const int rem = b - zb * nxb * nyb;
    const int yb = rem / nxb;
    const int x0 = (rem - yb * nxb) * TX, y0 = yb * TY, z0 = zb * TZ;

    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int li = lane & 15, lg = lane >> 4;
    const int part = lg & 1, second = lg >> 1;
    const int rows = min(ROWS, g.nz - z0);
    f32x4 acc[ROWS][2];
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) acc[r][nt] = (f32x4){0.f, 0.f, 0.f, 0.f};

    // B operand: column x' = li + 16 nt of the halo (x0 - 2 + x'); the columns
    // past the halo's 20 are not needed and read its last one.
    uint32_t col_base[2];
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
        col_base[nt] = (uint32_t)(part * HNODES + lnode(min(li + 16 * nt, HX - 1), w, 0)) * 16u;
    const uint32_t second_mask = second ? ~0u : 0u;
    constexpr uint32_t ROW_BYTES = HX * HY * 16;
    auto load_a = [&](int sq) { return *(const u32x4 *)(a.wp + ((size_t)sq * 64 + lane) * 8); };
    u32x4 wq = load_a(0);
    for (int hc = 0; hc < 2; ++hc) {
        if (hc) __syncthreads();
        stage_half(g, a.in, tile, x0, y0, z0, hc, lane);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < KD; ++q) {  // unrolled: the next step's LDS reads start early
            const uint32_t t0 = __builtin_amdgcn_readfirstlane(c_dydz_offsets.v[2 * q]);
            const uint32_t t1 = __builtin_amdgcn_readfirstlane(c_dydz_offsets.v[2 * q + 1]);
            const uint32_t off = t0 + ((t1 - t0) & second_mask);
            const bf16x8 wa = as_bf(wq);
            wq = load_a(hc * KD + q + 1);  // the pack ends in PACK_PAD zero steps
#pragma unroll
            for (int r = 0; r < ROWS; ++r)
#pragma unroll
                for (int nt = 0; nt < 2; ++nt) {
                    const bf16x8 bv = as_bf(*(const u32x4 *)((const char *)tile + col_base[nt] + off + r * ROW_BYTES));
                    acc[r][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa, bv, acc[r][nt], 0, 0, 0);
                }
        }
    }

    // P[r][m][x'] of the wave through LDS (the halo is no longer read), then
    // out[c][x0 + i] = b[c] + sum_dx P[r][5 c + dx][i + dx].
    __syncthreads();
    float *P = (float *)tile + w * (ROWS * 16 * 32);
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int j = 0; j < 4; ++j) P[(r * 16 + 4 * lg + j) * 32 + li + 16 * nt] = acc[r][nt][j];
    __syncthreads();
    for (int k = lane; k < ROWS * CO * 16; k += 64) {
        const int i = k & 15, c = (k >> 4) % CO, r = k / (16 * CO);
        if (r >= rows) continue;
        float v = a.bias[c];
#pragma unroll
        for (int dx = 0; dx < 5; ++dx) v += P[(r * 16 + 5 * c + dx) * 32 + i + dx];
        const size_t node = (size_t)(x0 + i) + (size_t)g.nx * ((y0 + w) + (size_t)g.ny * (z0 + r));
        a.out_f32[(size_t)c * g.N + node] = (a.out_zero >> c) & 1 ? 0.f : v;
    }
}

// ---------------------------------------------------- weight gradients

// 8 consecutive elements starting at element `sh` (in -2..2) of the chunk
// `cur`, continuing into `prv` / `nxt`.
__device__ __forceinline__ u32x4 shifted(const u32x4 &prv, const u32x4 &cur, const u32x4 &nxt, int sh)
{
    u32x4 o;
    if (sh == 0) return cur;
    if (sh == 2) {
        o[0] = cur[1];
        o[1] = cur[2];
        o[2] = cur[3];
        o[3] = nxt[0];
    } else if (sh == -2) {
        o[0] = prv[3];
        o[1] = cur[0];
        o[2] = cur[1];
        o[3] = cur[2];
    } else if (sh == 1) {
        o[0] = (cur[0] >> 16) | (cur[1] << 16);
        o[1] = (cur[1] >> 16) | (cur[2] << 16);
        o[2] = (cur[2] >> 16) | (cur[3] << 16);
        o[3] = (cur[3] >> 16) | (nxt[0] << 16);
    } else {
        o[0] = (prv[3] >> 16) | (cur[0] << 16);
        o[1] = (cur[0] >> 16) | (cur[1] << 16);
        o[2] = (cur[1] >> 16) | (cur[2] << 16);
        o[3] = (cur[2] >> 16) | (cur[3] << 16);
    }
    return o;
}

// rows (y, z) of the lattice split into chunks of rpw rows
struct RowSplit {
    int rows, rpw, chunks;
};

__host__ __device__ inline RowSplit row_split(const Geo &g, int max_chunks)
{
    RowSplit r;
    r.rows = g.ny * g.nz;
    const int c = r.rows < max_chunks ? r.rows : max_chunks;
    r.rpw = (r.rows + c - 1) / c;
    r.chunks = (r.rows + r.rpw - 1) / r.rpw;
    return r;
}

constexpr int WG_CHUNKS_TAP = 1024; // layer 1: waves = chunks

// Layers 2 and 3: M = input channel (2 x 16), N = output channel (NB x 16),
// K = nodes.  A block takes one dz and a run of lattice rows (a chunk), ten
// waves: wave (dy, mi) the five dx taps of one dy and 16 input channels.  The
// block marches along y, four rows a step (one on small lattices): the input rows
// y - 2 .. y + 5 of z + dz lie in a ring of sixteen LDS rows (with 8 nodes of x
// halo on either side, periodic), so that each is loaded once for the 25 taps, and
// the step's rows of the output gradient in a double buffer.  A step's rows are loaded two
// steps ahead and written to LDS behind the products of the step before it, one
// barrier a step.  A lane reads its 8 nodes and the chunks on either side and
// forms the five shifted operands by funnel shifts.  The rows' LDS strides are
// odd multiples of 16 bytes (no bank conflicts among the 16 channels of a read).
//   On 64 x 64 x 88, layer 2 (92 GFLOP) took 349 us with a wave per (dz, dy) and
// its operands straight from L2 (2.3 GB of it), 129 us with two rows a step,
// loaded one step ahead (each step then waits out a memory round trip), 102 us
// now; layer 3, whose products fill 3 of the 16 columns, 254 -> 72 us.
//   A chunk is summed in two halves, each from zero, and the halves meet in the
// FP64 sum of the reduction: one FP32 chain over the whole chunk is longer than
// that of the 64 chunks which a wave per (dz, dy) took, and its rounding larger
// (rms against FP64 sums, layer 2 on 64 x 64 x 88: 64 chunks 4.7e-7, 51 chunks
// 5.3e-7, 51 chunks in halves 3.6e-7 of the gradient's rms; the whole gradient
// takes 2 % longer, 637 -> 652 us, for the reduction's second 26 MB).
// partial[chunk][half][dz][dy][dx][32][16 NB]
constexpr int WG_CHUNKS = 51;  // x 5 dz: a block per compute unit
constexpr int WG_WAVES = 10, WG_RING = 16, WG_ROWS = 4, WG_STEPS = 112;

// x tile of a row: 64 nodes where they divide it, else 32
__host__ __device__ inline int wg_xt(const Geo &g) { return g.nx % 64 == 0 ? 64 : 32; }

// Rows a step and chunks of a lattice.  Up to WG_STEPS four-row steps it takes
// one row a step instead: a half of a chunk is then the longer FP32 chain, up to
// four rows where the 64 chunks of a wave per (dz, dy) had one (on 32 x 8 x 12
// rms 6.5e-8 against 4.9e-8; with one-row steps 3.9e-8).  One-row steps keep every
// chain at ceil(ceil(rows / 51) / 2) <= ceil(rows / 64) rows, four-row steps from
// 113 on (eight rows in a half against at least 452 / 64).  No more chunks than
// steps: the reductions of up to 102 empty sums took the whole gradient of
// 32 x 4 x 1 from 204 to 248 us.
struct WgSplit {
    int rs, chunks;
};
inline WgSplit wg_split(const Geo &g)
{
    const int tiles = g.nx / wg_xt(g) * g.nz;
    const int rs = tiles * (g.ny / WG_ROWS) <= WG_STEPS ? 1 : WG_ROWS;
    return {rs, std::min(WG_CHUNKS, tiles * (g.ny / rs))};
}

template <int NB, int XT, int RS>
__global__ __launch_bounds__(64 * WG_WAVES) void k_wgrad_rows(Geo g, int chunks, int cout, const uint16_t *__restrict__ actT,
                                                              const uint16_t *__restrict__ gT, float *__restrict__ partial)
{
    constexpr int SA = XT + 24, SB = XT + 8;       // row strides in elements
    constexpr int CA = XT / 8 + 2, CB = XT / 8;    // 16-byte chunks of a row
    constexpr int T = 64 * WG_WAVES;
    __shared__ __attribute__((aligned(16))) uint16_t s_a[WG_RING][32][SA];
    __shared__ __attribute__((aligned(16))) uint16_t s_b[2][RS][16 * NB][SB];
    // the five dz of a chunk and neighbouring chunks on one XCD: they share rows
    const int lb = xcd_block((int)blockIdx.x, (int)gridDim.x);
    const int chunk = lb / 5, dz = lb - 5 * chunk - 2;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int li = lane & 15, lg = lane >> 4;
    const int dy = w % 5 - 2, mi = w / 5;
    f32x4 acc[5][NB];
#pragma unroll
    for (int d = 0; d < 5; ++d)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[d][nb] = (f32x4){0.f, 0.f, 0.f, 0.f};
    if constexpr (NB == 1) {
        // channels past cout stay zero
        for (int q = threadIdx.x; q < 2 * RS * 16 * NB * SB / 8; q += T) ((u32x4 *)s_b)[q] = (u32x4){0u, 0u, 0u, 0u};
    }
    // layers z whose tap z + dz lies in the array, and this chunk's steps of them
    const int zfirst = g.zper || dz > 0 ? 0 : -dz;
    const int zcount = g.zper ? g.nz : max(0, g.nz - abs(dz));
    const int ph = g.ny / RS, steps = (g.nx / XT) * zcount * ph;
    const int p0 = (int)((int64_t)steps * chunk / chunks), p1 = (int)((int64_t)steps * (chunk + 1) / chunks);
    // 16-byte chunks of the thread: of the step's new input rows (halo included)
    // and of its output-gradient rows, at most two each
    constexpr int K = RS == 1 ? 1 : 2;
    static_assert(RS * 32 * CA <= K * T && RS * 16 * NB * CB <= K * T, "K chunks per thread and step");
    bool ha[K], hb[K];
    int ac[K], arow[K], aoff[K], lao[K], boff[K], brow[K], lbo[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int q = (int)threadIdx.x + k * T, ach = (q / CA) & 31, bch = (q / CB) % cout;
        ha[k] = q < RS * 32 * CA;
        hb[k] = q < RS * cout * CB;
        ac[k] = q % CA;
        arow[k] = q / (CA * 32);
        aoff[k] = ach * g.N;
        lao[k] = ach * SA + 8 * ac[k];
        brow[k] = q / (CB * cout);
        boff[k] = bch * g.N + 8 * (q % CB) + g.nx * brow[k];
        lbo[k] = (brow[k] * 16 * NB + bch) * SB + 8 * (q % CB);
    }
    struct Rows {
        u32x4 a[K], b[K];
    };
    // input rows Y .. Y + RS - 1 of layer zs (-2 <= Y < ny + 8), gradient rows
    // y .. y + RS - 1
    auto load_a = [&](Rows &v, int x0, int zs, int Y) {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (ha[k])
                v.a[k] = *(const u32x4 *)(actT + (size_t)aoff[k] +
                                          (wrapi(x0 - 8 + 8 * ac[k], g.nx) +
                                           g.nx * (mod_pos(Y + arow[k], g.ny) + g.ny * zs)));
    };
    auto load_b = [&](Rows &v, int x0, int z, int y) {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (hb[k]) v.b[k] = *(const u32x4 *)(gT + (size_t)boff[k] + (x0 + g.nx * (y + g.ny * z)));
    };
    auto put_a = [&](const Rows &v, int Y) {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (ha[k]) *(u32x4 *)(&s_a[0][0][0] + ((Y + arow[k]) & (WG_RING - 1)) * (32 * SA) + lao[k]) = v.a[k];
    };
    auto put_b = [&](const Rows &v, int buf) {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (hb[k]) *(u32x4 *)(&s_b[buf][0][0][0] + lbo[k]) = v.b[k];
    };
    int x0 = 0, z = 0, y = 0;
    if (p0 < p1) {
        const int col = p0 / ph, seg = col / zcount;
        y = RS * (p0 - col * ph);
        x0 = seg * XT;
        z = zfirst + col - seg * zcount;
    }
    Rows v0, v1;  // the next step's rows, the one after's
    int buf = 0, half = 0;
    const int pm = (p0 + p1 + 1) / 2;  // first step of the second half
    auto flush = [&](int h) {
        float *out = partial + ((size_t)((2 * chunk + h) * 5 + dz + 2) * 25 + (size_t)(dy + 2) * 5) * 32 * 16 * NB;
#pragma unroll
        for (int d = 0; d < 5; ++d)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    out[((size_t)d * 32 + 16 * mi + 4 * lg + j) * 16 * NB + 16 * nb + li] = acc[d][nb][j];
                acc[d][nb] = (f32x4){0.f, 0.f, 0.f, 0.f};
            }
    };
    for (int p = p0; p < p1;) {
        // a run: the steps of one column that belong to the chunk
        const int n = min(p1 - p, (g.ny - y) / RS);
        const int zs = g.zper ? mod_pos(z + dz, g.nz) : z + dz;
        // the first step's rows y - 2 .. y + RS + 1
        load_a(v0, x0, zs, y - 2);
        load_b(v0, x0, z, y);
        load_a(v1, x0, zs, y - 2 + RS);
        __syncthreads();  // every wave is done with the ring
        put_a(v0, y - 2);
        put_b(v0, buf);
        put_a(v1, y - 2 + RS);
        if constexpr (RS == 1) {
            Rows v[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) load_a(v[k], x0, zs, y + k);
#pragma unroll
            for (int k = 0; k < 3; ++k) put_a(v[k], y + k);
        }
        if (n > 1) {
            load_a(v0, x0, zs, y + RS + 2);
            load_b(v0, x0, z, y + RS);
        }
        __syncthreads();
        for (int i = 0; i < n; ++i) {
            if (p + i == pm) {
                flush(0);
                half = 1;
            }
            if (i + 2 < n) {
                load_a(v1, x0, zs, y + 2 * RS + 2);
                load_b(v1, x0, z, y + 2 * RS);
            }
#pragma unroll
            for (int row = 0; row < RS; ++row) {
                const uint16_t *ra = &s_a[(y + row + dy) & (WG_RING - 1)][16 * mi + li][8];
#pragma unroll
                for (int k = 0; k < XT / 32; ++k) {
                    const int x = 32 * k + 8 * lg;
                    bf16x8 bv[NB];
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) bv[nb] = as_bf(*(const u32x4 *)&s_b[buf][row][16 * nb + li][x]);
                    // whole chunks: single words at this stride would meet in
                    // 16 of the banks
                    const u32x4 cur = *(const u32x4 *)(ra + x);
                    u32x4 prv = *(const u32x4 *)(ra + x - 8), nxt = *(const u32x4 *)(ra + x + 8);
                    __asm__("" : "+v"(prv), "+v"(nxt));  // not narrowed to the words used
#pragma unroll
                    for (int d = 0; d < 5; ++d) {
                        const bf16x8 av = as_bf(shifted(prv, cur, nxt, d - 2));
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb)
                            acc[d][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv[nb], acc[d][nb], 0, 0, 0);
                    }
                }
            }
            if (i + 1 < n) {
                put_a(v0, y + RS + 2);
                put_b(v0, buf ^ 1);
                v0 = v1;
                __syncthreads();
            }
            buf ^= 1;
            y += RS;
        }
        p += n;
        if (y == g.ny) {
            y = 0;
            if (++z == zfirst + zcount) {
                z = zfirst;
                x0 += XT;
            }
        }
    }
    flush(half);
    if (half == 0) flush(1);  // a chunk of one step or none: the second half is empty
}

// dW[co][ci][t] = sum over the chunks' halves; threads run over co fastest, then ci, so
// that neighbouring threads read neighbouring partials
__global__ __launch_bounds__(256) void k_wgrad_ch_reduce(int chunks, int nb16, int cout, const float *__restrict__ partial,
                                                         float *__restrict__ dW)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= cout * 32 * NT) return;
    const int co = i % cout, ci = (i / cout) % 32, t = i / (cout * 32);
    double s = 0.0;
#pragma unroll 8
    for (int c = 0; c < chunks; ++c) s += partial[(((size_t)c * NT + t) * 32 + ci) * nb16 + co];
    dW[(co * 32 + ci) * NT + t] = (float)s;
}

// Layer 1: M = tap (8 x 16, taps >= 125 zero), N = output channel (2 x 16),
// K = nodes.  Each lane's tap has its own shift.  partial[wave][128][32]
__global__ __launch_bounds__(256) void k_wgrad_tap(Geo g, RowSplit rs, const uint16_t *__restrict__ x,
                                                   const uint16_t *__restrict__ gT, float *__restrict__ partial)
{
    const int lane = threadIdx.x & 63;
    const int wave = blockIdx.x * 4 + (int)(threadIdx.x >> 6);
    if (wave >= rs.chunks) return;
    const int li = lane & 15, lg = lane >> 4;
    f32x4 acc[8][2];
#pragma unroll
    for (int mi = 0; mi < 8; ++mi)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) acc[mi][nb] = (f32x4){0.f, 0.f, 0.f, 0.f};

    const int r0 = wave * rs.rpw, r1 = min(rs.rows, r0 + rs.rpw);
    for (int row = r0; row < r1; ++row) {
        const int y = row % g.ny, z = row / g.ny;
        const size_t orow = (size_t)g.nx * (y + g.ny * z);
        for (int x0 = 0; x0 < g.nx; x0 += 32) {
            const int xc = x0 + 8 * lg;
            bf16x8 bv[2];
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) bv[nb] = as_bf(*(const u32x4 *)(gT + (size_t)(16 * nb + li) * g.N + orow + xc));
            const int xp = xc == 0 ? g.nx - 8 : xc - 8, xn = xc + 8 == g.nx ? 0 : xc + 8;
#pragma unroll
            for (int mi = 0; mi < 8; ++mi) {
                const int t = 16 * mi + li;
                u32x4 v = {0u, 0u, 0u, 0u};
                if (t < NT) {
                    const int dz = t / 25 - 2, dy = (t / 5) % 5 - 2, dx = t % 5 - 2;
                    const int zs = zsrc(g, z + dz);
                    if (zs >= 0) {
                        const uint16_t *base = x + (size_t)g.nx * (wrapi(y + dy, g.ny) + g.ny * zs);
                        const u32x4 cur = *(const u32x4 *)(base + xc);
                        const u32x4 prv = dx < 0 ? *(const u32x4 *)(base + xp) : cur;
                        const u32x4 nxt = dx > 0 ? *(const u32x4 *)(base + xn) : cur;
                        v = shifted(prv, cur, nxt, dx);
                    }
                }
                const bf16x8 av = as_bf(v);
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
                    acc[mi][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv[nb], acc[mi][nb], 0, 0, 0);
            }
        }
    }
    float *out = partial + (size_t)wave * 128 * 32;
#pragma unroll
    for (int mi = 0; mi < 8; ++mi)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int j = 0; j < 4; ++j) out[(16 * mi + 4 * lg + j) * 32 + 16 * nb + li] = acc[mi][nb][j];
}

// dW1[co][0][t]: a block per tap, 8 groups of 32 threads (co) over the chunks,
// the groups' sums added in order (a thread per (co, t) walking all 1024 chunks
// left 240 of the 256 compute units idle and took 219 us)
__global__ __launch_bounds__(256) void k_wgrad_tap_reduce(int chunks, const float *__restrict__ partial,
                                                          float *__restrict__ dW)
{
    __shared__ double s_sum[8][32];
    const int co = threadIdx.x & 31, grp = threadIdx.x >> 5, t = blockIdx.x;
    double s = 0.0;
#pragma unroll 8
    for (int c = grp; c < chunks; c += 8) s += partial[((size_t)c * 128 + t) * 32 + co];
    s_sum[grp][co] = s;
    __syncthreads();
    if (grp == 0) {
#pragma unroll
        for (int k = 1; k < 8; ++k) s += s_sum[k][co];
        dW[co * NT + t] = (float)s;
    }
}

// --------------------------------------------------------- reductions

__device__ __forceinline__ double block_sum(double v, double *red)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    const double t = (red[0] + red[1]) + (red[2] + red[3]);
    __syncthreads();
    return t;
}

constexpr int COLSUM_CHUNKS = 64;

__device__ __forceinline__ double wave_sum64(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    return v;
}

// Bias gradients of all layers at once: blocks (chunk, channel), the channels of
// the three tensors in a row.  partial[c][chunk]
__global__ __launch_bounds__(256) void k_colsum(Geo g, ColSums cs, float *__restrict__ partial)
{
    __shared__ double red[4];
    int c = blockIdx.y, k = 0;
    while (c >= cs.nch[k]) c -= cs.nch[k++];
    const uint16_t *gT = cs.g[k] + (size_t)c * g.N;
    const int chunk = blockIdx.x;
    const int per = ((g.N + COLSUM_CHUNKS - 1) / COLSUM_CHUNKS + 7) / 8 * 8;  // N is a multiple of 128
    const int n0 = chunk * per, n1 = min(g.N, n0 + per);
    double s = 0.0;
    for (int n = n0 + 8 * (int)threadIdx.x; n < n1; n += 8 * 256) {
        const u32x4 v = *(const u32x4 *)(gT + n);
#pragma unroll
        for (int e = 0; e < 4; ++e) s += (double)bf2f(v[e] & 0xFFFFu) + (double)bf2f(v[e] >> 16);
    }
    const double t = block_sum(s, red);
    if (threadIdx.x == 0) partial[blockIdx.y * COLSUM_CHUNKS + chunk] = (float)t;
}

__global__ void k_colsum_reduce(ColSums cs, const float *__restrict__ partial)
{
    int c = blockIdx.x, k = 0;
    while (c >= cs.nch[k]) c -= cs.nch[k++];
    const double t = wave_sum64((double)partial[blockIdx.x * COLSUM_CHUNKS + threadIdx.x]);
    if (threadIdx.x == 0) cs.db[k][c] = (float)t;
}

// ------------------------------------------------------------ packing

__global__ __launch_bounds__(256) void k_pack(int kind, const float *__restrict__ w, uint16_t *__restrict__ out, int total)
{
    const int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    const int e = idx & 7, lane = (idx >> 3) & 63, rest = idx >> 9;
    const int li = lane & 15, lg = lane >> 4;
    const int H = kind == PK_F3 ? 1 : 2;
    const int h = rest % H, s = rest / H;
    const int col = 16 * h + li;
    float v = 0.f;
    if (kind == PK_F1) {
        const int t = 32 * s + 8 * lg + e;
        if (t < NT) v = w[OW1 + col * NT + t];
    } else if (kind == PK_F2) {
        // channel half hc, two-tap step q: lane group lg holds tap 2q + lg/2,
        // channels 16 hc + 8 (lg % 2) .. + 8 (k_conv_fwd_split); zero padding
        // steps after the second half
        const int hc = s / KQ, q = s - hc * KQ, t = 2 * q + (lg >> 1);
        if (hc < 2 && t < NT) v = w[OW2 + (col * CH + 16 * hc + 8 * (lg & 1) + e) * NT + t];
    } else if (kind == PK_F3) {
        // A operand of k_conv_out: row li = (output channel li / 5, dx li % 5),
        // channel half hc, (dy, dz) pair step q: lane group lg holds tap
        // (dy, dz) number 2q + lg/2 (dz major), channels 16 hc + 8 (lg % 2) .. + 8
        const int hc = s / KD, q = s - hc * KD, i = 2 * q + (lg >> 1);
        const int c = li / 5, dx = li % 5;
        if (hc < 2 && c < CO && i < 25) v = w[OW3 + (c * CH + 16 * hc + 8 * (lg & 1) + e) * NT + (i / 5) * 25 + (i % 5) * 5 + dx];
    } else if (kind == PK_D2) {
        // transposed, tap-flipped layer-2 weights in the split order of PK_F2
        const int hc = s / KQ, q = s - hc * KQ, t = 2 * q + (lg >> 1);
        if (hc < 2 && t < NT) v = w[OW2 + ((16 * hc + 8 * (lg & 1) + e) * CH + col) * NT + (NT - 1 - t)];
    } else {
        const int t = 8 * s + 2 * lg + (e >> 2), cf = e & 3;
        if (t < NT && cf < CO) v = w[OW3 + (cf * CH + col) * NT + (NT - 1 - t)];
    }
    out[idx] = (uint16_t)f2bf(v);
}

// --------------------------------------------------------------- misc

template <typename TM>
__global__ __launch_bounds__(256) void k_eta_input(Geo g, int hz, double eta_pref, const TM *__restrict__ n,
                                                   uint16_t *__restrict__ x)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= g.N) return;
    const int plane = g.nx * g.ny;
    x[i] = (uint16_t)d2bf(eta_pref * (double)n[i + hz * plane]);
}

__global__ __launch_bounds__(256) void k_to_bf16(const double *__restrict__ v, size_t count, uint16_t *__restrict__ out)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < count) out[i] = (uint16_t)d2bf(v[i]);
}

__global__ __launch_bounds__(256) void k_loss(Geo g, int wall_lo, int wall_hi, float scale, const float *__restrict__ out,
                                              const float *__restrict__ target, uint16_t *__restrict__ d_cl,
                                              uint16_t *__restrict__ d_cm, double *__restrict__ sq_partial)
{
    __shared__ double red[4];
    const int i = blockIdx.x * 256 + threadIdx.x;
    double sq = 0.0;
    if (i < g.N) {
        const int z = i / (g.nx * g.ny);
        const bool fl = z >= wall_lo && z < g.nz - wall_hi;
#pragma unroll
        for (int c = 0; c < CO; ++c) {
            const float d = fl ? out[(size_t)c * g.N + i] - target[(size_t)c * g.N + i] : 0.f;
            sq += (double)d * (double)d;
            const uint16_t b = (uint16_t)f2bf(d * scale);
            d_cl[(size_t)i * 4 + c] = b;
            d_cm[(size_t)c * g.N + i] = b;
        }
        d_cl[(size_t)i * 4 + 3] = 0;
    }
    const double t = block_sum(sq, red);
    if (threadIdx.x == 0) sq_partial[blockIdx.x] = t;
}

__global__ __launch_bounds__(256) void k_adam(int n, float *__restrict__ w, float *__restrict__ m, float *__restrict__ v,
                                              const float *__restrict__ g, float c1, float c2, float lr)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = 0.9f * m[i] + 0.1f * gi;
    const float vi = 0.999f * v[i] + 0.001f * gi * gi;
    m[i] = mi;
    v[i] = vi;
    w[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + 1e-8f);
}

// Residual of the force the surrogate path applies, fs F_hat + delta_old
// (delta_old only with use_prev), against the exact C1 over fluid nodes; then
// delta = C1 - fs F_hat (in place: each node reads its old value first).
__global__ __launch_bounds__(256) void k_judge(Geo g, int wall_lo, int wall_hi, double fs, const float *__restrict__ fhat,
                                               const double *__restrict__ c1, int use_prev, float *__restrict__ delta,
                                               double *__restrict__ partial)
{
    __shared__ double red[4];
    const int i = blockIdx.x * 256 + threadIdx.x;
    double a = 0.0, b = 0.0;
    if (i < g.N) {
        const int z = i / (g.nx * g.ny);
        const bool fl = z >= wall_lo && z < g.nz - wall_hi;
#pragma unroll
        for (int c = 0; c < CO; ++c) {
            const size_t k = (size_t)c * g.N + i;
            const double e = c1[k];
            const double f = fhat ? fs * (double)fhat[k] : 0.0;
            if (fl) {
                const double pred = f + (use_prev ? (double)delta[k] : 0.0);
                a += (e - pred) * (e - pred);
                b += e * e;
            }
            delta[k] = fl ? (float)(e - f) : 0.f;
        }
    }
    const double ta = block_sum(a, red);
    const double tb = block_sum(b, red);
    if (threadIdx.x == 0) {
        partial[2 * blockIdx.x] = ta;
        partial[2 * blockIdx.x + 1] = tb;
    }
}

__global__ __launch_bounds__(256) void k_f32_to_f64(const float *__restrict__ in, double s, size_t count,
                                                    double *__restrict__ out)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < count) out[i] = s * (double)in[i];
}

__global__ __launch_bounds__(256) void k_f64_to_f32(const double *__restrict__ in, double s, size_t count,
                                                    float *__restrict__ out)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < count) out[i] = (float)(s * in[i]);
}

__global__ __launch_bounds__(256) void k_cm_to_bf16(const float *__restrict__ in, int c, int cp, int N,
                                                    uint16_t *__restrict__ out_cl, uint16_t *__restrict__ out_cm)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (size_t)cp * N) return;
    const int n = (int)(i / cp), k = (int)(i % cp);
    const uint16_t b = k < c ? (uint16_t)f2bf(in[(size_t)k * N + n]) : (uint16_t)0;
    if (out_cl) out_cl[i] = b;
    if (out_cm && k < c) out_cm[(size_t)k * N + n] = b;
}

__global__ __launch_bounds__(256) void k_cl_bf16_to_cm(const uint16_t *__restrict__ in, int c, int N, float *__restrict__ out)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (size_t)c * N) return;
    const int k = (int)(i / N), n = (int)(i % N);
    out[i] = bf2f(in[(size_t)n * c + k]);
}

__global__ __launch_bounds__(256) void k_cl_f32_to_cm(const float *__restrict__ in, int c, int N, float *__restrict__ out)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (size_t)c * N) return;
    const int k = (int)(i / N), n = (int)(i % N);
    out[i] = in[(size_t)n * c + k];
}

inline unsigned nblocks(size_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

hipError_t launch_conv_fwd(hipStream_t s, int cin, int cout, int epi, const FwdArgs &a)
{
    const int blocks = (a.g.nx / TX) * (a.g.ny / TY) * ((a.g.nz + TZ - 1) / TZ);
    const dim3 grid(blocks), blk(256);
    const int nh = cout == 32 ? 2 : 1;
    const bool train = a.zfrag || a.out_f32 || a.out_cm || !a.out_cl;
    if (cin == 1 && nh == 2 && epi == EPI_GELU) {
        if (train) hipLaunchKernelGGL((k_conv_fwd<1, EPI_GELU, true>), grid, blk, 0, s, a);
        else hipLaunchKernelGGL((k_conv_fwd<1, EPI_GELU, false>), grid, blk, 0, s, a);
        return hipGetLastError();
    }
    if (cin == 32 && nh == 2 && epi == EPI_GELU) {
        if (train) hipLaunchKernelGGL((k_conv_fwd_split<2, EPI_GELU, true>), grid, blk, 0, s, a);
        else hipLaunchKernelGGL((k_conv_fwd_split<2, EPI_GELU, false>), grid, blk, 0, s, a);
        return hipGetLastError();
    }
    if (cin == 32 && nh == 2 && epi == EPI_DGELU) {
        hipLaunchKernelGGL((k_conv_fwd_split<2, EPI_DGELU, true>), grid, blk, 0, s, a);
        return hipGetLastError();
    }
    if (cin == 32 && nh == 1 && epi == EPI_OUT) {
        hipLaunchKernelGGL(k_conv_out, grid, blk, 0, s, a);
        return hipGetLastError();
    }
    if (cin == 4 && nh == 2 && epi == EPI_DGELU) {
        hipLaunchKernelGGL((k_conv_fwd<4, EPI_DGELU, true>), grid, blk, 0, s, a);
        return hipGetLastError();
    }
    return hipErrorInvalidValue;
}

size_t wgrad_partial_floats(const Geo &g, int layer)
{
    if (layer == 1) return (size_t)row_split(g, WG_CHUNKS_TAP).chunks * 128 * 32;
    return (size_t)2 * wg_split(g).chunks * NT * 32 * 16 * (layer == 2 ? 2 : 1);
}

template <int NB>
void launch_wgrad_rows(hipStream_t s, const Geo &g, const WgSplit &ws, int cout, const uint16_t *src, const uint16_t *gT,
                       float *partial)
{
    const dim3 grid(5 * ws.chunks), blk(64 * WG_WAVES);
    const bool x64 = wg_xt(g) == 64;
#define HSLB_WG(XT, RS) \
    hipLaunchKernelGGL((k_wgrad_rows<NB, XT, RS>), grid, blk, 0, s, g, ws.chunks, cout, src, gT, partial)
    if (ws.rs == 1) {
        if (x64) HSLB_WG(64, 1);
        else HSLB_WG(32, 1);
    } else {
        if (x64) HSLB_WG(64, WG_ROWS);
        else HSLB_WG(32, WG_ROWS);
    }
#undef HSLB_WG
}

hipError_t launch_wgrad(hipStream_t s, int layer, const Geo &g, const uint16_t *src, const uint16_t *gT,
                        float *partial, float *dW)
{
    if (layer == 1) {
        const RowSplit rs = row_split(g, WG_CHUNKS_TAP);
        hipLaunchKernelGGL(k_wgrad_tap, dim3((rs.chunks + 3) / 4), dim3(256), 0, s, g, rs, src, gT, partial);
        hipLaunchKernelGGL(k_wgrad_tap_reduce, dim3(NT), dim3(256), 0, s, rs.chunks, partial, dW);
        return hipGetLastError();
    }
    const WgSplit ws = wg_split(g);
    if (layer == 2) {
        launch_wgrad_rows<2>(s, g, ws, CH, src, gT, partial);
        hipLaunchKernelGGL(k_wgrad_ch_reduce, dim3(nblocks(CH * 32 * NT)), dim3(256), 0, s, 2 * ws.chunks, 32, CH, partial, dW);
    } else {
        launch_wgrad_rows<1>(s, g, ws, CO, src, gT, partial);
        hipLaunchKernelGGL(k_wgrad_ch_reduce, dim3(nblocks(CO * 32 * NT)), dim3(256), 0, s, 2 * ws.chunks, 16, CO, partial, dW);
    }
    return hipGetLastError();
}

size_t colsum_partial_floats(const Geo &, int nch) { return (size_t)nch * COLSUM_CHUNKS; }

hipError_t launch_colsum(hipStream_t s, const Geo &g, const ColSums &cs, float *partial)
{
    const int nch = cs.nch[0] + cs.nch[1] + cs.nch[2];
    hipLaunchKernelGGL(k_colsum, dim3(COLSUM_CHUNKS, nch), dim3(256), 0, s, g, cs, partial);
    hipLaunchKernelGGL(k_colsum_reduce, dim3(nch), dim3(COLSUM_CHUNKS), 0, s, cs, partial);
    return hipGetLastError();
}

hipError_t launch_pack(hipStream_t s, int kind, const float *w, uint16_t *out)
{
    const int total = pack_elems(kind);
    hipLaunchKernelGGL(k_pack, dim3(nblocks(total)), dim3(256), 0, s, kind, w, out, total);
    return hipGetLastError();
}

template <typename TM>
hipError_t launch_eta_input(hipStream_t s, const Geo &g, int hz, double eta_pref, const TM *n, uint16_t *x)
{
    hipLaunchKernelGGL(k_eta_input<TM>, dim3(nblocks(g.N)), dim3(256), 0, s, g, hz, eta_pref, n, x);
    return hipGetLastError();
}
template hipError_t launch_eta_input<float>(hipStream_t, const Geo &, int, double, const float *, uint16_t *);
template hipError_t launch_eta_input<double>(hipStream_t, const Geo &, int, double, const double *, uint16_t *);

hipError_t launch_to_bf16(hipStream_t s, const double *v, size_t count, uint16_t *out)
{
    hipLaunchKernelGGL(k_to_bf16, dim3(nblocks(count)), dim3(256), 0, s, v, count, out);
    return hipGetLastError();
}

unsigned loss_blocks(const Geo &g) { return nblocks(g.N); }

hipError_t launch_loss(hipStream_t s, const Geo &g, int wall_lo, int wall_hi, const float *out, const float *target,
                       uint16_t *d_cl, uint16_t *d_cm, double *sq_partial)
{
    const long nf = (long)g.nx * g.ny * (g.nz - wall_lo - wall_hi);
    const float scale = (float)(2.0 / (3.0 * (double)nf));
    hipLaunchKernelGGL(k_loss, dim3(loss_blocks(g)), dim3(256), 0, s, g, wall_lo, wall_hi, scale, out, target, d_cl, d_cm,
                       sq_partial);
    return hipGetLastError();
}

hipError_t launch_adam(hipStream_t s, int n, float *w, float *m, float *v, const float *g, int t, float lr)
{
    const float c1 = (float)(1.0 / (1.0 - std::pow(0.9, t)));
    const float c2 = (float)(1.0 / (1.0 - std::pow(0.999, t)));
    hipLaunchKernelGGL(k_adam, dim3(nblocks(n)), dim3(256), 0, s, n, w, m, v, g, c1, c2, lr);
    return hipGetLastError();
}

unsigned judge_blocks(const Geo &g) { return nblocks(g.N); }

hipError_t launch_cm_to_bf16(hipStream_t s, const float *in, int c, int cp, int N, uint16_t *out_cl, uint16_t *out_cm)
{
    hipLaunchKernelGGL(k_cm_to_bf16, dim3(nblocks((size_t)cp * N)), dim3(256), 0, s, in, c, cp, N, out_cl, out_cm);
    return hipGetLastError();
}

hipError_t launch_cl_bf16_to_cm(hipStream_t s, const uint16_t *in, int c, int N, float *out)
{
    hipLaunchKernelGGL(k_cl_bf16_to_cm, dim3(nblocks((size_t)c * N)), dim3(256), 0, s, in, c, N, out);
    return hipGetLastError();
}

hipError_t launch_cl_f32_to_cm(hipStream_t s, const float *in, int c, int N, float *out)
{
    hipLaunchKernelGGL(k_cl_f32_to_cm, dim3(nblocks((size_t)c * N)), dim3(256), 0, s, in, c, N, out);
    return hipGetLastError();
}

hipError_t launch_scale_f32_to_f64(hipStream_t st, const float *in, double s, size_t count, double *out)
{
    hipLaunchKernelGGL(k_f32_to_f64, dim3(nblocks(count)), dim3(256), 0, st, in, s, count, out);
    return hipGetLastError();
}

hipError_t launch_scale_f64_to_f32(hipStream_t st, const double *in, double s, size_t count, float *out)
{
    hipLaunchKernelGGL(k_f64_to_f32, dim3(nblocks(count)), dim3(256), 0, st, in, s, count, out);
    return hipGetLastError();
}

hipError_t launch_judge(hipStream_t s, const Geo &g, int wall_lo, int wall_hi, double fs, const float *fhat,
                        const double *c1, int use_prev, float *delta, double *partial)
{
    hipLaunchKernelGGL(k_judge, dim3(judge_blocks(g)), dim3(256), 0, s, g, wall_lo, wall_hi, fs, fhat, c1, use_prev,
                       delta, partial);
    return hipGetLastError();
}

}  // namespace cnn
}  // namespace hslb
