// The learned preconditioner network N for flexible CG: three 3x3x3
// convolutions (1 -> 16 -> 16 -> 1 channels, zero padding 1, ReLU between
// layers), its parameter gradients (for an MSE loss, or for any loss given
// its output gradient: the energy-norm error the preconditioner is trained
// on), and Adam.  The paper names
// preconditioning as the untried remedy for slow CG convergence (Sec.
// "Smooth Temporal Evolution"); the network approximates the inverse of the
// normal operator on residuals.
//
// gfx950 design:
// * Hidden activations are BF16, channels-last ([voxel][16], 32 B per voxel),
//   so one voxel's 16 channels are one contiguous 32-byte run.
// * Every layer is a contraction over (tap, input channel) and runs on MFMA
//   over row tiles of 16 voxels: D[cout][voxel] += A[cout][k] B[k][voxel],
//   with the weights held in registers and the inputs read from an LDS copy
//   of the tile's region.  For a 16-channel input the taps (dz, dy, dx) go
//   in nine x-triples: v_mfma_f32_16x16x32_bf16 takes dx = 0 and 1 (two
//   taps of 16 channels), v_mfma_f32_16x16x16_bf16 takes dx = 2.  The B
//   operand of an x-triple depends only on the input row (y + dy, z + dz),
//   so each input row read from LDS feeds the up to three output rows that
//   use it (dy = 0, 1, 2): half the LDS reads of pairing the taps in order.
//   D lands as out[voxel l % 16][4 (l / 16) .. +3]: one 8-byte store.  The
//   same kernel computes the 16 -> 16 data gradient with flipped, transposed
//   weights.
// * The 1 -> 16 layer takes its 27 taps as the contraction index; it and the
//   16 -> 1 layer keep ~16 significant bits of their weights by splitting
//   them into a BF16 value and a BF16 remainder (for the last layer the two
//   are rows 0 and 1 of one weight matrix, so the split costs nothing).
// * Workgroups march through z by columns of the volume, so that a plane read
//   once serves three planes of output.
// * Weight gradients are contractions over all voxels, on MFMA as well: BF16
//   for the 16 -> 16 layer (FP64 beyond 64 voxels), FP64 where one factor is
//   FP32.  Per-workgroup FP64 partial sums, reduced in a fixed order
//   (deterministic for a device).
#include <math.h>

#include <map>
#include <mutex>
#include <type_traits>

#include "common.h"

namespace tomo {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef short bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kC = 16;
constexpr int kTaps = 27;
constexpr int OW1 = 0, OB1 = 432, OW2 = 448, OB2 = 7360, OW3 = 7376, OB3 = 7808;
static_assert(OB3 + 1 == TOMO_CONVNET_NPARAMS, "parameter layout");
constexpr int kWgBlocks = 512;  // most workgroups of the 16 -> 16 weight gradient (the workspace holds their sums)

// round to nearest even (gfx950 converts in one instruction)
__device__ inline uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

__device__ inline float bf2f(uint16_t h) { return __builtin_bit_cast(float, (uint32_t)h << 16); }

struct Vol {
    int32_t nx, ny, nz;
    int64_t n;
};

// optional device scale sqrt(*norm2) (norm2 == nullptr: 1)
__device__ inline float read_scale(const double *norm2)
{
    return norm2 ? (float)sqrt(*norm2) : 1.0f;
}

// ------------------------------------------------------------- forward

// Activations past the marching kernels' reach take the 16 -> 16 layer by
// output tiles of 16 x 4 x 4 voxels (one per workgroup, on a 3-D grid: no
// index division).  The tile's input region
// with its one-voxel halo (18 x 6 x 6) is staged in LDS once, zero outside
// the volume, and every tap reads LDS instead of re-gathering from L2.
// Wavefront w takes the four 16-voxel rows (y = 0..3, z = w) of the tile,
// interleaved so that four independent MFMA accumulations are in flight.
constexpr int kTX = 16, kTY = 4, kTZ = 4;
constexpr int kRX = kTX + 2, kRY = kTY + 2, kRZ = kTZ + 2, kRegion = kRX * kRY * kRZ;
static_assert(kTY == 4 && kTZ * 64 == kThreads, "one wavefront per tile z, four rows each");

// region entry of output voxel (lx, ly, lz) of the tile at tap t
__device__ inline int region_index(int lx, int ly, int lz, int t)
{
    return ((lz + t / 9) * kRY + (ly + (t / 3) % 3)) * kRX + lx + t % 3;
}

// Stages the [voxel][16] BF16 region of the tile at (x0, y0, z0) into LDS as
// two planes of kRegion 16-byte entries: plane h holds channels 8h..8h+7.
// Sixteen lanes reading one plane at sixteen consecutive voxels then cover
// 256 contiguous bytes (no bank conflicts).
__device__ inline void stage_channels(const uint16_t *__restrict__ src, const Vol &d, int x0, int y0, int z0,
                                      uint4 *lds)
{
    for (int e = threadIdx.x; e < kRegion * 2; e += kThreads) {
        const int rv = e >> 1, h = e & 1;
        const int ex = rv % kRX, ey = (rv / kRX) % kRY, ez = rv / (kRX * kRY);
        const int gx = x0 + ex - 1, gy = y0 + ey - 1, gz = z0 + ez - 1;
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (gx >= 0 && gx < d.nx && gy >= 0 && gy < d.ny && gz >= 0 && gz < d.nz)
            v = reinterpret_cast<const uint4 *>(src + (((int64_t)gz * d.ny + gy) * d.nx + gx) * kC)[h];
        lds[h * kRegion + rv] = v;
    }
}

// MFMA weight fragments.  v_mfma_f32_16x16x32_bf16 computes D(16x16) +=
// A(16x32) B(32x16) with lane l holding A[l % 16][8 (l / 16) + e] and
// B[8 (l / 16) + e][l % 16] (e = 0..7) and D[4 (l / 16) + r][l % 16] (r =
// 0..3); v_mfma_f32_16x16x16_bf16 has the same D with A[l % 16][4 (l / 16) +
// e], e = 0..3.  A 16 -> C layer contracts over (tap, input channel), the
// taps t = 9 dz + 3 dy + dx taken in x-triples q = 3 dz + dy (t = 3 q + dx):
// the K = 32 instruction of triple q has k = 16 dx + c for dx = 0, 1 (lane
// group g = l / 16 reads dx = g / 2 from LDS plane g % 2), the K = 16
// instruction has k = c for dx = 2 (lane group g reads channels 4g..4g+3).
// Fragment f of a set is the 64 bf16x8 entries [64 f, 64 f + 64): f = q
// for the K = 32 fragment of triple q, f = 9 + q for its K = 16 fragment
// (elements 0..3).
//   forward set, kFragFwd entries:
//   * fragments 0-17: the 16 -> 16 layer, A[cout][k] = W2[cout][c][tap];
//   * fragments 18-35: the 16 -> 1 layer, row 0 = bf16(W3[0][c][tap]), row 1 =
//     its remainder W3 - bf16(W3), rows 2-15 zero: output row 0 + row 1 is
//     the layer with ~16 significant bits of weight at no extra instruction;
//   * fragments 36-37: the 1 -> 16 layer with the 27 taps as k (27-31 zero),
//     A[cout][k] = bf16(W1[cout][k]) and its remainder.
//   transposed set (transpose = 1), kFragConv entries: the 16 -> 16 data
//   gradient, A[cin][k] = W2[c][cin][26 - tap] (taps flipped).
constexpr int kTriples = 9;
constexpr int kConvFrags = 2 * kTriples;
constexpr int kFragConv = kConvFrags * 64;
constexpr int kFrag3 = kFragConv, kFrag1 = 2 * kFragConv;
constexpr int kFragFwd = 2 * kFragConv + 2 * 64;

__global__ void k_conv_frags(const float *__restrict__ P, int transpose, bf16x8 *__restrict__ frag)
{
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (transpose ? kFragConv : kFragFwd)) return;
    const int f = idx / 64, lane = idx % 64;
    const int row = lane % 16, g = lane / 16;
    bf16x8 out;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        float w = 0.0f;
        if (transpose || f < 2 * kConvFrags) {
            const int ff = f % kConvFrags;
            const bool k16 = ff >= kTriples;
            const int q = k16 ? ff - kTriples : ff;
            const int tap = 3 * q + (k16 ? 2 : (g >> 1));
            const int c = k16 ? 4 * g + e : 8 * (g & 1) + e;
            if (k16 && e >= 4) {
                w = 0.0f;
            } else if (transpose) {
                w = P[OW2 + (c * kC + row) * kTaps + (kTaps - 1 - tap)];
            } else if (f < kConvFrags) {
                w = P[OW2 + (row * kC + c) * kTaps + tap];
            } else if (row < 2) {
                w = P[OW3 + c * kTaps + tap];
                if (row == 1) w -= bf2f(f2bf(w));
            }
        } else {
            const int tap = 8 * g + e;
            if (tap < kTaps) {
                w = P[OW1 + row * kTaps + tap];
                if (f == 2 * kConvFrags + 1) w -= bf2f(f2bf(w));
            }
        }
        out[e] = (short)f2bf(w);
    }
    frag[idx] = out;
}

// Per-lane LDS byte offsets of the B operands for output voxel (vl, 0, lz)
// of the tile and input row (y, z) = (0, lz) of the region: k32 for the
// dx = 0, 1 pair, k16 for dx = 2.  Input row (dy', dz') further adds
// (dz' kRY + dy') kRX entries (a compile-time immediate).
struct ConvOffsets {
    uint32_t k32;
    uint32_t k16;
};

__device__ inline ConvOffsets conv_offsets(int vl, int lz, int g)
{
    ConvOffsets o;
    o.k32 = (uint32_t)(((g & 1) * kRegion + region_index(vl, 0, lz, g >> 1)) * 16);
    o.k16 = (uint32_t)(((g >> 1) * kRegion + region_index(vl, 0, lz, 2)) * 16 + (g & 1) * 8);
    return o;
}

// acc[y] += sum over taps and channels of A x region, for the four output
// rows y of the wavefront; w, wt: the K = 32 and K = 16 fragments of the
// nine x-triples of a 16 -> C layer, in registers.  Per input plane dz the
// six input rows (region rows lz + dz, yi) are read once; output row y takes
// row y + dy through triple 3 dz + dy.  The four rows are interleaved, so
// three independent MFMA instructions separate two that update the same
// accumulator: an instruction then never reads as its accumulator input the
// result of one still in flight.
// The K = 32 part of x-triples 3 dz .. 3 dz + 2.
__device__ inline void conv_k32(const bf16x8 (&b32)[kRY], int dz, const bf16x8 (&w)[kTriples], f32x4 (&acc)[kTY])
{
#pragma unroll
    for (int dy = 0; dy < 3; ++dy) {
#pragma unroll
        for (int y = 0; y < kTY; ++y)
            acc[y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[3 * dz + dy], b32[y + dy], acc[y], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);  // keep the four-row interleave as written
    }
}

// The K = 16 part of the same triples.
__device__ inline void conv_k16(const bf16x4 (&b16)[kRY], int dz, const bf16x4 (&wt)[kTriples], f32x4 (&acc)[kTY])
{
#pragma unroll
    for (int dy = 0; dy < 3; ++dy) {
#pragma unroll
        for (int y = 0; y < kTY; ++y)
            acc[y] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(wt[3 * dz + dy], b16[y + dy], acc[y], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    }
}

__device__ inline void conv_rows(const char *rbytes, const ConvOffsets &o, const bf16x8 (&w)[kTriples],
                                 const bf16x4 (&wt)[kTriples], f32x4 (&acc)[kTY])
{
#pragma unroll
    for (int dz = 0; dz < 3; ++dz) {
        bf16x8 b32[kRY];
        bf16x4 b16[kRY];
#pragma unroll
        for (int yi = 0; yi < kRY; ++yi) {
            const uint32_t row = (uint32_t)((dz * kRY + yi) * kRX * 16);
            b32[yi] = *reinterpret_cast<const bf16x8 *>(rbytes + o.k32 + row);
            b16[yi] = *reinterpret_cast<const bf16x4 *>(rbytes + o.k16 + row);
        }
        conv_k32(b32, dz, w, acc);
        conv_k16(b16, dz, wt, acc);
    }
}

__device__ inline void load_conv_frags(const bf16x8 *__restrict__ frag, int lane, bf16x8 (&w)[kTriples],
                                       bf16x4 (&wt)[kTriples])
{
#pragma unroll
    for (int q = 0; q < kTriples; ++q) {
        w[q] = frag[q * 64 + lane];
        const bf16x8 t = frag[(kTriples + q) * 64 + lane];
        wt[q] = __builtin_shufflevector(t, t, 0, 1, 2, 3);
    }
}

// Epilogue of a 16 -> 16 layer for the tile at (x0, y0, z0): out =
// act(bias + acc) as BF16, act as for conv16_tile.
__device__ inline void conv16_store(const f32x4 (&acc)[kTY], const float (&b)[4], const Vol &d, int x0, int y0,
                                    int z0, int relu, const uint16_t *__restrict__ mask, uint16_t *__restrict__ out)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int vl = lane % 16, cg = 4 * (lane / 16);
    const int xo = x0 + vl, zo = z0 + wave;
#pragma unroll
    for (int y = 0; y < kTY; ++y) {
        const int yo = y0 + y;
        if (xo < d.nx && yo < d.ny && zo < d.nz) {
            const int64_t vo = ((int64_t)zo * d.ny + yo) * d.nx + xo;
            bf16x4 m = {1, 1, 1, 1};
            if (mask) m = *reinterpret_cast<const bf16x4 *>(mask + vo * kC + cg);
            bf16x4 ov;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float val = acc[y][r] + b[r];
                if (relu) val = fmaxf(val, 0.0f);
                if (mask && !(bf2f((uint16_t)m[r]) > 0.0f)) val = 0.0f;
                ov[r] = (short)f2bf(val);
            }
            *reinterpret_cast<bf16x4 *>(out + vo * kC + cg) = ov;
        }
    }
}

// Epilogue of the 16 -> 1 layer: out = s (b3 + row 0 + row 1), zero where
// the map mask is 0.
__device__ inline void conv3_store(const f32x4 (&acc)[kTY], float s, float b3, const Vol &d, int x0, int y0, int z0,
                                   const uint8_t *__restrict__ map_mask, float *__restrict__ out)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int xo = x0 + lane % 16, zo = z0 + wave;
#pragma unroll
    for (int y = 0; y < kTY; ++y) {
        const int yo = y0 + y;
        if (lane < 16 && xo < d.nx && yo < d.ny && zo < d.nz) {
            const int64_t vo = ((int64_t)zo * d.ny + yo) * d.nx + xo;
            float ov = s * ((acc[y][0] + acc[y][1]) + b3);
            if (map_mask && !map_mask[vo]) ov = 0.0f;
            out[vo] = ov;
        }
    }
}

// 16 -> 16 convolution of the tile at (x0, y0, z0) from its staged LDS
// region: fourteen MFMA instructions per 16-voxel row with the weights in
// registers.  out = act(bias + conv) where act is ReLU (relu = 1), or
// multiplication by [mask > 0] (mask != nullptr, the ReLU derivative of the
// layer below), or nothing.  Starts with the barrier that publishes the
// region.
__device__ inline void conv16_tile(const uint4 *region, const bf16x8 *__restrict__ frag,
                                   const float *__restrict__ bias, const Vol &d, int x0, int y0, int z0,
                                   int relu, const uint16_t *__restrict__ mask, uint16_t *__restrict__ out)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    bf16x8 w[kTriples];
    bf16x4 wt[kTriples];
    load_conv_frags(frag, lane, w, wt);
    const int vl = lane % 16, g = lane / 16, cg = 4 * g;
    const ConvOffsets o = conv_offsets(vl, wave, g);
    float b[4] = {0.f, 0.f, 0.f, 0.f};
    if (bias)
#pragma unroll
        for (int r = 0; r < 4; ++r) b[r] = bias[cg + r];
    __syncthreads();
    f32x4 acc[kTY];
#pragma unroll
    for (int y = 0; y < kTY; ++y) acc[y] = f32x4{0.f, 0.f, 0.f, 0.f};
    conv_rows(reinterpret_cast<const char *>(region), o, w, wt, acc);
    conv16_store(acc, b, d, x0, y0, z0, relu, mask, out);
}

// 16 -> 16 convolution of a stored activation (training forward, and the
// data gradient with the transposed fragments).
__global__ __launch_bounds__(kThreads) void k_conv16(const uint16_t *__restrict__ in,
                                                     const bf16x8 *__restrict__ frag,
                                                     const float *__restrict__ bias, Vol d,
                                                     int relu, const uint16_t *__restrict__ mask,
                                                     uint16_t *__restrict__ out,
                                                     const int *__restrict__ skip)
{
    __shared__ uint4 region[kRegion * 2];
    if (skip && *skip) return;
    const int x0 = blockIdx.x * kTX, y0 = blockIdx.y * kTY, z0 = blockIdx.z * kTZ;
    stage_channels(in, d, x0, y0, z0, region);
    conv16_tile(region, frag, bias, d, x0, y0, z0, relu, mask, out);
}

// layer 3: out[v] = s * (b3 + sum_{c,t} w3[c][t] a2[v + t - 1][c]), zero
// where the map mask is 0.  On MFMA like the 16 -> 16 layer with the 1 x 16
// weight row as rows 0 (BF16 value) and 1 (BF16 remainder) of a 16 x 16
// matrix: D rows 0 and 1 land in lanes 0-15, elements 0 and 1.
__global__ __launch_bounds__(kThreads) void k_conv3(const bf16x8 *__restrict__ frag3,
                                                    const float *__restrict__ P,
                                                    const uint16_t *__restrict__ a2, Vol d,
                                                    const double *__restrict__ norm2,
                                                    const uint8_t *__restrict__ map_mask,
                                                    float *__restrict__ out,
                                                    const int *__restrict__ skip)
{
    __shared__ uint4 region[kRegion * 2];
    if (skip && *skip) return;
    const float s = read_scale(norm2);
    const int x0 = blockIdx.x * kTX, y0 = blockIdx.y * kTY, z0 = blockIdx.z * kTZ;
    stage_channels(a2, d, x0, y0, z0, region);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    bf16x8 w[kTriples];
    bf16x4 wt[kTriples];
    load_conv_frags(frag3, lane, w, wt);
    const int vl = lane % 16, g = lane / 16;
    const ConvOffsets o = conv_offsets(vl, wave, g);
    const float b3 = P[OB3];
    __syncthreads();
    f32x4 acc[kTY];
#pragma unroll
    for (int y = 0; y < kTY; ++y) acc[y] = f32x4{0.f, 0.f, 0.f, 0.f};
    conv_rows(reinterpret_cast<const char *>(region), o, w, wt, acc);
    conv3_store(acc, s, b3, d, x0, y0, z0, map_mask, out);
}

// ---- marching kernels: a workgroup owns a column of the volume over x and y
// and walks z plane by plane, so that a plane is read for the three planes of
// output it feeds while it is in LDS (or registers) instead of once per tile
// above and below: 1.27 reads per input voxel of a 16 x 16 column (plus two
// planes per workgroup) against 2.53 for 16 x 4 x 4 tiles.

// A marching launch: `items` runs of at most cz planes in the columns.  One
// workgroup per item, or (the weight gradients, whose per-workgroup sums have a
// limited place) items taken in turn.
struct March {
    int32_t ncx, ncy, cz;  // columns along x and y, planes per item
    int32_t items;
    int32_t by_column, inner;  // the order of the items (march_place), and how many share its outer index
};

// First item of this workgroup: neighbouring items on one XCD.
__device__ inline int march_first() { return (int)xcd_remap(blockIdx.x, gridDim.x); }

// Item's column (cx, cy) and planes [z0, z1).  Workgroups of an XCD take
// neighbouring items, and read the planes beside their own from its L2: a
// column's runs follow each other where there are more columns than planes,
// else the columns of one run do (forward, us, against the other order:
// 4x256x256 25.8 and 30.7, 6x128x128 19.2 and 22.7, 20x150x150 38.6 and 39.3;
// 100x33x17 20.9 and 22.0, 33^3 18.6 and 19.1).
__device__ inline void march_place(const March &m, const Vol &d, int item, int &cx, int &cy, int &z0, int &z1)
{
    const int q = item / m.inner, rest = item - q * m.inner;
    const int run = m.by_column ? rest : q, col = m.by_column ? q : rest;
    cy = col / m.ncx;
    cx = col - cy * m.ncx;
    z0 = run * m.cz;
    z1 = min(z0 + m.cz, d.nz);
}

constexpr int kZX = 16, kZY = 16, kZR = kZX + 2;  // a column's outputs; columns of its input plane
static_assert(kZY == 4 * (kThreads / 64), "four rows per wavefront");

// Largest activation the marching 16 -> 16 kernel addresses through one buffer
// resource (offsets below the out-of-range marker).
constexpr int64_t kMaxMarchVoxels = ((int64_t)1 << 27) - 1;

// A layer of 16 input channels by 16 x 16 columns.  Four input planes live in LDS (two
// 16-byte halves per voxel, as in stage_channels): three feed the current
// output plane while the fourth arrives by direct-to-LDS buffer loads, whose
// out-of-range offsets (voxels outside the volume) read zeros.  Each wavefront
// computes four rows per plane with conv_rows' arithmetic and order, and
// stores them after the next plane's barrier, so that the wait for the
// arriving plane never waits for a fresh store.
// 128^3: layer 2 34.2 us (40.7 with persistent 16 x 4 x 4 tiles, 2.53 reads per
// input voxel), its data gradient 39.1 (61.3), layer 3 30.4 (37.1).  The MFMA
// pipe is busy for 15 us of each and LDS reads take as long, in phases that
// the three workgroups of a CU overlap in part (35.9 and 32.4 before the reads
// were issued one group of products ahead; a whole plane ahead costs the
// third workgroup its registers and wins nothing).
// kWaves: four wavefronts on 16 rows, or two on 8 (half_columns).
// kMode: what the products become.
//   kForward: out = ReLU(bias + conv);
//   kMasked: out = conv where mask > 0, else 0 (the data gradient through the
//     ReLU below);
//   kLast: the 16 -> 1 layer, whose weights are rows 0 (BF16 value) and 1 (BF16
//     remainder) of the matrix: zout = s (bias + row 0 + row 1), s =
//     sqrt(*norm2) (or 1), zero where map_mask is 0.
enum { kForward = 0, kMasked = 1, kLast = 2 };
struct LastOut {
    float *zout;
    const double *norm2;
    const uint8_t *map_mask;
};
template <int kMode, int kWaves>
__global__ __launch_bounds__(kWaves * 64) void k_conv16z(const uint16_t *__restrict__ in,
                                                      const bf16x8 *__restrict__ frag,
                                                      const float *__restrict__ bias, Vol d, March m,
                                                      const uint16_t *__restrict__ mask,
                                                      uint16_t *__restrict__ out, LastOut last,
                                                      const int *__restrict__ skip)
{
    constexpr int kRows = 4 * kWaves, kZPlane = kZR * (kRows + 2);  // output rows; input voxels of a plane
    constexpr int kZLoads = (2 * kZPlane + kWaves * 64 - 1) / (kWaves * 64);
    __shared__ uint4 buf[4][2 * kZPlane];
    if (skip && *skip) return;
    int cx, cy, z0, z1;
    march_place(m, d, march_first(), cx, cy, z0, z1);
    const int x0 = cx * kZX, y0 = cy * kRows;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const auto rs = make_rsrc(in, (uint32_t)(d.n * kC * 2));
    const uint32_t plane_bytes = (uint32_t)(d.nx * d.ny) * (kC * 2);
    // this lane's in-plane offsets of the staging loads (or the marker)
    constexpr uint32_t kOut = 0xFFFFFFF0u;
    uint32_t poff[kZLoads];
#pragma unroll
    for (int u = 0; u < kZLoads; ++u) {
        const int sl = (u * kWaves + wave) * 64 + lane;
        const int h = sl >= kZPlane ? 1 : 0, rv = sl - h * kZPlane;
        const int gx = x0 + rv % kZR - 1, gy = y0 + rv / kZR - 1;
        const bool ok = sl < 2 * kZPlane && gx >= 0 && gx < d.nx && gy >= 0 && gy < d.ny;
        poff[u] = ok ? (uint32_t)(gy * d.nx + gx) * (kC * 2) + h * 16 : kOut;
    }
    auto stage = [&](int z) {
        const bool zin = z >= 0 && z < d.nz;
        const uint32_t zo = zin ? (uint32_t)z * plane_bytes : 0u;
#pragma unroll
        for (int u = 0; u < kZLoads; ++u) {
            const int c = u * kWaves + wave;
            if (c * 64 + lane < 2 * kZPlane) {
                const uint32_t off = zin && poff[u] != kOut ? poff[u] + zo : kOut;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(
                    rs, (__attribute__((address_space(3))) void *)(&buf[z & 3][c * 64]), 16, (int)off, 0, 0, 0);
            }
        }
    };
    bf16x8 w[kTriples];
    bf16x4 wt[kTriples];
    load_conv_frags(frag, lane, w, wt);
    const int vl = lane % 16, g = lane / 16, cg = 4 * g;
    f32x4 b = {0.f, 0.f, 0.f, 0.f};
    if constexpr (kMode == kForward) b = f32x4{bias[cg], bias[cg + 1], bias[cg + 2], bias[cg + 3]};
    const float scale = kMode == kLast ? read_scale(last.norm2) : 1.0f, b3 = kMode == kLast ? bias[0] : 0.0f;
    // byte offsets of the B operands for input row 4 * wave of a plane
    const uint32_t o32 = (uint32_t)(((g & 1) * kZPlane + 4 * wave * kZR + vl + (g >> 1)) * 16);
    const uint32_t o16 = (uint32_t)(((g >> 1) * kZPlane + 4 * wave * kZR + vl + 2) * 16 + (g & 1) * 8);
    const int xo = x0 + vl;
    bf16x4 res[kTY];
    float res3[kTY];
    auto store = [&](int z) {
#pragma unroll
        for (int y = 0; y < kTY; ++y) {
            const int yo = y0 + 4 * wave + y;
            if (xo >= d.nx || yo >= d.ny) continue;
            const int64_t vo = ((int64_t)z * d.ny + yo) * d.nx + xo;
            if constexpr (kMode != kLast) {
                *reinterpret_cast<bf16x4 *>(out + vo * kC + cg) = res[y];
            } else if (lane < 16) {
                last.zout[vo] = last.map_mask && !last.map_mask[vo] ? 0.0f : res3[y];
            }
        }
    };
    stage(z0 - 1);
    stage(z0);
    stage(z0 + 1);
    for (int z = z0; z < z1; ++z) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();  // planes z-1..z+1 published; every wave past the plane whose buffer is staged next
        if (z > z0) store(z - 1);
        bf16x4 mk[kTY];
        if constexpr (kMode == kMasked)
#pragma unroll
            for (int y = 0; y < kTY; ++y) {
                const int yo = y0 + 4 * wave + y;
                mk[y] = bf16x4{0, 0, 0, 0};
                if (xo < d.nx && yo < d.ny)
                    mk[y] = *reinterpret_cast<const bf16x4 *>(mask + (((int64_t)z * d.ny + yo) * d.nx + xo) * kC + cg);
            }
        if (z + 2 <= z1) stage(z + 2);
        f32x4 acc[kTY];
#pragma unroll
        for (int y = 0; y < kTY; ++y) acc[y] = f32x4{0.f, 0.f, 0.f, 0.f};
        // operands are read one group ahead: a plane's K = 16 operands under its
        // K = 32 products, the next plane's K = 32 operands under the K = 16 ones
        bf16x8 b32[kRY];
        bf16x4 b16[kRY];
        auto rows = [&](int dz) { return reinterpret_cast<const char *>(buf[(z - 1 + dz) & 3]); };
        auto fetch32 = [&](const char *rb) {
#pragma unroll
            for (int yi = 0; yi < kRY; ++yi) b32[yi] = *reinterpret_cast<const bf16x8 *>(rb + o32 + yi * kZR * 16);
        };
        fetch32(rows(0));
#pragma unroll
        for (int dz = 0; dz < 3; ++dz) {
            const char *rb = rows(dz);
#pragma unroll
            for (int yi = 0; yi < kRY; ++yi) b16[yi] = *reinterpret_cast<const bf16x4 *>(rb + o16 + yi * kZR * 16);
            __builtin_amdgcn_sched_barrier(0);
            conv_k32(b32, dz, w, acc);
            if (dz < 2) fetch32(rows(dz + 1));
            __builtin_amdgcn_sched_barrier(0);
            conv_k16(b16, dz, wt, acc);
        }
#pragma unroll
        for (int y = 0; y < kTY; ++y) {
            if constexpr (kMode == kLast) {
                res3[y] = scale * ((acc[y][0] + acc[y][1]) + b3);
                continue;
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float val = acc[y][r];
                if constexpr (kMode == kMasked) val = bf2f((uint16_t)mk[y][r]) > 0.0f ? val : 0.0f;
                else val = fmaxf(val + b[r], 0.0f);
                res[y][r] = (short)f2bf(val);
            }
        }
    }
    store(z1 - 1);
}

// layer 1: a1[v][c] = relu(b1[c] + sum_t w1[c][t] x[v + t - 1] / s), on MFMA
// with the taps as the contraction index (k = tap, 27-31 with zero weight), by
// 16 x 16 columns.  Weights and inputs are each split into a BF16 value and a
// BF16 remainder, and the three products that matter (hi hi, hi lo, lo hi) keep
// ~16 significant bits: three v_mfma_f32_16x16x32_bf16 per 16-voxel row.  The
// scaled and split input planes go through an LDS ring of four.  A plane's values are loaded into
// registers two planes ahead of their use, so the loop waits for no fresh load.
// The ring turns with z: a lane's eight tap offsets are kept for its four
// positions, and the loop body holds four planes.
// 128^3: 21.7 us (29.8 with one 16 x 4 x 4 tile per workgroup, each tap's input
// split where it was read); writing a1 alone takes about 10 us.
template <int kWaves>
__global__ __launch_bounds__(kWaves * 64) void k_conv1z(const bf16x8 *__restrict__ frag1, const float *__restrict__ P,
                                                     const float *__restrict__ x, Vol d, March m,
                                                     const double *__restrict__ norm2, uint16_t *__restrict__ a1,
                                                     const int *__restrict__ skip)
{
    constexpr int kLanes = kWaves * 64, kRows = 4 * kWaves, kZPlane = kZR * (kRows + 2);
    constexpr int kZ1Loads = (kZPlane + kLanes - 1) / kLanes;
    __shared__ uint32_t xs[4][kZPlane];
    if (skip && *skip) return;
    int cx, cy, z0, z1;
    march_place(m, d, march_first(), cx, cy, z0, z1);
    const float s = read_scale(norm2);
    const float inv = s > 0.0f ? 1.0f / s : 0.0f;
    const int x0 = cx * kZX, y0 = cy * kRows;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int64_t poff[kZ1Loads];  // in-plane offset of this thread's staged voxels (-1: outside)
#pragma unroll
    for (int u = 0; u < kZ1Loads; ++u) {
        const int e = u * kLanes + threadIdx.x;
        const int gx = x0 + e % kZR - 1, gy = y0 + e / kZR - 1;
        poff[u] = e < kZPlane && gx >= 0 && gx < d.nx && gy >= 0 && gy < d.ny ? (int64_t)gy * d.nx + gx : -1;
    }
    const int64_t plane = (int64_t)d.nx * d.ny;
    auto load = [&](int z, float (&v)[kZ1Loads]) {
#pragma unroll
        for (int u = 0; u < kZ1Loads; ++u) {
            v[u] = 0.0f;
            if (z >= 0 && z < d.nz && poff[u] >= 0) v[u] = x[(int64_t)z * plane + poff[u]];
        }
    };
    auto put = [&](int slot, const float (&v)[kZ1Loads]) {
#pragma clang fp contract(off)  // the remainder is that of the rounded product
#pragma unroll
        for (int u = 0; u < kZ1Loads; ++u) {
            const int e = u * kLanes + threadIdx.x;
            const float t = v[u] * inv;
            const uint16_t h = f2bf(t);
            if (e < kZPlane) xs[slot][e] = (uint32_t)h << 16 | f2bf(t - bf2f(h));
        }
    };
    const bf16x8 wh = frag1[lane], wl = frag1[64 + lane];
    const int vl = lane % 16, g = lane / 16, cg = 4 * g;
    // word offsets of taps 8g..8g+7 for output row 4 * wave when plane z - 1
    // sits in ring slot ph; taps past 26 read tap 26 (zero weight)
    int off[4][8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int t = min(8 * g + e, kTaps - 1);
#pragma unroll
        for (int ph = 0; ph < 4; ++ph)
            off[ph][e] = ((ph + t / 9) & 3) * kZPlane + (4 * wave + (t / 3) % 3) * kZR + vl + t % 3;
    }
    float b[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) b[r] = P[OB1 + cg + r];
    const uint32_t *ring = &xs[0][0];
    const int xo = x0 + vl;
    float v0[kZ1Loads], v1[kZ1Loads];
    // planes z0 - 1 and z0 go to slots 0 and 1; z0 + 1 and z0 + 2 follow in the loop
    load(z0 - 1, v0);
    load(z0, v1);
    put(0, v0);
    put(1, v1);
    load(z0 + 1, v0);
    load(z0 + 2, v1);
    auto step = [&](auto phase, int z, float (&v)[kZ1Loads]) {
        constexpr int ph = decltype(phase)::value;
        put((ph + 2) & 3, v);  // plane z + 1: its slot held plane z - 3
        __syncthreads();       // (every wave is past plane z - 1's products, which read no other slot)
        load(z + 3, v);
#pragma unroll
        for (int y = 0; y < kTY; ++y) {
            uint32_t hi[4], lo[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t p = ring[off[ph][2 * e] + y * kZR], q = ring[off[ph][2 * e + 1] + y * kZR];
                hi[e] = __builtin_amdgcn_perm(q, p, 0x07060302u);
                lo[e] = __builtin_amdgcn_perm(q, p, 0x05040100u);
            }
            const bf16x8 xh = __builtin_bit_cast(bf16x8, hi), xl = __builtin_bit_cast(bf16x8, lo);
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wh, xh, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wh, xl, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wl, xh, acc, 0, 0, 0);
            const int yo = y0 + 4 * wave + y;
            if (xo < d.nx && yo < d.ny) {
                bf16x4 o;
#pragma unroll
                for (int r = 0; r < 4; ++r) o[r] = (short)f2bf(fmaxf(acc[r] + b[r], 0.0f));
                *reinterpret_cast<bf16x4 *>(a1 + (((int64_t)z * d.ny + yo) * d.nx + xo) * kC + cg) = o;
            }
        }
    };
    for (int z = z0;; z += 4) {
        step(std::integral_constant<int, 0>{}, z, v0);
        if (z + 1 >= z1) break;
        step(std::integral_constant<int, 1>{}, z + 1, v1);
        if (z + 2 >= z1) break;
        step(std::integral_constant<int, 2>{}, z + 2, v0);
        if (z + 3 >= z1) break;
        step(std::integral_constant<int, 3>{}, z + 3, v1);
        if (z + 4 >= z1) break;
    }
}

// ------------------------------------------------------------ training

// g[v] = 2 (out[v] - target[v]) / n; loss = mean((out - target)^2) (FP64).
__global__ __launch_bounds__(kThreads) void k_mse(const float *__restrict__ out,
                                                  const float *__restrict__ target, int64_t n,
                                                  float *__restrict__ g, double *__restrict__ partial)
{
    __shared__ double lds[4];
    double acc = 0.0;
    const float sc = 2.0f / (float)n;
    for (int64_t v = (int64_t)blockIdx.x * kThreads + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * kThreads) {
        const float e = out[v] - target[v];
        g[v] = sc * e;
        acc += (double)e * e;
    }
    const double s = block_sum(acc, lds);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// ---- marching training kernels: workgroups own columns of the volume over x
// and y and walk z, with the planes they need in LDS rings (as the layers do).

// Stages planes of a float field over a column of W x H voxels plus a one-voxel
// rim into an LDS ring of four: load() reads plane z into registers (zero
// outside the volume), put() stores it.
template <int W, int H, int NT>
struct FieldRing {
    static constexpr int R = W + 2, N = R * (H + 2), kLoads = (N + NT - 1) / NT;
    int64_t off[kLoads];  // in-plane offset of this thread's voxels (-1: outside)
    __device__ void init(const Vol &d, int x0, int y0)
    {
#pragma unroll
        for (int u = 0; u < kLoads; ++u) {
            const int e = u * NT + threadIdx.x;
            const int gx = x0 + e % R - 1, gy = y0 + e / R - 1;
            off[u] = e < N && gx >= 0 && gx < d.nx && gy >= 0 && gy < d.ny ? (int64_t)gy * d.nx + gx : -1;
        }
    }
    __device__ void load(const float *__restrict__ f, const Vol &d, int z, float (&v)[kLoads]) const
    {
#pragma unroll
        for (int u = 0; u < kLoads; ++u) {
            v[u] = 0.0f;
            if (z >= 0 && z < d.nz && off[u] >= 0) v[u] = f[(int64_t)z * d.nx * d.ny + off[u]];
        }
    }
    __device__ void put(float *plane, const float (&v)[kLoads]) const
    {
#pragma unroll
        for (int u = 0; u < kLoads; ++u) {
            const int e = u * NT + threadIdx.x;
            if (e < N) plane[e] = v[u];
        }
    }
};

// g_h2[v][c] = [a2[v][c] > 0] * sum_t w3[c][t] g[v - t + 1]  (data gradient of
// layer 3), FP32 sums over t in order.  Columns of 64 x 16: a thread takes four
// rows at one x, so that a weight (a scalar register) serves four products and
// each LDS value up to three rows.  Bound by its 432 FMAs per voxel (46 us at
// one per lane and clock): 107 -> 55 us at 128^3 (one voxel per thread from
// global memory before).  All 432 weights in registers at once spill (66 us from
// LDS instead), and a store per dword rather than per 16 bytes takes 183 us.
constexpr int kBX = 64, kBY = 16;
__global__ __launch_bounds__(kThreads) void k_conv3_bwd(const float *__restrict__ P, const float *__restrict__ g,
                                                        const uint16_t *__restrict__ a2, Vol d, March m,
                                                        uint16_t *__restrict__ gh2)
{
    using Ring = FieldRing<kBX, kBY, kThreads>;
    __shared__ float gs[4][Ring::N];
    typedef const __attribute__((address_space(4))) float weight;  // scalar loads
    weight *pw = reinterpret_cast<weight *>(reinterpret_cast<uintptr_t>(P + OW3));
    int cx, cy, z0, z1;
    march_place(m, d, march_first(), cx, cy, z0, z1);
    const int x0 = cx * kBX, y0 = cy * kBY;
    const int tx = threadIdx.x & 63, ty = 4 * (threadIdx.x >> 6);
    const int xo = x0 + tx;
    Ring ring;
    ring.init(d, x0, y0);
    float v[Ring::kLoads];
    for (int k = -1; k <= 0; ++k) {
        ring.load(g, d, z0 + k, v);
        ring.put(gs[(z0 + k) & 3], v);
    }
    ring.load(g, d, z0 + 1, v);
    for (int z = z0; z < z1; ++z) {
        ring.put(gs[(z + 1) & 3], v);
        __syncthreads();
        if (z + 1 < z1) ring.load(g, d, z + 2, v);
        // gin[dz][y][dx] = g at (x + dx - 1, y - 1, z + dz - 1) of the thread's column
        float gin[3][kTY + 2][3];
#pragma unroll
        for (int dz = 0; dz < 3; ++dz)
#pragma unroll
            for (int y = 0; y < kTY + 2; ++y)
#pragma unroll
                for (int dx = 0; dx < 3; ++dx)
                    gin[dz][y][dx] = gs[(z - 1 + dz) & 3][(ty + y) * Ring::R + tx + dx];
        // two channels at a time, in a loop of their own: 54 of the 432 weights
        // fit the scalar registers (all at once were spilled: 107 us).  The mask
        // and the results turn through four dwords, so that both move 16 bytes
        const int64_t vo = ((int64_t)z * d.ny + y0 + ty) * d.nx + xo;
        weight *pc = pw;
        uint4 mk[kTY], res[kTY];
#pragma unroll
        for (int y = 0; y < kTY; ++y) mk[y] = res[y] = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll 1
        for (int i = 0; i < kC / 2; ++i, pc += 2 * kTaps) {
            if ((i & 3) == 0) {
#pragma unroll
                for (int y = 0; y < kTY; ++y) {
                    mk[y] = make_uint4(0u, 0u, 0u, 0u);
                    if (xo < d.nx && y0 + ty + y < d.ny)
                        mk[y] = reinterpret_cast<const uint4 *>(a2 + (vo + (int64_t)y * d.nx) * kC)[i >> 2];
                }
            }
            float s0[kTY], s1[kTY];
#pragma unroll
            for (int y = 0; y < kTY; ++y) s0[y] = s1[y] = 0.f;
#pragma unroll
            for (int t = 0; t < kTaps; ++t) {  // output voxel v - (t - 1) used input v at tap t
                const float w0 = pc[t], w1 = pc[kTaps + t];
#pragma unroll
                for (int y = 0; y < kTY; ++y) {
                    const float gv = gin[2 - t / 9][y + 2 - (t / 3) % 3][2 - t % 3];
                    s0[y] = fmaf(w0, gv, s0[y]);
                    s1[y] = fmaf(w1, gv, s1[y]);
                }
            }
#pragma unroll
            for (int y = 0; y < kTY; ++y) {
                const uint32_t lo = f2bf(bf2f((uint16_t)(mk[y].x & 0xffffu)) > 0.f ? s0[y] : 0.f);
                const uint32_t hi = f2bf(bf2f((uint16_t)(mk[y].x >> 16)) > 0.f ? s1[y] : 0.f);
                mk[y] = make_uint4(mk[y].y, mk[y].z, mk[y].w, 0u);
                res[y] = make_uint4(res[y].y, res[y].z, res[y].w, lo | hi << 16);
            }
            if ((i & 3) == 3) {
#pragma unroll
                for (int y = 0; y < kTY; ++y)
                    if (xo < d.nx && y0 + ty + y < d.ny)
                        reinterpret_cast<uint4 *>(gh2 + (vo + (int64_t)y * d.nx) * kC)[i >> 2] = res[y];
            }
        }
    }
}

// Weight gradients of the layers with one channel on one side, per-workgroup
// partial sums in FP64 on v_mfma_f64_16x16x4_f64 (products of a BF16 and an
// FP32 value are exact in FP64): D[c][t] += act[v][c] field[v + o_t], four
// voxels per instruction, the 27 taps as the columns of two tiles.
//   kFirst: gw1[c][t] = sum_v gh1[v][c] x[v + t - 1], gb1[c] = sum_v gh1[v][c]
//     (the column after the taps: a field of ones); part rows of 448:
//     [16][27] then [16].
//   otherwise: gw3[c][t] = sum_u a2[u][c] g[u - (t - 1)] (the same sum over
//     input voxels), gb3 = sum_v g[v]; part rows of 433: [16][27] then 1.
// Lane l holds act[v + l / 16][l % 16], field[v + l / 16 + o_t] for t = l % 16
// (and 16 + l % 16), and rows 4 r + l / 16, r = 0..3, of column l % 16 of the
// result.  Columns of 16 x 16, a wavefront taking four rows of each plane.
// Bound by the FP64 matrix rate (27 us of products at 128^3): 3435 -> 44 us
// (first layer) and 2627 -> 44 us there (one thread per output element before).
constexpr int kFPart1 = 448, kFPart3 = 433;
constexpr int kFieldBlocks = 4096;  // most workgroups
template <bool kFirst>
__global__ __launch_bounds__(kThreads) void k_wgrad_field(const uint16_t *__restrict__ act,
                                                          const float *__restrict__ field, Vol d, March m,
                                                          double *__restrict__ part)
{
    typedef double f64x4 __attribute__((ext_vector_type(4)));
    using Ring = FieldRing<kZX, kZY, kThreads>;
    __shared__ float fs[4][Ring::N];
    __shared__ uint4 as[2][kZX * kZY * 2];  // two planes of act: [voxel][16] BF16
    __shared__ double red[kThreads / 64][8][64];
    __shared__ double gsum[kThreads / 64];
    constexpr int kWidth = kFirst ? kFPart1 : kFPart3;
    double *dst = part + (int64_t)blockIdx.x * kWidth;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane % 16, k = lane / 16;
    // word offsets of this lane's two taps for voxel (k, 4 wave) when plane
    // z - 1 sits in ring slot ph
    int off[4][2];
    const int t1 = min(16 + n, kTaps - 1);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int tt = j == 0 ? n : t1, t = kFirst ? tt : kTaps - 1 - tt;
#pragma unroll
        for (int ph = 0; ph < 4; ++ph)
            off[ph][j] = ((ph + t / 9) & 3) * Ring::N + (4 * wave + (t / 3) % 3) * Ring::R + k + t % 3;
    }
    const bool live1 = 16 + n < kTaps;                       // tile 1: taps 16..26,
    const double rest = kFirst && 16 + n == kTaps ? 1.0 : 0.0;  // ones after them, then zeros
    f64x4 acc[2][2];  // [voxel parity][tile]: independent products back to back
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f64x4{0., 0., 0., 0.};
    double gb = 0.0;
    const float *fw = &fs[0][0];
    for (int it = march_first(); it < m.items; it += gridDim.x) {
        int cx, cy, z0, z1;
        march_place(m, d, it, cx, cy, z0, z1);
        const int x0 = cx * kZX, y0 = cy * kZY;
        Ring ring;
        ring.init(d, x0, y0);
        // act voxel of this thread: slots 2 v and 2 v + 1, v = threadIdx.x
        const bool ain = x0 + (int)(threadIdx.x & 15) < d.nx && y0 + (int)(threadIdx.x >> 4) < d.ny;
        const int64_t aoff = ((int64_t)(y0 + (threadIdx.x >> 4)) * d.nx + x0 + (threadIdx.x & 15)) * kC;
        float v[Ring::kLoads];
        uint4 av[2];
        auto load_act = [&](int z) {
            av[0] = av[1] = make_uint4(0u, 0u, 0u, 0u);
            if (ain) {
                const uint4 *p = reinterpret_cast<const uint4 *>(act + (int64_t)z * d.nx * d.ny * kC + aoff);
                av[0] = p[0];
                av[1] = p[1];
            }
        };
        __syncthreads();  // the previous item's planes are done with
        ring.load(field, d, z0 - 1, v);
        ring.put(fs[0], v);
        ring.load(field, d, z0, v);
        ring.put(fs[1], v);
        ring.load(field, d, z0 + 1, v);
        load_act(z0);
        auto step = [&](auto phase, int z) {
            constexpr int ph = decltype(phase)::value;
            ring.put(fs[(ph + 2) & 3], v);
            as[ph & 1][2 * threadIdx.x] = av[0];
            as[ph & 1][2 * threadIdx.x + 1] = av[1];
            __syncthreads();
            if (z + 1 < z1) {
                ring.load(field, d, z + 2, v);
                load_act(z + 1);
            }
            const uint16_t *ap = reinterpret_cast<const uint16_t *>(as[ph & 1]) + ((4 * wave * kZX + k) * kC + n);
#pragma unroll
            for (int y = 0; y < 4; ++y)
#pragma unroll
                for (int q = 0; q < kZX / 4; ++q) {
                    const double a = (double)bf2f(ap[(y * kZX + 4 * q) * kC]);
                    const double b0 = (double)fw[off[ph][0] + y * Ring::R + 4 * q];
                    const double f1 = (double)fw[off[ph][1] + y * Ring::R + 4 * q];
                    const double b1 = live1 ? f1 : rest;
                    acc[q & 1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b0, acc[q & 1][0], 0, 0, 0);
                    acc[q & 1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b1, acc[q & 1][1], 0, 0, 0);
                }
            if (!kFirst)  // this thread's own voxel (zero outside the volume)
                gb += (double)fs[(ph + 1) & 3][((threadIdx.x >> 4) + 1) * Ring::R + (threadIdx.x & 15) + 1];
        };
        for (int z = z0;; z += 4) {
            step(std::integral_constant<int, 0>{}, z);
            if (z + 1 >= z1) break;
            step(std::integral_constant<int, 1>{}, z + 1);
            if (z + 2 >= z1) break;
            step(std::integral_constant<int, 2>{}, z + 2);
            if (z + 3 >= z1) break;
            step(std::integral_constant<int, 3>{}, z + 3);
            if (z + 4 >= z1) break;
        }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wave][4 * j + r][lane] = acc[0][j][r] + acc[1][j][r];
    if (!kFirst) {
        for (int o = 32; o > 0; o >>= 1) gb += __shfl_down(gb, o, 64);
        if (lane == 0) gsum[wave] = gb;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 512; e += kThreads) {
        const int q = e >> 6, l = e & 63;
        const double sum = (red[0][q][l] + red[1][q][l]) + (red[2][q][l] + red[3][q][l]);
        const int c = 4 * (q & 3) + l / 16, t = 16 * (q >> 2) + l % 16;
        if (t < kTaps) dst[c * kTaps + t] = sum;
        else if (kFirst && t == kTaps) dst[16 * kTaps + c] = sum;
    }
    if (!kFirst && threadIdx.x == 0) dst[16 * kTaps] = (gsum[0] + gsum[1]) + (gsum[2] + gsum[3]);
}

// Per-workgroup partial sums of the 16 -> 16 weight gradient on MFMA:
// gw2[co][ci][t] = sum_v gh2[v][co] a1[v + t - 1][ci]; gb2[co] = sum_v gh2[v][co].
// The contraction runs over voxels, 32 along x per v_mfma_f32_16x16x32_bf16
// (BF16 products are exact in FP32), so both operands are staged with voxels
// along a lane's elements: LDS rows [channel][x].  Columns of 32 x 8; nine
// wavefronts, one per x-triple of taps, each over the plane's eight rows: its
// three sums are FP32 over two instructions (64 voxels) and FP64 beyond.  A
// tap's shift along x is taken in registers from the five dwords around the
// lane's eight voxels (dx = 1: a 16-bit funnel shift).  The bias sums in FP64
// throughout, a row per wavefront.  Bound by VALU (the FP64 folds) and LDS
// reads, about 18 us each, next to 12 us of products at 128^3, and by one
// workgroup per CU (134 registers; held to 96 for two, 35 spill): 9650 -> 69
// us there (one thread per output before, its products in FP32 over 64 voxels and
// FP64 beyond as well).  Against FP64 sums of the same factors the gradient is
// off by 3.3e-8 of its norm at 48^3 and 3.5e-8 at 96x100x90 (4.2e-8 before), its
// rounding to FP32 included.
constexpr int kWX = 32, kWY = 8, kWThreads = 576, kWPart = 6928;
constexpr int kWRow = 20;                           // dwords per [channel] row: 36 voxels, padded off the banks
constexpr int kWA1 = (kWY + 2) * kC * kWRow;        // dwords of an a1 plane: [row][channel][x + 1]
constexpr int kWGh = kWY * kC * kWRow;              // dwords of a gh2 plane: [row][channel][x]
static_assert(kWThreads == kTriples * 64 && kWY <= kTriples, "a wavefront per x-triple, a bias row per wavefront");
__global__ __launch_bounds__(kWThreads) void k_wgrad2(const uint16_t *__restrict__ gh2,
                                                      const uint16_t *__restrict__ a1, Vol d, March m,
                                                      double *__restrict__ part)
{
    __shared__ __align__(16) uint32_t sa[4][kWA1];
    __shared__ __align__(16) uint32_t sg[2][kWGh];
    __shared__ double bred[kWY][64];
    double *dst = part + (int64_t)blockIdx.x * kWPart;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int dz = wave / 3, dy = wave % 3;
    const int n = lane % 16, g = lane / 16;
    // staging: a share is a pair of x neighbours and half of their channels,
    // two 16-byte loads transposed into eight dwords (one per channel)
    constexpr int kSharesA = (kWY + 2) * (kWX / 2 + 1) * 2;  // pairs x = -1 .. 32
    constexpr int kSharesG = kWY * (kWX / 2) * 2;            // taken by the last threads
    static_assert(kSharesA <= kWThreads && kSharesG <= kWThreads, "one share per thread");
    struct Share {
        int64_t off;   // of the pair's first voxel in a plane, in elements
        bool in0, in1; // voxels inside the volume
        int lds;       // dword of channel 0 of the half
    };
    auto share = [&](int i, int pairs, int rim, int x0, int y0) {
        Share t;
        const int h = i & 1, r = i >> 1, px = r % pairs, row = r / pairs;
        const int gx = x0 + 2 * px - rim, gy = y0 + row - rim;
        const bool yin = gy >= 0 && gy < d.ny;
        t.in0 = yin && gx >= 0 && gx < d.nx;
        t.in1 = yin && gx + 1 >= 0 && gx + 1 < d.nx;
        t.off = ((int64_t)gy * d.nx + gx) * kC + 8 * h;
        t.lds = (row * kC + 8 * h) * kWRow + px;
        return t;
    };
    const int64_t plane = (int64_t)d.nx * d.ny * kC;
    auto load = [&](const uint16_t *src, const Share &t, int z, uint4 (&v)[2]) {
        v[0] = v[1] = make_uint4(0u, 0u, 0u, 0u);
        if (z < 0 || z >= d.nz) return;
        if (t.in0) v[0] = *reinterpret_cast<const uint4 *>(src + z * plane + t.off);
        if (t.in1) v[1] = *reinterpret_cast<const uint4 *>(src + z * plane + t.off + kC);
    };
    auto put = [&](uint32_t *dst_, const Share &t, const uint4 (&v)[2]) {
        const uint32_t lo[4] = {v[0].x, v[0].y, v[0].z, v[0].w}, hi[4] = {v[1].x, v[1].y, v[1].z, v[1].w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            dst_[t.lds + (2 * c) * kWRow] = __builtin_amdgcn_perm(hi[c], lo[c], 0x05040100u);
            dst_[t.lds + (2 * c + 1) * kWRow] = __builtin_amdgcn_perm(hi[c], lo[c], 0x07060302u);
        }
    };
    const bool has_a = (int)threadIdx.x < kSharesA, has_g = (int)threadIdx.x >= kWThreads - kSharesG;
    double dacc[3][4];
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) dacc[t][r] = 0.0;
    double bacc = 0.0;
    for (int it = march_first(); it < m.items; it += gridDim.x) {
        int cx, cy, z0, z1;
        march_place(m, d, it, cx, cy, z0, z1);
        Share ia = share(has_a ? (int)threadIdx.x : 0, kWX / 2 + 1, 1, cx * kWX, cy * kWY);
        Share ig = share(has_g ? (int)threadIdx.x - (kWThreads - kSharesG) : 0, kWX / 2, 0, cx * kWX, cy * kWY);
        ia.in0 = ia.in0 && has_a;
        ia.in1 = ia.in1 && has_a;
        ig.in0 = ig.in0 && has_g;
        ig.in1 = ig.in1 && has_g;
        uint4 va[2], vg[2];
        __syncthreads();  // the previous item's planes are done with
        for (int q = -1; q <= 0; ++q) {
            load(a1, ia, z0 + q, va);
            if (has_a) put(sa[(z0 + q) & 3], ia, va);
        }
        load(a1, ia, z0 + 1, va);
        load(gh2, ig, z0, vg);
        for (int z = z0; z < z1; ++z) {
            if (has_a) put(sa[(z + 1) & 3], ia, va);
            if (has_g) put(sg[z & 1], ig, vg);
            __syncthreads();
            if (z + 1 < z1) {
                load(a1, ia, z + 2, va);
                load(gh2, ig, z + 1, vg);
            }
            const uint32_t *pa = sa[(z - 1 + dz) & 3] + (dy * kC + n) * kWRow + 4 * g;
            const uint32_t *pg = sg[z & 1] + n * kWRow + 4 * g;
#pragma unroll
            for (int yp = 0; yp < kWY; yp += 4) {  // two pairs of rows, a sum each
                f32x4 acc[2][3];
#pragma unroll
                for (int p = 0; p < 2; ++p)
#pragma unroll
                    for (int t = 0; t < 3; ++t) acc[p][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < 2; ++i) {
#pragma unroll
                    for (int p = 0; p < 2; ++p) {
                        const int y = yp + 2 * p + i;
                        const uint4 q = *reinterpret_cast<const uint4 *>(pg + y * kC * kWRow);
                        const bf16x8 av = __builtin_bit_cast(bf16x8, q);
                        if (y == wave) {
                            const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                bacc += (double)bf2f((uint16_t)(w[e] & 0xffffu)) + (double)bf2f((uint16_t)(w[e] >> 16));
                        }
                        const uint4 u = *reinterpret_cast<const uint4 *>(pa + y * kC * kWRow);
                        const uint32_t w[5] = {u.x, u.y, u.z, u.w, pa[y * kC * kWRow + 4]};
#pragma unroll
                        for (int dx = 0; dx < 3; ++dx) {
                            uint32_t s4[4];
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                s4[e] = dx == 0 ? w[e]
                                                : (dx == 1 ? __builtin_amdgcn_alignbit(w[e + 1], w[e], 16) : w[e + 1]);
                            acc[p][dx] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, s4),
                                                                                acc[p][dx], 0, 0, 0);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);  // five products between two of one sum
                }
#pragma unroll
                for (int p = 0; p < 2; ++p)
#pragma unroll
                    for (int t = 0; t < 3; ++t)
#pragma unroll
                        for (int r = 0; r < 4; ++r) dacc[t][r] += (double)acc[p][t][r];
            }
        }
    }
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) dst[((4 * g + r) * kC + n) * kTaps + 3 * wave + t] = dacc[t][r];
    if (wave < kWY) bred[wave][lane] = bacc;
    __syncthreads();
    if (threadIdx.x < kC) {
        double b = 0.0;
        for (int w = 0; w < kWY; ++w)
            for (int q = 0; q < 4; ++q) b += bred[w][16 * q + threadIdx.x];
        dst[kC * kC * kTaps + threadIdx.x] = b;
    }
}

// The two factors of a layer's weight gradient, gw[t] = sum_v f(v) h(v + o_t)
// over the pairs of voxels inside the volume: f is the layer's data gradient
// (BF16 [voxel][16]; the output gradient for layer 3, FP32), h its input (BF16
// [voxel][16]; x for layer 1, FP32).  gb = sum_v f(v).
struct GradFactors {
    const uint16_t *fb, *hb;  // BF16 factors (null: the FP32 ones)
    const float *ff, *hf;
};

// This thread's share of output o of layer kLayer's gradient, pair by pair in
// FP64: voxels outside the volume have no part, nor (layer 2) have zeros of f.
// A wavefront takes runs of eight rows, so that sixteen loads are under way; a
// NaN in one thread's share is the result (*stop), and the others end.
template <int kLayer>
__device__ inline double grad_by_pairs(int o, const GradFactors &p, const Vol &d, volatile int *stop)
{
    constexpr int kRun = 8;
    const int nw = (kLayer == 2 ? kC : 1) * kC * kTaps;
    const bool bias = o >= nw;
    const int q = bias ? 0 : o / kTaps, t = bias ? 13 : o % kTaps;  // 13: the voxel itself
    const int cf = kLayer == 3 ? 0 : (bias ? o - nw : (kLayer == 2 ? q / kC : q));
    const int ch = q % kC;
    const int ox = t % 3 - 1, oy = (t / 3) % 3 - 1, oz = t / 9 - 1;
    const int rows = d.ny * d.nz;
    double acc = 0.0;
    for (int row0 = (threadIdx.x >> 6) * kRun; row0 < rows && !*stop; row0 += kThreads / 64 * kRun) {
        int64_t h0[kRun];  // voxel (0, row) shifted by the tap's rows (-1: no pair)
        int j = row0 % d.ny, k = row0 / d.ny;
#pragma unroll
        for (int u = 0; u < kRun; ++u) {
            const int jj = j + oy, kk = k + oz;
            const bool in = row0 + u < rows && jj >= 0 && jj < d.ny && kk >= 0 && kk < d.nz;
            h0[u] = in ? ((int64_t)kk * d.ny + jj) * d.nx : -1;
            if (++j == d.ny) {
                j = 0;
                ++k;
            }
        }
        for (int i = threadIdx.x & 63; i < d.nx; i += 64) {
            if (i + ox < 0 || i + ox >= d.nx) continue;
            float f[kRun], h[kRun];
#pragma unroll
            for (int u = 0; u < kRun; ++u) {
                const int64_t v = h0[u] < 0 ? 0 : (int64_t)(row0 + u) * d.nx + i, w = h0[u] < 0 ? 0 : h0[u] + i + ox;
                f[u] = kLayer == 3 ? p.ff[v] : bf2f(p.fb[v * kC + cf]);
                h[u] = bias ? 1.0f : (kLayer == 1 ? p.hf[w] : bf2f(p.hb[w * kC + ch]));
            }
#pragma unroll
            for (int u = 0; u < kRun; ++u)
                if (h0[u] >= 0 && !(kLayer == 2 && f[u] == 0.0f)) acc += (double)f[u] * (double)h[u];
        }
        if (acc != acc) *stop = 1;
    }
    return acc;
}

// grad[off + o] = sum over blocks of part[b][o], in a fixed order: eight
// threads per output take the blocks b = k, k + 8, ... and are added in turn.
// The matrix products also multiply what the sum leaves out, by zeros (voxels
// of a column outside the volume, zeros of layer 2's data gradient), which an
// infinite or NaN factor turns into NaN.  Such a factor is in a product of
// every sum it belongs to as well, so a finite sum is right as it stands, and
// the others are taken again pair by pair.
constexpr int kRedOut = 32;
template <int kLayer>
__global__ __launch_bounds__(kThreads) void k_reduce_parts(const double *__restrict__ part, int nblocks, int width,
                                                           float *__restrict__ grad, int off, GradFactors factors, Vol d)
{
    static_assert(kThreads == 8 * kRedOut, "eight threads per output");
    __shared__ double red[8][kRedOut];
    const int l = threadIdx.x % kRedOut, k = threadIdx.x / kRedOut, o = blockIdx.x * kRedOut + l;
    double s = 0.0;
    if (o < width) {
#pragma unroll 8
        for (int b = k; b < nblocks; b += 8) s += part[(int64_t)b * width + o];
    }
    red[k][l] = s;
    __syncthreads();
    if (k == 0 && o < width) {
        for (int q = 1; q < 8; ++q) s += red[q][l];
        grad[off + o] = (float)s;
        red[0][l] = s;
    }
    const bool again = k == 0 && o < width && !isfinite(s);
    if (!__syncthreads_or(again ? 1 : 0)) return;
    __shared__ double lds[4];
    __shared__ int stop;
    for (int q = 0; q < kRedOut && blockIdx.x * kRedOut + q < width; ++q) {
        if (isfinite(red[0][q])) continue;
        if (threadIdx.x == 0) stop = 0;
        __syncthreads();
        const double sum = block_sum(grad_by_pairs<kLayer>(blockIdx.x * kRedOut + q, factors, d, &stop), lds);
        if (threadIdx.x == 0) grad[off + blockIdx.x * kRedOut + q] = (float)sum;
    }
}

__global__ void k_adam(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                       float *__restrict__ v, int n, double lr, double b1, double b2, double eps,
                       double c1, double c2)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double gi = g[i];
    const double mi = b1 * m[i] + (1.0 - b1) * gi;
    const double vi = b2 * v[i] + (1.0 - b2) * gi * gi;
    m[i] = (float)mi;
    v[i] = (float)vi;
    p[i] = (float)((double)p[i] - lr * (mi / c1) / (sqrt(vi / c2) + eps));
}

// ------------------------------------------------------------ host side

struct NetWs {
    uint16_t *a1, *a2, *gh;  // [n][16] each
    float *out, *g;          // [n]
    bf16x8 *frag, *fragT;    // forward and transposed fragment sets
    double *part;            // weight-gradient partials
    double *loss_part;       // [kRedLossBlocks]
};
constexpr int kLossBlocks = 1024;
static_assert((int64_t)kFieldBlocks * kFPart1 <= (int64_t)kWgBlocks * kWPart, "the partial sums' place");

static size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

static size_t ws_layout(int64_t n, NetWs *w, char *base)
{
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char *p = base ? base + off : nullptr;
        off += align256(bytes);
        return p;
    };
    NetWs t;
    t.a1 = (uint16_t *)take(sizeof(uint16_t) * kC * n);
    t.a2 = (uint16_t *)take(sizeof(uint16_t) * kC * n);
    t.gh = (uint16_t *)take(sizeof(uint16_t) * kC * n);
    t.out = (float *)take(sizeof(float) * n);
    t.g = (float *)take(sizeof(float) * n);
    t.frag = (bf16x8 *)take(sizeof(bf16x8) * kFragFwd);
    t.fragT = (bf16x8 *)take(sizeof(bf16x8) * kFragConv);
    t.part = (double *)take(sizeof(double) * kWgBlocks * kWPart);
    t.loss_part = (double *)take(sizeof(double) * kLossBlocks);
    if (w) *w = t;
    return off;
}

// Forward-only workspace (activations and fragments) for flexible CG.
size_t convnet_forward_ws_bytes(int64_t n)
{
    return align256(sizeof(uint16_t) * kC * n) * 2 + align256(sizeof(bf16x8) * kFragFwd);
}

static dim3 tile_grid(const Vol &d)
{
    return dim3((unsigned)((d.nx + kTX - 1) / kTX), (unsigned)((d.ny + kTY - 1) / kTY),
                (unsigned)((d.nz + kTZ - 1) / kTZ));
}

// Launch of a marching kernel of nt lanes over columns of cx x cy outputs: as
// many planes per item as leave about one round of the workgroups that stay
// resident on the device (occupancy x compute units, queried once per kernel);
// one workgroup per item, or at most `most` that take the items in turn.
static unsigned march_grid(const void *kernel, const Vol &d, int cx, int cy, March &m, int64_t most = 0,
                           int nt = kThreads)
{
    static std::mutex mu;
    static std::map<const void *, int64_t> resident;
    int64_t r = 0;
    {
        std::lock_guard<std::mutex> lock(mu);
        auto it = resident.find(kernel);
        if (it != resident.end()) {
            r = it->second;
        } else {
            int dev = 0, cus = 0, per = 0;
            (void)hipGetDevice(&dev);
            (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
            (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, nt, 0);
            r = (int64_t)(cus > 0 ? cus : 256) * (per > 0 ? per : 1);
            resident[kernel] = r;
        }
    }
    if (most > 0 && r > most) r = most;
    m.ncx = (d.nx + cx - 1) / cx;
    m.ncy = (d.ny + cy - 1) / cy;
    const int64_t cols = (int64_t)m.ncx * m.ncy;
    int64_t chunks = r / cols;
    chunks = chunks < 1 ? 1 : (chunks > d.nz ? d.nz : chunks);
    m.cz = (int32_t)((d.nz + chunks - 1) / chunks);
    const int64_t runs = (d.nz + m.cz - 1) / m.cz;
    m.items = (int32_t)(cols * runs);
    m.by_column = cols >= d.nz;
    m.inner = (int32_t)(m.by_column ? runs : cols);
    return (unsigned)(most > 0 && m.items > most ? most : m.items);
}

// Columns of 8 rows instead of 16, two wavefronts each, where a workgroup has
// one plane, there are more of them than CUs and 8-row columns hold at least a
// tenth fewer rows past the volume's edge: 33^3 18.6 -> 17.5 us, 100x33x17 20.9
// -> 19.1, 25x40x60 19.0 -> 17.9 (forward).  More columns read more rim: 48^3,
// whose rows fill 16, 19.3 and 20.0; up to one per CU they add waits: 17x33x50
// 16.4 and 17.6.  A training pass keeps 16 rows, nearer to its gradients' columns
// (20x50x50 68 us, 70 with 8).
static bool half_columns(const Vol &d)
{
    const int64_t items = (int64_t)((d.nx + kZX - 1) / kZX) * ((d.ny + kZY - 1) / kZY) * d.nz;
    return items > 256 && items <= 768 && 10 * ((d.ny + 7) / 8 * 8) <= 9 * ((d.ny + kZY - 1) / kZY * kZY);
}

template <int kMode, int kWaves>
static void launch_conv16z(const uint16_t *in, const bf16x8 *frag, const float *bias, const Vol &d,
                           const uint16_t *mask, uint16_t *out, const LastOut &last, const int *skip, hipStream_t s)
{
    March m;
    const unsigned nb = march_grid(reinterpret_cast<const void *>(k_conv16z<kMode, kWaves>), d, kZX, 4 * kWaves, m, 0,
                                   kWaves * 64);
    hipLaunchKernelGGL((k_conv16z<kMode, kWaves>), dim3(nb), dim3(kWaves * 64), 0, s, in, frag, bias, d, m, mask, out,
                       last, skip);
}

// The layers on a stored activation: the marching kernels, or one tile per
// workgroup where an activation passes the marching kernel's reach.
template <int kMode>
static void launch_conv16(const uint16_t *in, const bf16x8 *frag, const float *bias, const Vol &d,
                          const uint16_t *mask, uint16_t *out, bool half, const int *skip, hipStream_t s)
{
    if (d.n > kMaxMarchVoxels)
        hipLaunchKernelGGL(k_conv16, tile_grid(d), dim3(kThreads), 0, s, in, frag, bias, d, kMode == kForward ? 1 : 0,
                           mask, out, skip);
    else if (half)
        launch_conv16z<kMode, 2>(in, frag, bias, d, mask, out, LastOut{}, skip, s);
    else
        launch_conv16z<kMode, 4>(in, frag, bias, d, mask, out, LastOut{}, skip, s);
}

template <int kWaves>
static void launch_conv1z(const bf16x8 *frag1, const float *P, const float *x, const Vol &d, const double *norm2,
                          uint16_t *a1, const int *skip, hipStream_t s)
{
    March m;
    const unsigned nb = march_grid(reinterpret_cast<const void *>(k_conv1z<kWaves>), d, kZX, 4 * kWaves, m, 0, kWaves * 64);
    hipLaunchKernelGGL(k_conv1z<kWaves>, dim3(nb), dim3(kWaves * 64), 0, s, frag1, P, x, d, m, norm2, a1, skip);
}

static void launch_conv1(const bf16x8 *frag1, const float *P, const float *x, const Vol &d, const double *norm2,
                         uint16_t *a1, bool half, const int *skip, hipStream_t s)
{
    if (half) launch_conv1z<2>(frag1, P, x, d, norm2, a1, skip, s);
    else launch_conv1z<4>(frag1, P, x, d, norm2, a1, skip, s);
}

static void launch_conv3(const bf16x8 *frag3, const float *P, const uint16_t *a2, const Vol &d, const double *norm2,
                         const uint8_t *map_mask, float *out, bool half, const int *skip, hipStream_t s)
{
    const LastOut last{out, norm2, map_mask};
    if (d.n > kMaxMarchVoxels)
        hipLaunchKernelGGL(k_conv3, tile_grid(d), dim3(kThreads), 0, s, frag3, P, a2, d, norm2, map_mask, out, skip);
    else if (half)
        launch_conv16z<kLast, 2>(a2, frag3, P + OB3, d, nullptr, nullptr, last, skip, s);
    else
        launch_conv16z<kLast, 4>(a2, frag3, P + OB3, d, nullptr, nullptr, last, skip, s);
}

// z = s N(x / s) on the device (s = sqrt(*norm2), or 1), zero where the map
// mask is 0; nothing happens while *skip != 0.  ws: convnet_forward_ws_bytes(n)
// bytes; prep_frags = false reuses the weight fragments of an earlier call.
int convnet_forward_dev(const tomo_cube &c, const float *P, const float *x, float *out,
                        const double *norm2, const uint8_t *map_mask, void *ws, hipStream_t s,
                        bool prep_frags, const int *skip)
{
    const Vol d{c.nx, c.ny, c.nz, (int64_t)c.nx * c.ny * c.nz};
    char *base = (char *)ws;
    uint16_t *a1 = (uint16_t *)base;
    uint16_t *a2 = (uint16_t *)(base + align256(sizeof(uint16_t) * kC * d.n));
    bf16x8 *frag = (bf16x8 *)(base + 2 * align256(sizeof(uint16_t) * kC * d.n));
    if (prep_frags)
        hipLaunchKernelGGL(k_conv_frags, dim3((kFragFwd + 255) / 256), dim3(256), 0, s, P, 0, frag);
    const bool half = half_columns(d);
    launch_conv1(frag + kFrag1, P, x, d, norm2, a1, half, skip, s);
    launch_conv16<kForward>(a1, frag, P + OB2, d, nullptr, a2, half, skip, s);
    launch_conv3(frag + kFrag3, P, a2, d, norm2, map_mask, out, half, skip, s);
    return hip_fail(hipGetLastError(), "convnet forward launch");
}

}  // namespace tomo

using namespace tomo;

static int check_net_cube(const tomo_cube *c)
{
    int rc = validate_cube(c);
    if (rc) return rc;
    if (c->nframes != 1) return set_error(TOMO_EINVAL, "convnet: the cube must hold one frame");
    return TOMO_OK;
}

extern "C" {

size_t tomo_convnet_workspace_bytes(const tomo_cube *cube)
{
    if (!cube || validate_cube(cube)) return 0;
    return ws_layout((int64_t)cube->nx * cube->ny * cube->nz, nullptr, nullptr);
}

int tomo_convnet_forward(const tomo_cube *cube, const float *params_d, const float *x_d,
                         float *out_d, void *ws_d, size_t ws_bytes, tomo_stream stream)
{
    int rc = check_net_cube(cube);
    if (rc) return rc;
    if (!params_d || !x_d || !out_d || !ws_d)
        return set_error(TOMO_EINVAL, "tomo_convnet_forward: NULL argument");
    const int64_t n = (int64_t)cube->nx * cube->ny * cube->nz;
    if (ws_bytes < ws_layout(n, nullptr, nullptr))
        return set_error(TOMO_EINVAL, "tomo_convnet_forward: workspace too small");
    return convnet_forward_dev(*cube, params_d, x_d, out_d, nullptr, nullptr, ws_d,
                               (hipStream_t)stream, true, nullptr);
}

// Forward pass that keeps the activations, then back-propagation of the
// output gradient g_d (d loss / d out, one value per voxel) into grad_d.  With
// target_d set, g_d is ignored and replaced by the MSE gradient
// 2 (out - target) / n, whose per-block loss partials land in w.loss_part.
static int convnet_train_pass(const tomo_cube *cube, const float *params_d, const float *x_d,
                              const float *target_d, const float *g_d, float *grad_d, void *ws_d,
                              hipStream_t s)
{
    const int64_t n = (int64_t)cube->nx * cube->ny * cube->nz;
    NetWs w;
    ws_layout(n, &w, (char *)ws_d);
    const Vol d{cube->nx, cube->ny, cube->nz, n};
    // forward, keeping activations
    hipLaunchKernelGGL(k_conv_frags, dim3((kFragFwd + 255) / 256), dim3(256), 0, s, params_d, 0, w.frag);
    hipLaunchKernelGGL(k_conv_frags, dim3((kFragConv + 255) / 256), dim3(256), 0, s, params_d, 1, w.fragT);
    const int *noskip = nullptr;
    launch_conv1(w.frag + kFrag1, params_d, x_d, d, nullptr, w.a1, false, noskip, s);
    launch_conv16<kForward>(w.a1, w.frag, params_d + OB2, d, nullptr, w.a2, false, noskip, s);
    if (target_d) {
        launch_conv3(w.frag + kFrag3, params_d, w.a2, d, nullptr, nullptr, w.out, false, noskip, s);
        // loss and d loss / d out
        hipLaunchKernelGGL(k_mse, dim3(kLossBlocks), dim3(kThreads), 0, s, w.out, target_d, n, w.g,
                           w.loss_part);
        g_d = w.g;
    }
    March m;
    unsigned nb;
    auto reduce = [&](auto layer, unsigned blocks, int width, int off, const GradFactors &f) {
        hipLaunchKernelGGL(k_reduce_parts<decltype(layer)::value>, dim3((unsigned)((width + kRedOut - 1) / kRedOut)),
                           dim3(kThreads), 0, s, w.part, (int)blocks, width, grad_d, off, f, d);
    };
    // layer 3
    nb = march_grid(reinterpret_cast<const void *>(k_wgrad_field<false>), d, kZX, kZY, m, kFieldBlocks);
    hipLaunchKernelGGL(k_wgrad_field<false>, dim3(nb), dim3(kThreads), 0, s, w.a2, g_d, d, m, w.part);
    reduce(std::integral_constant<int, 3>{}, nb, kFPart3, OW3, GradFactors{nullptr, w.a2, g_d, nullptr});
    nb = march_grid(reinterpret_cast<const void *>(k_conv3_bwd), d, kBX, kBY, m);
    hipLaunchKernelGGL(k_conv3_bwd, dim3(nb), dim3(kThreads), 0, s, params_d, g_d, w.a2, d, m, w.gh);
    // layer 2 (gh = d loss / d h2)
    nb = march_grid(reinterpret_cast<const void *>(k_wgrad2), d, kWX, kWY, m, kWgBlocks, kWThreads);
    hipLaunchKernelGGL(k_wgrad2, dim3(nb), dim3(kWThreads), 0, s, w.gh, w.a1, d, m, w.part);
    reduce(std::integral_constant<int, 2>{}, nb, kWPart, OW2, GradFactors{w.gh, w.a1, nullptr, nullptr});
    // d loss / d h1 = [a1 > 0] conv^T(gh); written over a2 (no longer needed)
    launch_conv16<kMasked>(w.gh, w.fragT, nullptr, d, w.a1, w.a2, false, noskip, s);
    // layer 1
    nb = march_grid(reinterpret_cast<const void *>(k_wgrad_field<true>), d, kZX, kZY, m, kFieldBlocks);
    hipLaunchKernelGGL(k_wgrad_field<true>, dim3(nb), dim3(kThreads), 0, s, w.a2, x_d, d, m, w.part);
    reduce(std::integral_constant<int, 1>{}, nb, kFPart1, OW1, GradFactors{w.a2, nullptr, nullptr, x_d});
    return hip_fail(hipGetLastError(), "convnet backward launch");
}

int tomo_convnet_loss_grad(const tomo_cube *cube, const float *params_d, const float *x_d,
                           const float *target_d, float *grad_d, double *loss_h, void *ws_d,
                           size_t ws_bytes, tomo_stream stream)
{
    int rc = check_net_cube(cube);
    if (rc) return rc;
    if (!params_d || !x_d || !target_d || !grad_d || !ws_d)
        return set_error(TOMO_EINVAL, "tomo_convnet_loss_grad: NULL argument");
    const int64_t n = (int64_t)cube->nx * cube->ny * cube->nz;
    if (ws_bytes < ws_layout(n, nullptr, nullptr))
        return set_error(TOMO_EINVAL, "tomo_convnet_loss_grad: workspace too small");
    hipStream_t s = (hipStream_t)stream;
    rc = convnet_train_pass(cube, params_d, x_d, target_d, nullptr, grad_d, ws_d, s);
    if (rc) return rc;
    if (loss_h) {
        NetWs w;
        ws_layout(n, &w, (char *)ws_d);
        double parts[kLossBlocks];
        rc = hip_fail(hipMemcpyAsync(parts, w.loss_part, sizeof(parts), hipMemcpyDeviceToHost, s), "loss copy");
        if (!rc) rc = hip_fail(hipStreamSynchronize(s), "loss synchronise");
        if (rc) return rc;
        double acc = 0.0;
        for (int b = 0; b < kLossBlocks; ++b) acc += parts[b];
        *loss_h = acc / (double)n;
    }
    return TOMO_OK;
}

int tomo_convnet_backward(const tomo_cube *cube, const float *params_d, const float *x_d,
                          const float *dout_d, float *grad_d, void *ws_d, size_t ws_bytes,
                          tomo_stream stream)
{
    int rc = check_net_cube(cube);
    if (rc) return rc;
    if (!params_d || !x_d || !dout_d || !grad_d || !ws_d)
        return set_error(TOMO_EINVAL, "tomo_convnet_backward: NULL argument");
    const int64_t n = (int64_t)cube->nx * cube->ny * cube->nz;
    if (ws_bytes < ws_layout(n, nullptr, nullptr))
        return set_error(TOMO_EINVAL, "tomo_convnet_backward: workspace too small");
    return convnet_train_pass(cube, params_d, x_d, nullptr, dout_d, grad_d, ws_d, (hipStream_t)stream);
}

int tomo_adam_step(float *params_d, const float *grad_d, float *m_d, float *v_d, int32_t n,
                   int32_t step, double lr, double beta1, double beta2, double eps,
                   tomo_stream stream)
{
    if (!params_d || !grad_d || !m_d || !v_d || n < 1 || step < 1 || !(lr > 0) || !(beta1 >= 0) ||
        !(beta1 < 1) || !(beta2 >= 0) || !(beta2 < 1) || !(eps > 0))
        return set_error(TOMO_EINVAL, "tomo_adam_step: invalid argument");
    const double c1 = 1.0 - pow(beta1, step), c2 = 1.0 - pow(beta2, step);
    hipLaunchKernelGGL(k_adam, dim3((n + 255) / 256), dim3(256), 0, (hipStream_t)stream, params_d, grad_d,
                       m_d, v_d, n, lr, beta1, beta2, eps, c1, c2);
    return hip_fail(hipGetLastError(), "adam launch");
}

}  // extern "C"
