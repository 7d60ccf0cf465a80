// Voxel-embedding LOCC variant (Sec. III, appendix "Architecture Details").
//
// Shape encoder (once per shape, at upload; float32 arithmetic, float64 grid
// assignment): cell_sort_kernel orders each shape's points by grid cell;
// point_mlp_kernel runs the per-point MLP over chunks of 64 points in that
// order (layers 2-3 on the matrix cores) and keeps the channel-wise max per
// grid cell (an atomic max per run of equal cells, on the bit patterns, which
// order like the values for the non-negative ReLU outputs);
// conv_kernel runs every convolution and transposed convolution of the
// U-Net as an implicit GEMM on the matrix cores (the skip concatenation read
// from two inputs); global_kernel takes max and mean over the bottleneck cells;
// embed_kernel maps [last layer, global feature] to the 16-float embedding;
// consts_kernel writes the float64 cell size and margin of each shape.
//
// Predictor, two launches.  select_kernel: one wave per pair validates it,
// puts it in canonical order, computes the float64 relative pose
// (wave-uniform), runs each object's 216 cell tests (centres formed in
// registers; float64, fixed order, contraction off) as four 64-lane ballots
// and the means of the selected cells' embeddings (lane = 4 features x cell
// residue mod 16, the float4 loads of both objects issued together, summed
// across the residues by shuffles), and writes both objects' predictor input
// rows to the workspace; with small register use many waves are in flight
// to hide the load latency (80 registers, six waves per SIMD: 35 us at
// 16,384 pairs; 86 registers: 1.4 us more).  mlp_kernel: 32 pairs per workgroup of
// eight waves run the per-object MLP on the 64 rows, the pair max, the pair
// MLP and the output layer as products of halves on the 16-bit matrix cores,
// activations in LDS, each layer in place.
#include <cmath>
#include <cstring>

#include "geometry.h"
#include "halves.h"
#include "voxel.h"

namespace locc {
namespace vox {
namespace {

__device__ __forceinline__ float relu(float x) { return x > 0.f ? x : 0.f; }

// Where the U-Net's activations keep channel c of shape s (of S) at grid position x: [x][c / 8][c % 2][s][(c % 8) / 2],
// so that 16 bytes hold four channels of a column and a half-wave's loads are contiguous.
__device__ __forceinline__ size_t act_at(int x, int c, int s, int C, int S) {
  return ((((size_t)x * (C / 8) + c / 8) * 2 + (c & 1)) * S + s) * 4 + ((c & 7) >> 1);
}

// Grid cell of a stored point (float64, the order of the reading).
__device__ __forceinline__ int cell_of(float x, float y, float z, const Shape& sh) {
#pragma clang fp contract(off)
  const float p[3] = {x, y, z};
  int idx = 0;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double lo = sh.lo[k], hi = sh.hi[k];
    const double ext = hi - lo;
    int i = 0;
    if (ext > 0.0) {
      const double t = (((double)p[k] - lo) * (double)kM) / ext;
      i = (int)__builtin_floor(t);
      i = i < 0 ? 0 : (i > kM - 1 ? kM - 1 : i);
    }
    idx = idx * kM + i;
  }
  return idx;
}

// Counting sort of each shape's points by grid cell (a workgroup per shape):
// the cell histogram, its exclusive scan, then each point's slot from its
// cell's cursor.  The order within a cell depends on the timing of the LDS
// atomics; the cell max built from it does not.
__global__ __launch_bounds__(1024) void cell_sort_kernel(const Shape* shapes, const float* xyz, int64_t n_points,
                                                          int32_t* order, uint8_t* cells) {
  __shared__ int hist[kCells];
  const Shape sh = shapes[blockIdx.x];
  const int t = threadIdx.x;
  auto cell_at = [&](int i) {
    const int64_t r = (int64_t)sh.off + i;
    return cell_of(xyz[r], xyz[n_points + r], xyz[2 * n_points + r], sh);
  };
  for (int c = t; c < kCells; c += 1024) hist[c] = 0;
  __syncthreads();
  for (int i = t; i < sh.n; i += 1024) atomicAdd(&hist[cell_at(i)], 1);
  __syncthreads();
  if (t == 0) {  // exclusive scan: hist[c] becomes the first slot of cell c
    int run = 0;
    for (int c = 0; c < kCells; ++c) {
      const int h = hist[c];
      hist[c] = run;
      run += h;
    }
  }
  __syncthreads();
  for (int i = t; i < sh.n; i += 1024) {
    const int c = cell_at(i);
    const int slot = atomicAdd(&hist[c], 1);
    order[sh.off + slot] = i;
    cells[sh.off + slot] = (uint8_t)c;
  }
}

constexpr int kPts = 64;  // points per workgroup of the point MLP

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

struct PointShared {
  union {
    unsigned short h[2][kPts][kH + 8];  // activations: [part][point][channel], 16 bytes past a multiple of 128
    float out[kH][kPts + 1];            // the last layer's, for the pooling walk; as FP32 products every layer's
  };
  float top[4][kPts];                   // per wave and point: a layer's largest output
  int32_t again;                        // a point whose layers are FP32 products
};

// Layers 1 to 3 of the per-point MLP 3 -> 256 -> 256 -> 256 for 64 points (a lane's in x, y, z) as FP32 products.
// Layer 1 on the vector units (a wave per 64 channels, a lane per point);
// layers 2 and 3 on the matrix cores (v_mfma_f32_32x32x2f32, bias as the
// accumulator's start): wave w owns output channels [64 w, 64 w + 64), two
// 32-channel tiles over the two 32-point tiles, its A operands the rows of
// the transposed weights Wt[in][out] (coalesced, four steps ahead), its B
// operands the activations, kept channel-major in LDS (HT[c][p]: a step
// reads two rows of 32 points).  The last layer's outputs go to LDS too.
// Lane layouts as in conv_kernel below.
__device__ __forceinline__ void point_fp32(const PackedNet& w, float x, float y, float z, float (&HT)[kH][kPts + 1]) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, g = lane >> 5, l32 = lane & 31;
  for (int k = 0; k < 64; ++k) {  // lane = point, the wave's 64 channels in turn
    const int o = wave * 64 + k;
    HT[o][lane] = relu(((w.P1[3 * o] * x + w.P1[3 * o + 1] * y) + w.P1[3 * o + 2] * z) + w.p1[o]);
  }
  __syncthreads();
  f32x16 acc[2][2];  // [channel tile][point tile]
  for (int layer = 0; layer < 2; ++layer) {
    const float* Wt = (layer ? w.P3t : w.P2t) + (size_t)g * kH + wave * 64 + l32;
    const float* bias = (layer ? w.p3 : w.p2) + wave * 64 + 4 * g;
#pragma unroll
    for (int ot = 0; ot < 2; ++ot)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float b = bias[32 * ot + 8 * (r >> 2) + (r & 3)];
        acc[ot][0][r] = b;
        acc[ot][1][r] = b;
      }
    constexpr int kAhead = 4;
    float ar[kAhead][2];
#pragma unroll
    for (int d = 0; d < kAhead; ++d)
#pragma unroll
      for (int ot = 0; ot < 2; ++ot) ar[d][ot] = Wt[(size_t)2 * d * kH + 32 * ot];
    for (int k = 0; k < kH; k += 2 * kAhead) {
#pragma unroll
      for (int d = 0; d < kAhead; ++d) {
        const int kk = k + 2 * d;
        const float b0 = HT[kk + g][l32], b1 = HT[kk + g][32 + l32];
#pragma unroll
        for (int ot = 0; ot < 2; ++ot) {
          acc[ot][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(ar[d][ot], b0, acc[ot][0], 0, 0, 0);
          acc[ot][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(ar[d][ot], b1, acc[ot][1], 0, 0, 0);
        }
        const int kn = kk + 2 * kAhead;
        if (kn < kH) {
#pragma unroll
          for (int ot = 0; ot < 2; ++ot) ar[d][ot] = Wt[(size_t)kn * kH + 32 * ot];
        }
      }
    }
    __syncthreads();  // every wave has read HT
#pragma unroll
    for (int ot = 0; ot < 2; ++ot)
#pragma unroll
      for (int pt = 0; pt < 2; ++pt)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          HT[wave * 64 + 32 * ot + 8 * (r >> 2) + 4 * g + (r & 3)][32 * pt + l32] = relu(acc[ot][pt][r]);
    __syncthreads();
  }
}

// v * scale as halves, four in a row of each part.
__device__ __forceinline__ void put_halves(unsigned short* part0, unsigned short* part1, const float (&v)[4],
                                           float scale) {
  float a = v[0] * scale, b = v[1] * scale, c = v[2] * scale, d = v[3] * scale;
  uint2 h, l;
  h.x = split_part(a, b);
  h.y = split_part(c, d);
  l.x = last_part(a, b);
  l.y = last_part(c, d);
  *reinterpret_cast<uint2*>(part0) = h;
  *reinterpret_cast<uint2*>(part1) = l;
}

// The per-point MLP over 64 points, taken in cell order, and the cell max: a thread per channel walks the 64 points,
// whose cells come in runs, and issues one atomic max per run.
// Layers 2 and 3 are products of halves (halves.h) on the 16-bit matrix cores (v_mfma_f32_32x32x16_f16, FP32
// accumulation).  A weight row is scaled by a power of two to a largest magnitude in [2^14, 2^15), and so are a point's
// inputs of a layer, by their own largest; both are undone exactly on the sums.
// Three 16-bit products of 16 steps take 96 cycles where FP32 takes 512: 70 us at 32 shapes of 2,048 points, 168 with
// the FP32 products.  Those stay for weights that have not all the bits they need as halves (fp32), and for 64 points
// one of which has a value near the end of the exponents or too many inputs of a layer short of bits.
constexpr float kHalvesMost = 0x1p90f;
__global__ __launch_bounds__(256, 2) void point_mlp_kernel(PackedNet w, int fp32, const Shape* shapes, const float* xyz,
                                                           int64_t n_points, const int32_t* order,
                                                           const uint8_t* cells, float* grid) {
  constexpr int KS = kH / 16, kAhead = 4;
  __shared__ PointShared S;
  const int s = blockIdx.y;
  const Shape sh = shapes[s];
  const int base = blockIdx.x * kPts;
  if (base >= sh.n) return;  // uniform
  const int np = sh.n - base < kPts ? sh.n - base : kPts;
  const int t = threadIdx.x, lane = t & 63, wave = wave_index(), g = lane >> 5, l32 = lane & 31;
  // lane = point, in every wave
  float x = 0.f, y = 0.f, z = 0.f;
  int cell = -1;
  if (lane < np) {
    const int64_t q = (int64_t)sh.off + base + lane;
    const int64_t r = (int64_t)sh.off + order[q];
    x = xyz[r];
    y = xyz[n_points + r];
    z = xyz[2 * n_points + r];
    cell = cells[q];
  }
  // marks the points whose inputs of a layer (largest: top) are out of range, or whose `least` says that some are short
  // of bits and count(below) that too many of a wave's 64 channels are
  auto check = [&](float top, unsigned least, bool mine, auto count) {
    const float below = kHalvesLeast * halves_unscale(halves_scale(top));
    bool bad = !(top < kHalvesMost);
    if (__ballot((least < __float_as_uint(below)) & (top > 0.f)) != 0)
      bad |= halves_short(count(below), kShortActivations);
    if (bad && mine) S.again = 1;
  };
  if (!fp32) {
    if (t == 0) S.again = 0;
    float scale[2];  // of the inputs of this lane's columns, points 32 pt + l32
    {                // layer 1: the wave's 64 channels, whose weights the lanes hold
      const int own = wave * 64 + lane;
      const float c0 = w.P1[3 * own], c1 = w.P1[3 * own + 1], c2 = w.P1[3 * own + 2], cb = w.p1[own];
      auto of = [](float v, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); };
      float v[64], top = 0.f;
      unsigned least = ~0u;  // bits of the smallest output that is not negative
#pragma unroll
      for (int k = 0; k < 64; ++k) {
        v[k] = ((of(c0, k) * x + of(c1, k) * y) + of(c2, k) * z) + of(cb, k);
        top = fmaxf(top, v[k]);
        least = min(least, __float_as_uint(v[k]));
      }
      S.top[wave][lane] = top;
      __syncthreads();
      top = fmaxf(fmaxf(S.top[0][lane], S.top[1][lane]), fmaxf(S.top[2][lane], S.top[3][lane]));
      check(top, least, lane < np, [&](float below) {
        int some = 0, lost = 0;
#pragma unroll
        for (int k = 0; k < 64; ++k) {
          some += v[k] > 0.f;
          lost += v[k] > 0.f && v[k] < below;
        }
        return some << 16 | lost;
      });
      const float up = halves_scale(top);
#pragma unroll
      for (int k = 0; k < 64; k += 4) {
        float a[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] = relu(v[k + e]);
        put_halves(&S.h[0][lane][wave * 64 + k], &S.h[1][lane][wave * 64 + k], a, up);
      }
#pragma unroll
      for (int pt = 0; pt < 2; ++pt) scale[pt] = __shfl(up, 32 * pt + l32, 64);
    }
    __syncthreads();
#pragma unroll 1
    for (int layer = 0; layer < 2; ++layer) {
      // A operands: [k-step][part][channel tile][lane][8]
      const u32x4* Wt = reinterpret_cast<const u32x4*>(layer ? w.P3s : w.P2s) + wave * 2 * 64 + lane;
      const float* bias = (layer ? w.p3 : w.p2) + wave * 64 + 4 * g;
      const float* unscale = (layer ? w.u3 : w.u2) + wave * 64 + 4 * g;
      u32x4 ar[kAhead][2][2];  // [ahead][part][channel tile]
      auto fetch = [&](int ks, u32x4 (&a)[2][2]) {
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int ot = 0; ot < 2; ++ot) a[q][ot] = Wt[(size_t)((ks * 2 + q) * (kH / 32) + ot) * 64];
      };
#pragma unroll
      for (int d = 0; d < kAhead; ++d) fetch(d, ar[d]);
      f32x16 acc[2][2];  // [channel tile][point tile]
#pragma unroll
      for (int ot = 0; ot < 2; ++ot) acc[ot][0] = acc[ot][1] = f32x16{};
#pragma unroll 1
      for (int k0 = 0; k0 < KS; k0 += kAhead) {
#pragma unroll
        for (int d = 0; d < kAhead; ++d) {
          const int ks = k0 + d;
          f16x8 b[2][2];  // [part][point tile]
#pragma unroll
          for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int pt = 0; pt < 2; ++pt)
              b[q][pt] = *reinterpret_cast<const f16x8*>(&S.h[q][32 * pt + l32][16 * ks + 8 * g]);
#pragma unroll
          for (int part = 2; part >= 0; --part)  // the small products first
#pragma unroll
            for (int ot = 0; ot < 2; ++ot)
#pragma unroll
              for (int pt = 0; pt < 2; ++pt)
                acc[ot][pt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, ar[d][part == 2][ot]),
                                                                     b[part == 1][pt], acc[ot][pt], 0, 0, 0);
          fetch(ks + kAhead < KS ? ks + kAhead : 0, ar[d]);  // past the end: loaded, not used
        }
      }
      float top[2] = {0.f, 0.f};
      unsigned least[2] = {~0u, ~0u};
#pragma unroll
      for (int ot = 0; ot < 2; ++ot)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float4 u4 = *reinterpret_cast<const float4*>(unscale + 32 * ot + 8 * q);
          const float4 b4 = *reinterpret_cast<const float4*>(bias + 32 * ot + 8 * q);
          const float u[4] = {u4.x, u4.y, u4.z, u4.w}, b[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
          for (int pt = 0; pt < 2; ++pt)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float v = fmaf(acc[ot][pt][4 * q + e], u[e] * halves_unscale(scale[pt]), b[e]);
              acc[ot][pt][4 * q + e] = v;
              top[pt] = fmaxf(top[pt], v);
              least[pt] = min(least[pt], __float_as_uint(v));
            }
        }
      if (!layer)
#pragma unroll
        for (int pt = 0; pt < 2; ++pt) {
          top[pt] = fmaxf(top[pt], __shfl_xor(top[pt], 32, 64));
          if (lane < 32) S.top[wave][32 * pt + lane] = top[pt];
        }
      __syncthreads();  // every wave has read the activations
#pragma unroll
      for (int pt = 0; pt < 2; ++pt) {
        const int point = 32 * pt + l32;
        if (!layer) {
          const float mx = fmaxf(fmaxf(S.top[0][point], S.top[1][point]), fmaxf(S.top[2][point], S.top[3][point]));
          check(mx, least[pt], point < np, [&](float below) {
            int some = 0, lost = 0;
#pragma unroll
            for (int ot = 0; ot < 2; ++ot)
#pragma unroll
              for (int r = 0; r < 16; ++r) {
                some += acc[ot][pt][r] > 0.f;
                lost += acc[ot][pt][r] > 0.f && acc[ot][pt][r] < below;
              }
            const int count = some << 16 | lost;
            return count + __shfl_xor(count, 32, 64);
          });
          scale[pt] = halves_scale(mx);
        }
#pragma unroll
        for (int ot = 0; ot < 2; ++ot)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int c = wave * 64 + 32 * ot + 8 * q + 4 * g;
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = relu(acc[ot][pt][4 * q + e]);
            if (layer) {
#pragma unroll
              for (int e = 0; e < 4; ++e) S.out[c + e][point] = v[e];
            } else {
              put_halves(&S.h[0][point][c], &S.h[1][point][c], v, scale[pt]);
            }
          }
      }
      __syncthreads();
    }
  }
  if (fp32 || S.again) {  // uniform
    __syncthreads();
    point_fp32(w, x, y, z, S.out);
  }
  // max over each run of equal cells (the grid starts at 0 and the outputs are >= 0)
  unsigned int* gp = reinterpret_cast<unsigned int*>(grid) + act_at(0, t, s, kH, gridDim.y);
  const size_t cell_stride = (size_t)kH * gridDim.y;
  int cur = __builtin_amdgcn_readlane(cell, 0);
  float m = 0.f;
  for (int p0 = 0; p0 < np; p0 += 8) {
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = S.out[t][p0 + k];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (p0 + k >= np) break;  // uniform
      const int c = __builtin_amdgcn_readlane(cell, p0 + k);
      if (c != cur) {  // uniform
        atomicMax(gp + cur * cell_stride, __float_as_uint(m));
        cur = c;
        m = 0.f;
      }
      m = fmaxf(m, v[k]);
    }
  }
  atomicMax(gp + cur * cell_stride, __float_as_uint(m));
}

// The halves of a weight matrix P [out][in] (a wave per row): dst[k-step][part][row tile][lane][8], lane l of k-step ks
// of tile ot holding row 32 ot + l % 32, columns 16 ks + 8 (l / 32) + e (0 past in); unscale[row] the inverse of the
// row's power of two.
__global__ __launch_bounds__(64) void halves_kernel(const float* P, int in, int k_steps, unsigned short* dst,
                                                    float* unscale) {
  const int row = blockIdx.x, lane = threadIdx.x, tiles = gridDim.x / 32;
  float mx = 0.f;
  for (int c = lane; c < in; c += 64) mx = fmaxf(mx, fabsf(P[(size_t)row * in + c]));
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) mx = fmaxf(mx, __shfl_xor(mx, d, 64));
  const float up = halves_scale(mx);
  if (lane == 0) unscale[row] = 1.f / up;
  for (int c = lane; c < 16 * k_steps; c += 64) {
    const int ks = c / 16, l = 32 * ((c % 16) / 8) + row % 32;
    const float x = c < in ? P[(size_t)row * in + c] * up : 0.f;
#pragma unroll
    for (int q = 0; q < 2; ++q)
      dst[((size_t)((ks * 2 + q) * tiles + row / 32) * 64 + l) * 8 + c % 8] =
          __builtin_bit_cast(unsigned short, (_Float16)(q ? x - (float)(_Float16)x : x));
  }
}

// Convolutions and transposed convolutions of the U-Net as implicit GEMMs on
// the matrix cores (v_mfma_f32_32x32x2f32): out[s][o][x] = ReLU(b[o] +
// sum_{u, c} W[o][c][u] in(c, u, s, x)) over the 27 taps u and the input
// channels c (the skip concatenation read from two inputs), in(c, u, s, x) =
// input c of shape s at x + u - pad (conv) or x - u + pad (transposed), 0
// outside the grid.  A workgroup owns 32 output channels x 32 output
// columns n = p S + s (p: positions, the middle first); its eight waves take an eighth of the channels each, NP
// pairs of them, over the taps, tap-major.  Columns of a tile are mostly shapes
// at one position, so that a tap outside the grid is skipped for the whole tile
// (of the last layer's taps 70%).  The next tap's operands load while the
// current tap's NP products issue.  The waves' 32 x 32 partial sums meet in LDS
// and are added in wave order (a fixed order: a launch is reproducible bit for
// bit).  Lane layouts of 32x32x2: A[i][k] and B[k][j] with i, j = l % 32 and
// k = l / 32 (here the channel parity); D[i][j] with j = l % 32 and
// i = 8 (r / 4) + 4 (l / 32) + r % 4 for register r.
//
// Both operands lie in memory as a lane reads them: channels 8 q + 2 v + g,
// v = 0..3, of a weight row or a column in one 16-byte load, which serves four
// products.  Bound by the products (FP32 matrix cores): 18 us a layer of 128
// input channels and 32 of 256 at 32 shapes, 46 the last (28 and 56 with a
// 4-byte load per operand and product, which kept the address units busy
// longer than the matrix cores, and 180 the last, its outside taps included).
struct ConvArgs {
  const float* in1;  // act_at() layout, c1 channels, D^3 positions
  int c1;
  const float* in2;  // as in1, c2 channels (the concatenated skip), or null with c2 = 0
  int c2;
  const float* Wt;   // [27][(c1 + c2) / 8][2 g][O][4 v]
  const float* b;    // [O]
  float* out;        // act_at() layout, O channels, Do^3 positions
  int O, D, Do, pad, transposed, n_shapes;
};

constexpr int kConvWaves = 8;

// Position p of n = p S + s: the middle of the grid first, whose taps all lie inside, so that the workgroups with the
// most work start first.
__device__ __forceinline__ int conv_axis(int k, int Do) { return (k & 1) ? Do / 2 + (k >> 1) : Do / 2 - 1 - (k >> 1); }
__device__ __forceinline__ void conv_position(int p, int Do, int& x0, int& x1, int& x2) {
  x0 = conv_axis(p / (Do * Do), Do);
  x1 = conv_axis((p / Do) % Do, Do);
  x2 = conv_axis(p % Do, Do);
}

template <int NP>  // channel pairs per wave: (c1 + c2) = 16 NP
__global__ __launch_bounds__(64 * kConvWaves) void conv_kernel(ConvArgs A) {
  __shared__ float part[kConvWaves][32][33];
  constexpr int NQ = NP / 4;  // 16-byte loads per operand and tap
  const int lane = threadIdx.x & 63, wave = wave_index(), g = lane >> 5, l32 = lane & 31;
  const int D = A.D, Do = A.Do, Do3 = Do * Do * Do, S = A.n_shapes;
  const int N = S * Do3, C = A.c1 + A.c2, O = A.O;
  const int n0 = blockIdx.y * 32, o0 = blockIdx.x * 32;
  // this lane's output column (B column)
  const int n = n0 + l32;
  const bool live = n < N;
  const int sh = live ? n % S : 0;
  int x0, x1, x2;
  conv_position(live ? n / S : 0, Do, x0, x1, x2);
  // this wave's channels c_begin + 2 j + g, all from one input (c1 is a multiple of 2 NP)
  const int c_begin = wave * 2 * NP;
  const bool second = c_begin >= A.c1;
  const int c_in = second ? A.c2 : A.c1, c_own = c_begin - (second ? A.c1 : 0);
  // raw buffer views of the wave's channels and weights: a load past the end reads zeros and no memory, so that a
  // column outside the grid needs neither a branch nor a select
  const float* src = (second ? A.in2 : A.in1) + (size_t)c_own * S;
  const __amdgpu_buffer_rsrc_t in =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(src), (short)0, (c_in * D * D * D - c_own) * S * 4, 0x00020000);
  const __amdgpu_buffer_rsrc_t wts =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(A.Wt), (short)0, 27 * C * O * 4, 0x00020000);
  const unsigned pos_bytes = (unsigned)c_in * S * 4, in_lane = (unsigned)(g * S + sh) * 16;
  const unsigned tap_bytes = (unsigned)C * O * 4, w_lane = (unsigned)((c_begin / 4 + g) * O + o0 + l32) * 16;
  // the taps with an input in the grid for some column of the tile: per axis three bits a column, then their product
  unsigned axis[3];
  {
    const int xs[3] = {x0, x1, x2};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      axis[k] = 0;
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        const int y = A.transposed ? xs[k] - u + A.pad : xs[k] + u - A.pad;
        axis[k] |= (live & ((unsigned)y < (unsigned)D)) ? 1u << u : 0u;
      }
    }
  }
  const unsigned row = (axis[1] & 1 ? axis[2] : 0u) | (axis[1] & 2 ? axis[2] << 3 : 0u) | (axis[1] & 4 ? axis[2] << 6 : 0u);
  const unsigned mine = (axis[0] & 1 ? row : 0u) | (axis[0] & 2 ? row << 9 : 0u) | (axis[0] & 4 ? row << 18 : 0u);
  unsigned taps = mine;
#pragma unroll
  for (int d = 1; d < 32; d <<= 1) taps |= __shfl_xor(taps, d, 64);
  taps = __builtin_amdgcn_readfirstlane(taps);
  const int step = A.transposed ? -1 : 1;
  const int y_base = ((x0 - step * A.pad) * D + (x1 - step * A.pad)) * D + (x2 - step * A.pad);
  auto load = [&](int u, float4 (&a)[NQ], float4 (&b)[NQ]) {  // u past the last tap: zeros
    const int u0 = u / 9, u1 = (u / 3) % 3, u2 = u % 3;       // uniform
    const unsigned y = (unsigned)(y_base + step * ((u0 * D + u1) * D + u2));
    const unsigned b_at = (mine >> u) & 1u ? y * pos_bytes + in_lane : 0x80000000u, w_at = (unsigned)u * tap_bytes + w_lane;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      a[q] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(wts, w_at + (unsigned)(2 * q * O) * 16, 0, 0));
      b[q] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(in, b_at + (unsigned)(2 * q * S) * 16, 0, 0));
    }
  };
  f32x16 acc = f32x16{};
  auto products = [&](const float4 (&a)[NQ], const float4 (&b)[NQ]) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q].x, b[q].x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q].y, b[q].y, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q].z, b[q].z, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q].w, b[q].w, acc, 0, 0, 0);
    }
  };
  // taps in ascending order, the next three loading (counts of taps are mostly multiples of three)
  auto next = [&]() -> int {
    const int u = taps ? __builtin_ctz(taps) : 27;
    taps &= taps - 1;
    return u;
  };
  constexpr int DEPTH = 3;
  const int rounds = (__builtin_popcount(taps) + DEPTH - 1) / DEPTH;
  float4 a[DEPTH][NQ], b[DEPTH][NQ];
#pragma unroll
  for (int d = 0; d < DEPTH; ++d) load(next(), a[d], b[d]);
#pragma unroll 1
  for (int r = 0; r < rounds; ++r)
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      products(a[d], b[d]);
      load(next(), a[d], b[d]);
    }
#pragma unroll
  for (int r = 0; r < 16; ++r) part[wave][8 * (r >> 2) + 4 * g + (r & 3)][l32] = acc[r];
  __syncthreads();
  for (int e = threadIdx.x; e < 8 * 32; e += 64 * kConvWaves) {
    const int j = e & 31, cg = e >> 5;  // column n0 + j; channels o0 + 8 (cg / 2) + 2 v + cg % 2
    const int nn = n0 + j;
    if (nn >= N) continue;
    float4 v4;
    float* v = reinterpret_cast<float*>(&v4);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = 8 * (cg >> 1) + 2 * k + (cg & 1);
      float w = A.b[o0 + i];
#pragma unroll
      for (int q = 0; q < kConvWaves; ++q) w += part[q][i][j];
      v[k] = relu(w);
    }
    int z0, z1, z2;
    conv_position(nn / S, Do, z0, z1, z2);
    *reinterpret_cast<float4*>(A.out + act_at((z0 * Do + z1) * Do + z2, o0 + 8 * (cg >> 1) + (cg & 1), nn % S, O, S)) = v4;
  }
}

// A lane per (shape, channel) of the bottleneck's channels with one q and g.
__global__ __launch_bounds__(64) void global_kernel(const float* c4, float* glob, int n_shapes) {
  const int v = threadIdx.x & 3, s = blockIdx.x * 16 + (threadIdx.x >> 2);
  const int c = 8 * (blockIdx.y >> 1) + 2 * v + (blockIdx.y & 1);
  if (s >= n_shapes) return;
  const float* src = c4 + act_at(0, c, s, kC, n_shapes);
  const size_t stride = (size_t)kC * n_shapes;
  float m = src[0], sum = 0.f;
#pragma unroll 8
  for (int x = 0; x < kB; ++x) {
    const float f = src[x * stride];
    m = f > m ? f : m;
    sum += f;
  }
  glob[(size_t)s * 2 * kC + c] = m;
  glob[(size_t)s * 2 * kC + kC + c] = sum / (float)kB;
}

// E[s][cell][f] = l[f] + L[f] . [d4[s][:][cell], glob[s]]: a workgroup per shape and 16 cells, a thread per cell and
// feature, L transposed in LDS; the global feature's part is the same for every cell and summed once (13 us at 32 shapes;
// 28 with L from memory and that part in every cell).
constexpr int kEmbedCells = 256 / kF;
__global__ __launch_bounds__(256) void embed_kernel(PackedNet w, const float* d4, const float* glob, float* emb,
                                                    int n_shapes) {
  __shared__ float L[3 * kC][kF + 1];
  __shared__ float part[16][kF];
  const int t = threadIdx.x, f = t % kF, c = t / kF;
  const int s = blockIdx.x, cell = blockIdx.y * kEmbedCells + c;
  for (int i = t; i < kF * 3 * kC; i += 256) L[i % (3 * kC)][i / (3 * kC)] = w.L[i];
  __syncthreads();
  {
    const float* gs = glob + (size_t)s * 2 * kC + c * (2 * kC / 16);
    float v = 0.f;
#pragma unroll
    for (int k = 0; k < 2 * kC / 16; ++k) v = fmaf(L[kC + c * (2 * kC / 16) + k][f], gs[k], v);
    part[c][f] = v;
  }
  __syncthreads();
  if (cell >= kCells) return;
  float acc = w.l[f];
#pragma unroll 4
  for (int q = 0; q < kC / 8; ++q) {
    const float4 e = *reinterpret_cast<const float4*>(d4 + act_at(cell, 8 * q, s, kC, n_shapes));
    const float4 o = *reinterpret_cast<const float4*>(d4 + act_at(cell, 8 * q + 1, s, kC, n_shapes));
    const float d[8] = {e.x, o.x, e.y, o.y, e.z, o.z, e.w, o.w};
#pragma unroll
    for (int k = 0; k < 8; ++k) acc = fmaf(L[8 * q + k][f], d[k], acc);
  }
#pragma unroll
  for (int k = 0; k < 16; ++k) acc += part[k][f];
  emb[((size_t)s * kCells + cell) * kF + f] = acc;
}

// Per shape: the cell size s = (hi - lo) / 6 per axis and the margin
// sqrt((s0^2 + s1^2) + s2^2) / 2, float64 (cell centres lo + (i + 1/2) s are
// formed from these where they are used).
__global__ __launch_bounds__(64) void consts_kernel(const Shape* shapes, int n_shapes, double* consts) {
#pragma clang fp contract(off)
  const int s = blockIdx.x * 64 + threadIdx.x;
  if (s >= n_shapes) return;
  const Shape sh = shapes[s];
  double step[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) step[a] = ((double)sh.hi[a] - (double)sh.lo[a]) / (double)kM;
  double* c = consts + (size_t)s * 4;
  c[0] = step[0];
  c[1] = step[1];
  c[2] = step[2];
  c[3] = __builtin_sqrt((step[0] * step[0] + step[1] * step[1]) + step[2] * step[2]) * 0.5;
}

// ------------------------------------------------------------------ pairs --

// Cell selection and mean embeddings: one wave per pair (grid P).  The
// pair's validation, canonical order and float64 relative pose are
// wave-uniform; both objects' cell tests and embedding loads are then issued
// together, and each object's predictor input row [mean (16), pose in the
// other object's frame (12)] goes to the workspace.
__global__ __launch_bounds__(64, 6) void select_kernel(PairArgs A) {
  const int q = blockIdx.x, lane = threadIdx.x;
  if (q >= A.n_pairs) return;
  float* zrow = A.z + (size_t)q * 2 * kIn;
  const int i = A.pairs[2 * q], j = A.pairs[2 * q + 1];
  bool valid = i >= 0 && i < A.n_objs && j >= 0 && j < A.n_objs && i != j;
  const int swp = i > j;
  locc_object oa{}, ob{};
  if (valid) {
    oa = A.objs[swp ? j : i];
    ob = A.objs[swp ? i : j];
    valid = oa.shape >= 0 && oa.shape < A.n_shapes && ob.shape >= 0 && ob.shape < A.n_shapes;
  }
  if (!valid) {  // uniform
    const float nan = __builtin_nanf("");
    if (lane < 2 * kIn / 4) reinterpret_cast<float4*>(zrow)[lane] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (A.pooled && lane < 2 * kF) A.pooled[(size_t)q * 2 * kF + lane] = nan;
    if (lane == 0) {
      A.out[2 * q] = nan;
      A.out[2 * q + 1] = nan;
      if (A.counts) {
        A.counts[2 * q] = -1;
        A.counts[2 * q + 1] = -1;
      }
      A.valid[q] = 0;
      atomicAdd(A.err, 1ull);
    }
    return;
  }
  // float64 relative pose of b in a's frame (the same in every lane)
  double R[9], tt[3];
  {
#pragma clang fp contract(off)
    double Ra[9], Rb[9];
    geo_quat_to_rot(oa.q, Ra);
    geo_quat_to_rot(ob.q, Rb);
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int c = 0; c < 3; ++c) R[3 * r + c] = (Ra[r] * Rb[c] + Ra[3 + r] * Rb[3 + c]) + Ra[6 + r] * Rb[6 + c];
    const double d0 = (double)ob.p[0] - (double)oa.p[0];
    const double d1 = (double)ob.p[1] - (double)oa.p[1];
    const double d2 = (double)ob.p[2] - (double)oa.p[2];
#pragma unroll
    for (int r = 0; r < 3; ++r) tt[r] = (Ra[r] * d0 + Ra[3 + r] * d1) + Ra[6 + r] * d2;
  }
  const Shape box_a = A.shapes[oa.shape], box_b = A.shapes[ob.shape];
  unsigned long long m[2][4];
#pragma unroll
  for (int side = 0; side < 2; ++side) {
    const double* kc = A.consts + (size_t)(side ? ob.shape : oa.shape) * 4;
    const double step[3] = {kc[0], kc[1], kc[2]}, e = kc[3];
    double own_lo[3], lo_w[3], hi_w[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      own_lo[k] = side ? box_b.lo[k] : box_a.lo[k];
      lo_w[k] = (double)(side ? box_a.lo[k] : box_b.lo[k]) - e;
      hi_w[k] = (double)(side ? box_a.hi[k] : box_b.hi[k]) + e;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int k = 64 * r + lane;
      bool in = false;
      if (k < kCells) {
#pragma clang fp contract(off)
        const int ci[3] = {k / (kM * kM), (k / kM) % kM, k % kM};
        double c[3], x[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) c[a] = own_lo[a] + ((double)ci[a] + 0.5) * step[a];
        if (side == 0) {  // a's cell into b's frame: R^T (c - t)
          const double e0 = c[0] - tt[0], e1 = c[1] - tt[1], e2 = c[2] - tt[2];
#pragma unroll
          for (int a = 0; a < 3; ++a) x[a] = (R[a] * e0 + R[3 + a] * e1) + R[6 + a] * e2;
        } else {          // b's cell into a's frame: R c + t
#pragma unroll
          for (int a = 0; a < 3; ++a) x[a] = ((R[3 * a] * c[0] + R[3 * a + 1] * c[1]) + R[3 * a + 2] * c[2]) + tt[a];
        }
        in = (x[0] >= lo_w[0]) & (x[0] <= hi_w[0]) & (x[1] >= lo_w[1]) & (x[1] <= hi_w[1]) & (x[2] >= lo_w[2]) &
             (x[2] <= hi_w[2]);
      }
      m[side][r] = __ballot(in);
    }
  }
  // lane = 4 features (f4) x cell residue g mod 16: float4 loads of the selected cells of both
  // objects, issued together, then sums over the 16 residues by shuffles
  const int f4 = lane & 3, g = lane >> 2;
  float4 acc[2];
#pragma unroll
  for (int side = 0; side < 2; ++side) {
    const float4* E = reinterpret_cast<const float4*>(A.emb + (size_t)(side ? ob.shape : oa.shape) * kCells * kF) + f4;
    acc[side] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int it = 0; it < (kCells + 15) / 16; ++it) {
      const int k = 16 * it + g;  // 16 consecutive cells per step: one ballot word, m[side][it / 4]
      if (k < kCells && ((m[side][it >> 2] >> (k & 63)) & 1ull)) {
        const float4 v = E[k * (kF / 4)];
        acc[side].x += v.x;
        acc[side].y += v.y;
        acc[side].z += v.z;
        acc[side].w += v.w;
      }
    }
  }
#pragma unroll
  for (int side = 0; side < 2; ++side)
#pragma unroll
    for (int d = 4; d < 64; d <<= 1) {
      acc[side].x += __shfl_xor(acc[side].x, d, 64);
      acc[side].y += __shfl_xor(acc[side].y, d, 64);
      acc[side].z += __shfl_xor(acc[side].z, d, 64);
      acc[side].w += __shfl_xor(acc[side].w, d, 64);
    }
  const int count_a = (int)(__popcll(m[0][0]) + __popcll(m[0][1]) + __popcll(m[0][2]) + __popcll(m[0][3]));
  const int count_b = (int)(__popcll(m[1][0]) + __popcll(m[1][1]) + __popcll(m[1][2]) + __popcll(m[1][3]));
  // lanes 0..3 / 4..7: the means of a / b (4 features each)
  const int side = (lane >> 2) & 1;
  if (lane < 8) {
    const float4 sum = side ? acc[1] : acc[0];
    const int cnt = side ? count_b : count_a;
    const float inv = cnt > 0 ? 1.f / (float)cnt : 0.f;
    const float mean[4] = {sum.x * inv, sum.y * inv, sum.z * inv, sum.w * inv};
    const int f0 = 4 * (lane & 3), cpos = side ^ swp;  // the object's position in the caller's pair
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      zrow[side * kIn + f0 + f] = mean[f];
      if (A.pooled) A.pooled[((size_t)q * 2 + cpos) * kF + f0 + f] = mean[f];
    }
  }
  // the poses, written by one lane each with fixed indices: a in b's frame (-R^T t, R^T), b in
  // a's frame (t, R)
  if (lane == 8) {
#pragma clang fp contract(off)
#pragma unroll
    for (int a = 0; a < 3; ++a) zrow[kF + a] = (float)(-((R[a] * tt[0] + R[3 + a] * tt[1]) + R[6 + a] * tt[2]));
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int c = 0; c < 3; ++c) zrow[kF + 3 + 3 * r + c] = (float)R[3 * c + r];
  } else if (lane == 9) {
#pragma unroll
    for (int a = 0; a < 3; ++a) zrow[kIn + kF + a] = (float)tt[a];
#pragma unroll
    for (int a = 0; a < 9; ++a) zrow[kIn + kF + 3 + a] = (float)R[a];
  }
  if (lane == 0) {
    if (A.counts) {
      A.counts[(size_t)q * 2 + swp] = count_a;
      A.counts[(size_t)q * 2 + (swp ^ 1)] = count_b;
    }
    A.valid[q] = 1;
  }
}

constexpr int kTP = 32;                  // pairs per workgroup of the predictor
constexpr int kWaves = 8;                // waves per workgroup, one 16-column stripe each
constexpr int kThreads = 64 * kWaves;
constexpr int kZS = 36;                  // LDS row strides (floats): the inputs padded to 32 columns,
constexpr int kHS = kHP + 4;             // +4 so that 8 consecutive rows start in different banks

struct MlpShared {
  alignas(16) float Z[2 * kTP][kZS];
  alignas(16) float H[2 * kTP][kHS];     // activations, overwritten layer by layer
};

typedef float f32x4 __attribute__((ext_vector_type(4)));

// One layer, Out = ReLU(In W^T + b), over RT row tiles of 16 rows, for this
// wave's 16 output columns c0.. (v_mfma_f32_16x16x4f32).  The reduction index
// is permuted so that each lane reads four consecutive inputs at once: at
// k-step 4u + v, lane group g = lane / 16 holds k = 16u + 4g + v, in A (the
// rows, from LDS) and in B (the weight row W[c0 + lane % 16][...], from L2)
// alike.  K16 = K / 16 rounded up; inputs past K are zero in both.
template <int RT, int K, int K16, int IS>
__device__ __forceinline__ void mfma_layer(const float* In, float* Out, const float* __restrict__ W,
                                           const float* __restrict__ bias, int c0, int lane) {
  const int j = lane & 15, g = lane >> 4;
  float4 b[K16];
#pragma unroll
  for (int u = 0; u < K16; ++u) {
    const int k = 16 * u + 4 * g;
    b[u] = k < K ? *reinterpret_cast<const float4*>(W + (size_t)(c0 + j) * K + k) : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  const float bj = bias[c0 + j];
  f32x4 acc[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) acc[rt] = f32x4{bj, bj, bj, bj};
#pragma unroll
  for (int u = 0; u < K16; ++u) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const float4 a = *reinterpret_cast<const float4*>(In + (rt * 16 + j) * IS + 16 * u + 4 * g);
      acc[rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b[u].x, acc[rt], 0, 0, 0);
      acc[rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, b[u].y, acc[rt], 0, 0, 0);
      acc[rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, b[u].z, acc[rt], 0, 0, 0);
      acc[rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, b[u].w, acc[rt], 0, 0, 0);
    }
  }
  __syncthreads();  // every wave has read In (Out may be the same buffer)
  // D[i][j]: row 4 g + r of the tile, column j
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int r = 0; r < 4; ++r) Out[(rt * 16 + 4 * g + r) * kHS + c0 + j] = relu(acc[rt][r]);
  __syncthreads();
}

// The predictor MLPs of a tile as FP32 products; writes the outputs of the pairs wanted.
__device__ __forceinline__ void mlp_fp32(const PairArgs& A, MlpShared& S, int q0, int n, const int32_t* wanted) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  for (int id = t; id < 2 * kTP * 8; id += kThreads) {  // 64 rows x 8 float4 (28 inputs, zero to 32)
    const int row = id >> 3, c4 = id & 7;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (row < 2 * n && c4 < kIn / 4) v = *reinterpret_cast<const float4*>(A.z + ((size_t)q0 * 2 + row) * kIn + 4 * c4);
    *reinterpret_cast<float4*>(&S.Z[row][4 * c4]) = v;
  }
  __syncthreads();
  const int c0 = 16 * wave;
  const float* H = &S.H[0][0];
  float* Hw = &S.H[0][0];
  mfma_layer<4, kIn, 2, kZS>(&S.Z[0][0], Hw, A.w.A[0], A.w.a[0], c0, lane);
  mfma_layer<4, kHP, kHP / 16, kHS>(H, Hw, A.w.A[1], A.w.a[1], c0, lane);
  mfma_layer<4, kHP, kHP / 16, kHS>(H, Hw, A.w.A[2], A.w.a[2], c0, lane);
  {  // max over the two objects of each pair: rows 2q, 2q + 1 -> row q
    float mx[kTP * kHP / kThreads];
#pragma unroll
    for (int r = 0; r < kTP * kHP / kThreads; ++r) {
      const int id = t + r * kThreads, q = id / kHP, c = id % kHP;
      const float u = S.H[2 * q][c], v = S.H[2 * q + 1][c];
      mx[r] = u > v ? u : v;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kTP * kHP / kThreads; ++r) {
      const int id = t + r * kThreads;
      S.H[id / kHP][id % kHP] = mx[r];
    }
    __syncthreads();
  }
  mfma_layer<2, kHP, kHP / 16, kHS>(H, Hw, A.w.Bw[0], A.w.b[0], c0, lane);
  mfma_layer<2, kHP, kHP / 16, kHS>(H, Hw, A.w.Bw[1], A.w.b[1], c0, lane);
  mfma_layer<2, kHP, kHP / 16, kHS>(H, Hw, A.w.Bw[2], A.w.b[2], c0, lane);
  // output layer and sigmoid: a wave per kTP / kWaves pairs
  const float w_lo = A.w.B4[lane], w_hi = A.w.B4[lane + 64], b4 = A.w.b[3][0];
#pragma unroll
  for (int k = 0; k < kTP / kWaves; ++k) {
    const int q = wave * (kTP / kWaves) + k;
    float v = fmaf(w_lo, S.H[q][lane], w_hi * S.H[q][lane + 64]);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    if (lane == 0 && wanted[q]) {
      const float logit = v + b4;
      A.out[2 * (q0 + q)] = logit;
      A.out[2 * (q0 + q) + 1] = 1.f / (1.f + expf(-logit));
    }
  }
}


// Predictor MLPs: 32 pairs per workgroup; the 64 object rows come from the workspace.  The layers are products of
// halves as in point_mlp_kernel, weights x rows, so that a lane has one row: every row has its own scale at every
// layer, from its largest value (a bound of it through six layers cost the logits half a digit).  A wave has one 32 x 32
// tile of a layer (of the pair layers' 32 rows only four waves), the maximum over a pair's objects is taken between
// neighbouring lanes, and the weights of a layer load while the one before it ends.  A pair with a value past
// kHalvesMost, NaN inputs, or too many inputs of a layer short of bits, is computed as FP32 products after the others,
// and every pair where the weights are short of them (A.fp32).  24.7 us at 16,384 pairs, 13.8 at 8 (as FP32 products on
// 16x16x4 tiles, bound by them, 43 and 21.9); at most 128 registers keep two workgroups per compute unit (134: 32 us).
struct MlpSplitShared {
  unsigned short h[2][2 * kTP][kHP + 8];  // object rows: [part][row][channel]
  unsigned short p[2][kTP][kHP + 8];      // pairs
  float top[4][2 * kTP];                  // a layer's largest output per row and column tile
  float pscale[kTP];                      // the scale of a pair's maximum
  float part[4][kTP];
};

// The products of one 32 x 32 tile: weights (tile ct of the packed halves) x rows 32 rt + l32 of h.
template <int KS>
struct TileWeights {
  u32x4 w[KS][2];
};
template <int KS>
__device__ __forceinline__ void load_tile(const unsigned short* __restrict__ pack, int ct, int lane,
                                          TileWeights<KS>& T) {
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
#pragma unroll
    for (int q = 0; q < 2; ++q)
      T.w[ks][q] = reinterpret_cast<const u32x4*>(pack)[(size_t)((ks * 2 + q) * (kHP / 32) + ct) * 64 + lane];
}
template <int KS, int ROWS>
__device__ __forceinline__ f32x16 tile_products(const TileWeights<KS>& T, const unsigned short (&h)[2][ROWS][kHP + 8],
                                                int row, int g) {
  f32x16 acc = f32x16{};
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    f16x8 b[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) b[q] = *reinterpret_cast<const f16x8*>(&h[q][row][16 * ks + 8 * g]);
#pragma unroll
    for (int part = 2; part >= 0; --part)  // the small products first
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, T.w[ks][part == 2]), b[part == 1], acc, 0, 0, 0);
  }
  return acc;
}
__global__ __launch_bounds__(kThreads, 4) void mlp_kernel(PairArgs A) {
  __shared__ union {
    MlpSplitShared split;
    MlpShared fp32;
  } U;
  __shared__ int32_t valid[kTP], again[kTP], any_again;  // again: valid pairs for the FP32 products
  MlpSplitShared& S = U.split;
  const int t = threadIdx.x, lane = t & 63, wave = wave_index(), g = lane >> 5, l32 = lane & 31;
  const int q0 = blockIdx.x * kTP;
  const int n = A.n_pairs - q0 < kTP ? A.n_pairs - q0 : kTP;  // pairs of this workgroup
  const int ct = wave & 3, rt = wave >> 2;  // this wave's tile of an object layer; waves 0-3 have the pair layers'
  TileWeights<2> w0;
  TileWeights<kHP / 16> w1;
  load_tile<2>(A.w.As[0], ct, lane, w0);
  if (t < kTP) {
    valid[t] = t < n ? A.valid[q0 + t] : 0;
    again[t] = 0;
  }
  if (t == 0) any_again = 0;
  __syncthreads();
  if (A.fp32) {  // uniform
    mlp_fp32(A, U.fp32, q0, n, valid);
    return;
  }
  {  // 64 rows x 8 float4 (28 inputs, zero to 32); a row's eight lanes find its scales
    const int row = t >> 3, c4 = t & 7;
    float4 v4 = make_float4(0.f, 0.f, 0.f, 0.f);
    if (row < 2 * n && c4 < kIn / 4) v4 = *reinterpret_cast<const float4*>(A.z + ((size_t)q0 * 2 + row) * kIn + 4 * c4);
    const float v[4] = {v4.x, v4.y, v4.z, v4.w};
    float top = 0.f, sum = 0.f;  // sum: NaN or inf where an input is
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      top = fmaxf(top, fabsf(v[e]));
      sum += fabsf(v[e]);
    }
#pragma unroll
    for (int d = 1; d < 8; d <<= 1) {
      top = fmaxf(top, __shfl_xor(top, d, 64));
      sum += __shfl_xor(sum, d, 64);
    }
    if (c4 == 0) S.top[0][row] = top;
    bool bad = !(sum < kHalvesMost);
    const float below = kHalvesLeast * halves_unscale(halves_scale(top));
    bool some_short = false;
#pragma unroll
    for (int e = 0; e < 4; ++e) some_short |= (v[e] != 0.f) & (fabsf(v[e]) < below);
    if (__ballot(some_short) != 0) {
      // (the embedding, the offset and the rotation's entries are of different sizes by nature: half of them may be)
      int count = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        count += (v[e] != 0.f ? 1 << 16 : 0) + ((v[e] != 0.f) & (fabsf(v[e]) < below) ? 1 : 0);
#pragma unroll
      for (int d = 1; d < 8; d <<= 1) count += __shfl_xor(count, d, 64);
      bad |= halves_short(count, 2);
    }
    if (bad && c4 == 0 && valid[row >> 1]) again[row >> 1] = any_again = 1;
    put_halves(&S.h[0][row][4 * c4], &S.h[1][row][4 * c4], v, halves_scale(top));
  }
  __syncthreads();
  const int row = 32 * rt + l32;
  float v[4][4];          // a layer's outputs of this lane's row: channels 32 ct + 8 q + 4 g + e
  unsigned least = ~0u;   // bits of the smallest that is not negative (before the ReLU)
  auto outputs = [&](const f32x16& acc, int layer, float scale) {
    const float down = halves_unscale(scale);
    least = ~0u;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c = 32 * ct + 8 * q + 4 * g;
      const float4 u4 = *reinterpret_cast<const float4*>(A.w.us[layer] + c);
      const float4 b4 = *reinterpret_cast<const float4*>((layer < 3 ? A.w.a[layer] : A.w.b[layer - 3]) + c);
      const float u[4] = {u4.x, u4.y, u4.z, u4.w}, b[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[q][e] = fmaf(acc[4 * q + e], u[e] * down, b[e]);
        least = min(least, __float_as_uint(v[q][e]));
        v[q][e] = relu(v[q][e]);
      }
    }
  };
  auto put_tile = [&](auto& h, int r, int q, float scale) {  // v[q] as halves of row r
    put_halves(&h[0][r][32 * ct + 8 * q + 4 * g], &h[1][r][32 * ct + 8 * q + 4 * g], v[q], scale);
  };
  // the largest of v in row r, over the column tiles' waves (a barrier, before which every wave has read the inputs)
  auto row_top = [&](int r, bool mine) -> float {
    float top = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) top = fmaxf(top, v[q][e]);
    top = fmaxf(top, __shfl_xor(top, 32, 64));
    if (mine && lane < 32) S.top[ct][r] = top;
    __syncthreads();
    return fmaxf(fmaxf(S.top[0][r], S.top[1][r]), fmaxf(S.top[2][r], S.top[3][r]));
  };
  auto check = [&](float top, int pair) {
    const float below = kHalvesLeast * halves_unscale(halves_scale(top));
    bool bad = !(top < kHalvesMost);
    if (__ballot((least < __float_as_uint(below)) & (top > 0.f)) != 0) {  // rare: of the wave's 32 channels
      int some = 0, lost = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          some += v[q][e] > 0.f;
          lost += v[q][e] > 0.f && v[q][e] < below;
        }
      int count = some << 16 | lost;
      count += __shfl_xor(count, 32, 64);
      bad |= halves_short(count, kShortActivations);
    }
    if (bad && valid[pair]) again[pair] = any_again = 1;
  };
  float scale = halves_scale(S.top[0][row]);
  f32x16 acc = tile_products<2>(w0, S.h, row, g);
  load_tile<kHP / 16>(A.w.As[1], ct, lane, w1);
  __syncthreads();  // every wave has read the inputs' scales, which the first layer's largest outputs replace
#pragma unroll 1
  for (int layer = 0; layer < 2; ++layer) {
    outputs(acc, layer, scale);
    const float top = row_top(row, true);
    check(top, row >> 1);
    scale = halves_scale(top);
#pragma unroll
    for (int q = 0; q < 4; ++q) put_tile(S.h, row, q, scale);
    __syncthreads();
    acc = tile_products<kHP / 16>(w1, S.h, row, g);
    load_tile<kHP / 16>(layer ? A.w.Bs[0] : A.w.As[2], ct, lane, w1);
  }
  outputs(acc, 2, scale);
  least = ~0u;
#pragma unroll
  for (int q = 0; q < 4; ++q)  // the maximum over the pair's two rows, lanes 2 k and 2 k + 1
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[q][e] = fmaxf(v[q][e], __shfl_xor(v[q][e], 1, 64));
      least = min(least, v[q][e] > 0.f ? __float_as_uint(v[q][e]) : ~0u);
    }
  {
    const float top = row_top(row, true);
    check(top, row >> 1);
    if (!(lane & 1)) {
      if (ct == 0 && g == 0) S.pscale[row >> 1] = halves_scale(top);
#pragma unroll
      for (int q = 0; q < 4; ++q) put_tile(S.p, row >> 1, q, halves_scale(top));
    }
  }
  __syncthreads();
  // pair layers, in place, by waves 0-3 (a lane per pair)
  scale = S.pscale[l32];
#pragma unroll 1
  for (int layer = 0; layer < 2; ++layer) {
    if (wave < 4) {
      acc = tile_products<kHP / 16>(w1, S.p, l32, g);
      load_tile<kHP / 16>(A.w.Bs[layer + 1], ct, lane, w1);
      outputs(acc, 3 + layer, scale);
    }
    const float top = row_top(l32, wave < 4);
    if (wave < 4) {
      check(top, l32);
      scale = halves_scale(top);
#pragma unroll
      for (int q = 0; q < 4; ++q) put_tile(S.p, l32, q, scale);
    }
    __syncthreads();
  }
  if (wave < 4) {  // the last pair layer and the output row's products
    acc = tile_products<kHP / 16>(w1, S.p, l32, g);
    outputs(acc, 5, scale);
    float sum = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 o4 = *reinterpret_cast<const float4*>(A.w.B4 + 32 * ct + 8 * q + 4 * g);
      sum = fmaf(v[q][0], o4.x, fmaf(v[q][1], o4.y, fmaf(v[q][2], o4.z, fmaf(v[q][3], o4.w, sum))));
    }
    sum += __shfl_xor(sum, 32, 64);
    if (lane < 32) S.part[ct][lane] = sum;
  }
  __syncthreads();
  if (t < kTP && valid[t] && !again[t]) {
    const float logit = ((S.part[0][t] + S.part[1][t]) + S.part[2][t]) + S.part[3][t] + A.w.b[3][0];
    A.out[2 * (q0 + t)] = logit;
    A.out[2 * (q0 + t) + 1] = 1.f / (1.f + expf(-logit));
  }
  if (any_again) {  // uniform
    __syncthreads();
    mlp_fp32(A, U.fp32, q0, n, again);
  }
}

}  // namespace

// ------------------------------------------------------------------- host --

namespace {

// Floats of each array of the flat weight vector, in order (W, bias per layer).
constexpr size_t kSizes[] = {
    kH * 3, kH, kH * kH, kH, kH * kH, kH,                                  // point MLP
    (size_t)kC * kH * 27, kC, (size_t)kC * kC * 27, kC, (size_t)kC * kC * 27, kC, (size_t)kC * kC * 27, kC,
    (size_t)kC * kC * 27, kC, (size_t)kC * 2 * kC * 27, kC, (size_t)kC * 2 * kC * 27, kC,
    (size_t)kC * 2 * kC * 27, kC,                                          // U-Net
    (size_t)kF * 3 * kC, kF,                                               // embedding map
    (size_t)kHP * kIn, kHP, (size_t)kHP * kHP, kHP, (size_t)kHP * kHP, kHP,  // per-object MLP
    (size_t)kHP * kHP, kHP, (size_t)kHP * kHP, kHP, (size_t)kHP * kHP, kHP, kHP, 1,  // pair MLP, output
};
constexpr int kArrays = sizeof(kSizes) / sizeof(kSizes[0]);

constexpr size_t total_weights() {
  size_t n = 0;
  for (size_t v : kSizes) n += v;
  return n;
}
static_assert(total_weights() == kWeightCount, "weight count");

void offsets(size_t* off) {
  size_t o = 0;
  for (int i = 0; i < kArrays; ++i) {
    off[i] = o;
    o += kSizes[i];
  }
}

// [rows][cols] -> [cols][rows]
void transpose(const float* src, int rows, int cols, float* dst) {
  for (int r = 0; r < rows; ++r)
    for (int c = 0; c < cols; ++c) dst[(size_t)c * rows + r] = src[(size_t)r * cols + c];
}

// Packed buffer: P2t, P3t, then the U-Net weights transposed to [27][in / 8][2][out][4]:
// C[0..3], D[0..3] (input channels 256, 128, 128, 128, 128, 256, 256, 256).
constexpr int kConvIn[8] = {kH, kC, kC, kC, kC, 2 * kC, 2 * kC, 2 * kC};
constexpr size_t kPackSizes[] = {kH * kH, kH * kH,
                                 (size_t)27 * kH * kC, (size_t)27 * kC * kC, (size_t)27 * kC * kC,
                                 (size_t)27 * kC * kC, (size_t)27 * kC * kC, (size_t)27 * 2 * kC * kC,
                                 (size_t)27 * 2 * kC * kC, (size_t)27 * 2 * kC * kC,
                                 (size_t)kH * kH, kH, (size_t)kH * kH, kH,  // halves of P2 and P3, their rows' scales
                                 (size_t)kHP * 32, kHP, (size_t)kHP * kHP, kHP, (size_t)kHP * kHP, kHP,
                                 (size_t)kHP * kHP, kHP, (size_t)kHP * kHP, kHP, (size_t)kHP * kHP, kHP};  // predictor's

// [O][C][27] -> [27][C / 8][2][O][4]: channel 8 q + 2 v + g at [q][g][.][v]
void conv_transpose(const float* src, int C, float* dst) {
  constexpr int kRow = 4 * kC;  // floats per tap, q and g
  float tile[27][kRow + 16];  // padded: the taps' rows start in different cache sets
  for (int qg = 0; qg < C / 4; ++qg) {
    for (int o = 0; o < kC; ++o)
      for (int v = 0; v < 4; ++v) {
        const float* w = src + ((size_t)o * C + 8 * (qg >> 1) + 2 * v + (qg & 1)) * 27;
        for (int u = 0; u < 27; ++u) tile[u][4 * o + v] = w[u];
      }
    for (int u = 0; u < 27; ++u) std::memcpy(dst + ((size_t)u * (C / 4) + qg) * kRow, tile[u], sizeof(float) * kRow);
  }
}

}  // namespace

size_t packed_floats() {
  size_t n = 0;
  for (size_t v : kPackSizes) n += v;
  return n;
}

void pack_transposed(const float* flat, float* dst) {
  size_t off[kArrays];
  offsets(off);
  float* d = dst;
  transpose(flat + off[2], kH, kH, d);                 // P2
  d += kH * kH;
  transpose(flat + off[4], kH, kH, d);                 // P3
  d += kH * kH;
  for (int i = 0; i < 8; ++i) {                        // U-Net, in the order of kConvIn
    const size_t o = i < 4 ? off[6 + 2 * i] : off[14 + 2 * (i - 4)];
    conv_transpose(flat + o, kConvIn[i], d);
    d += (size_t)27 * kConvIn[i] * kC;
  }
}

// Whether the halves of a matrix have the bits its products need, row by row (halves_kernel scales a row to 2^14 to
// 2^15).  On the bits of the magnitudes, which order like them.
static bool matrix_halves(const float* W, int out, int in) {
  constexpr int kMaxIn = 256;
  uint32_t row[kMaxIn];
  for (int o = 0; o < out; ++o, W += in) {
    std::memcpy(row, W, sizeof(float) * in);
    uint32_t mx = 0;
    for (int c = 0; c < in; ++c) {
      row[c] &= 0x7fffffffu;
      mx = row[c] > mx ? row[c] : mx;
    }
    if (mx >= 217u << 23) return false;  // 2^90
    // kHalvesLeast lies 2^16 below the row's largest power of two; nothing but 0 does below 2^-100 2^-16
    const uint32_t e = mx >> 23, below = ((e > 27u ? e : 27u) - 16u) << 23;
    int some = 0, lost = 0;
    for (int c = 0; c < in; ++c) {
      some += row[c] != 0u;
      lost += (row[c] != 0u) & (row[c] < below);
    }
    if (halves_short(some << 16 | lost, kShortWeights)) return false;
  }
  return true;
}

bool point_halves(const float* flat) {
  size_t off[kArrays];
  offsets(off);
  return matrix_halves(flat + off[2], kH, kH) && matrix_halves(flat + off[4], kH, kH);
}

bool pair_halves(const float* flat) {
  size_t off[kArrays];
  offsets(off);
  for (int i = 0; i < 6; ++i)
    if (!matrix_halves(flat + off[24 + 2 * i], kHP, i ? kHP : kIn)) return false;
  return true;
}

hipError_t launch_halves(const float* raw, float* packed, hipStream_t s) {
  const PackedNet w = packed_view(raw, packed);
  size_t off[kArrays];
  offsets(off);
  auto pack = [&](int array, int out, int in, const unsigned short* dst, const float* unscale) {
    kernel_launch(halves_kernel, dim3(out), dim3(64), 0, s, raw + off[array], in, (in + 15) / 16,
                  const_cast<unsigned short*>(dst), const_cast<float*>(unscale));
  };
  pack(2, kH, kH, w.P2s, w.u2);
  pack(4, kH, kH, w.P3s, w.u3);
  for (int i = 0; i < 6; ++i) pack(24 + 2 * i, kHP, i ? kHP : kIn, i < 3 ? w.As[i] : w.Bs[i - 3], w.us[i]);
  return hipGetLastError();
}

PackedNet packed_view(const float* raw, const float* packed) {
  size_t off[kArrays];
  offsets(off);
  PackedNet w{};
  w.P1 = raw + off[0];
  w.p1 = raw + off[1];
  w.p2 = raw + off[3];
  w.p3 = raw + off[5];
  for (int i = 0; i < 4; ++i) {
    w.k[i] = raw + off[7 + 2 * i];
    w.e[i] = raw + off[15 + 2 * i];
  }
  w.L = raw + off[22];
  w.l = raw + off[23];
  for (int i = 0; i < 3; ++i) {
    w.a[i] = raw + off[25 + 2 * i];
    w.b[i] = raw + off[31 + 2 * i];
  }
  w.B4 = raw + off[36];
  w.b[3] = raw + off[37];
  const float* d = packed;
  w.P2t = d;
  d += kH * kH;
  w.P3t = d;
  d += kH * kH;
  for (int i = 0; i < 8; ++i) {
    (i < 4 ? w.C[i] : w.D[i - 4]) = d;
    d += (size_t)27 * kConvIn[i] * kC;
  }
  w.P2s = reinterpret_cast<const unsigned short*>(d);
  d += kH * kH;
  w.u2 = d;
  d += kH;
  w.P3s = reinterpret_cast<const unsigned short*>(d);
  d += kH * kH;
  w.u3 = d;
  d += kH;
  for (int i = 0; i < 6; ++i) {
    (i < 3 ? w.As[i] : w.Bs[i - 3]) = reinterpret_cast<const unsigned short*>(d);
    d += kHP * (i ? kHP : 32);
    w.us[i] = d;
    d += kHP;
  }
  for (int i = 0; i < 3; ++i) {
    w.A[i] = raw + off[24 + 2 * i];
    w.Bw[i] = raw + off[30 + 2 * i];
  }
  return w;
}

// Floats that order and cell take, to the next 256 bytes (the activations behind them are read 16 bytes at a time).
static size_t encoder_index_floats(size_t n_points) { return (n_points + (n_points + 3) / 4 + 63) / 64 * 64; }

size_t encoder_scratch_floats(int n_shapes, int64_t n_points) {
  const size_t S = (size_t)n_shapes, P = (size_t)n_points;
  return encoder_index_floats(P) + S * kH * kCells + 7 * S * kC * kB + S * kC * kCells + S * 2 * kC;
}

EncoderBuffers encoder_carve(float* base, int n_shapes, int64_t n_points) {
  const size_t S = (size_t)n_shapes, P = (size_t)n_points;
  EncoderBuffers b{};
  float* p = base;
  b.order = reinterpret_cast<int32_t*>(p);
  p += P;
  b.cell = reinterpret_cast<uint8_t*>(p);
  p = base + encoder_index_floats(P);
  b.grid = p;
  p += S * kH * kCells;
  for (int i = 0; i < 4; ++i) {
    b.c[i] = p;
    p += S * kC * kB;
  }
  for (int i = 0; i < 3; ++i) {
    b.d[i] = p;
    p += S * kC * kB;
  }
  b.d4 = p;
  p += S * kC * kCells;
  b.glob = p;
  return b;
}

namespace {

hipError_t conv(const float* in1, int c1, const float* in2, int c2, const float* Wt, const float* bias, float* out,
                int D, int Do, int pad, int transposed, int n_shapes, hipStream_t s) {
  static_assert(kC % 32 == 0, "output channels in tiles of 32");
  const int C = c1 + c2;
  // eight waves of C / 8 channels each, every wave's channels from one input
  if (C % 16 != 0 || c1 % (C / 8) != 0) return hipErrorInvalidValue;
  ConvArgs a{in1, c1, in2, c2, Wt, bias, out, kC, D, Do, pad, transposed, n_shapes};
  const int N = n_shapes * Do * Do * Do;
  const dim3 grid(kC / 32, (unsigned)((N + 31) / 32)), block(64 * kConvWaves);
  switch (C / 16) {
    case 8: kernel_launch(conv_kernel<8>, grid, block, 0, s, a); break;
    case 16: kernel_launch(conv_kernel<16>, grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_encoder(const PackedNet& w, const Shape* shapes, int n_shapes, int max_points, const float* xyz,
                          int64_t n_points, const EncoderBuffers& b, float* emb, double* consts,
                          bool fp32, hipStream_t s) {
  if (n_shapes <= 0 || n_shapes > kEncodeShapes || max_points <= 0) return hipErrorInvalidValue;
  kernel_launch(cell_sort_kernel, dim3(n_shapes), dim3(1024), 0, s, shapes, xyz, n_points, b.order, b.cell);
  kernel_launch(point_mlp_kernel, dim3((max_points + kPts - 1) / kPts, n_shapes), dim3(256), 0, s, w, (int)fp32, shapes,
                xyz, n_points, b.order, b.cell, b.grid);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = conv(b.grid, kH, nullptr, 0, w.C[0], w.k[0], b.c[0], kM, 4, 0, 0, n_shapes, s);
  for (int i = 1; i < 4 && e == hipSuccess; ++i)
    e = conv(b.c[i - 1], kC, nullptr, 0, w.C[i], w.k[i], b.c[i], 4, 4, 1, 0, n_shapes, s);
  if (e == hipSuccess) {
    kernel_launch(global_kernel, dim3((n_shapes + 15) / 16, kC / 4), dim3(64), 0, s, b.c[3], b.glob, n_shapes);
    e = hipGetLastError();
  }
  // transposed convs: on the bottleneck, then on [previous, matching conv output]
  if (e == hipSuccess) e = conv(b.c[3], kC, nullptr, 0, w.D[0], w.e[0], b.d[0], 4, 4, 1, 1, n_shapes, s);
  if (e == hipSuccess) e = conv(b.d[0], kC, b.c[2], kC, w.D[1], w.e[1], b.d[1], 4, 4, 1, 1, n_shapes, s);
  if (e == hipSuccess) e = conv(b.d[1], kC, b.c[1], kC, w.D[2], w.e[2], b.d[2], 4, 4, 1, 1, n_shapes, s);
  if (e == hipSuccess) e = conv(b.d[2], kC, b.c[0], kC, w.D[3], w.e[3], b.d4, 4, kM, 0, 1, n_shapes, s);
  if (e == hipSuccess) {
    kernel_launch(embed_kernel, dim3(n_shapes, (kCells + kEmbedCells - 1) / kEmbedCells), dim3(256), 0, s, w, b.d4,
                  b.glob, emb, n_shapes);
    kernel_launch(consts_kernel, dim3((n_shapes + 63) / 64), dim3(64), 0, s, shapes, n_shapes, consts);
    e = hipGetLastError();
  }
  return e;
}

size_t pair_workspace_bytes(int n_pairs) {
  const size_t P = (size_t)n_pairs;
  return ((P * 2 * kIn * sizeof(float) + 255) & ~size_t(255)) + P * sizeof(int32_t);
}

void pair_workspace_carve(void* base, int n_pairs, PairArgs& a) {
  const size_t P = (size_t)n_pairs;
  a.z = static_cast<float*>(base);
  a.valid = reinterpret_cast<int32_t*>(static_cast<char*>(base) + ((P * 2 * kIn * sizeof(float) + 255) & ~size_t(255)));
}

hipError_t launch_pairs(const PairArgs& a, hipStream_t s) {
  if (a.n_pairs <= 0) return hipSuccess;
  if (!a.z || !a.valid) return hipErrorInvalidValue;
  kernel_launch(select_kernel, dim3(a.n_pairs), dim3(64), 0, s, a);
  kernel_launch(mlp_kernel, dim3((a.n_pairs + kTP - 1) / kTP), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace vox
}  // namespace locc
