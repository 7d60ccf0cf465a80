// The bf16 head on the pooled features that an encoder kernel (fused.hip, fused_fp8.hip) left in memory: a workgroup of
// HH / 64 waves per 32 RT pairs, two column tiles per wave, every layer in place in LDS.
//
// Bound by the stream of the head's weights (1 MB at width 512) from L2 into each compute unit: about 10 us of the
// 12.7 us that 8 pairs take (one workgroup), 14.1 us at 1,061.  Two row tiles per workgroup halve that stream once
// every compute unit has a tile, and two workgroups per unit overlap their barriers: 27 us at 16,384 pairs (one row
// tile: 37).  Four row tiles fill the LDS with one workgroup and were slower (210,040 pairs: 285 us
// against 242), more k-steps in flight than four changed nothing, nor did another order of the fragments.
#include "fused.h"
#include "geometry.h"
#include "head_bf16.h"
#include "post.h"

namespace locc {
namespace {

using head_bf16::f32x16;
using head_bf16::u16x8;

// The first D k-steps of a layer's weight fragments for this wave's two column tiles.
template <int KDIM, int D>
__device__ __forceinline__ void prefetch(const unsigned short* __restrict__ pack, u16x8 (&bq)[D][2]) {
  constexpr int KS = KDIM / 16;
  const u16x8* bp = reinterpret_cast<const u16x8*>(pack) + (size_t)wave_index() * 2 * KS * 64 + (threadIdx.x & 63);
#pragma unroll
  for (int d = 0; d < D; ++d)
#pragma unroll
    for (int c = 0; c < 2; ++c) bq[d][c] = bp[((size_t)c * KS + d) * 64];
}

// One hidden layer of RT row tiles in place: buf = bf16(ReLU(buf W^T + bias)), rows of stride SS; this wave's two
// column tiles, its first fragments in bq.  Every output sums the same products in the same order for every RT.
// next() runs between the products and the barrier that ends the reads of buf.
template <int KDIM, int SS, int RT, int D, class Next>
__device__ __forceinline__ void layer_in_place(const unsigned short* __restrict__ pack, const float* __restrict__ bias,
                                               unsigned short* buf, u16x8 (&bq)[D][2], Next next) {
  constexpr int KS = KDIM / 16;
  static_assert(KS % D == 0, "k-steps per head layer");
  const int lane = threadIdx.x & 63, wave = wave_index(), g = lane >> 5, l32 = lane & 31;
  const u16x8* bp = reinterpret_cast<const u16x8*>(pack) + (size_t)wave * 2 * KS * 64 + lane;
  const unsigned short* arow = buf + l32 * SS + 8 * g;
  f32x16 acc[RT][2];
#pragma unroll
  for (int r = 0; r < RT; ++r) acc[r][0] = acc[r][1] = f32x16{};
  float bc[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) bc[c] = bias[(wave * 2 + c) * 32 + l32];
#pragma unroll 1
  for (int s0 = 0; s0 < KS; s0 += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int s = s0 + d;
      u16x8 av[RT];
#pragma unroll
      for (int r = 0; r < RT; ++r) av[r] = *reinterpret_cast<const u16x8*>(arow + r * 32 * SS + 16 * s);
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int c = 0; c < 2; ++c) acc[r][c] = head_bf16::mfma(av[r], bq[d][c], acc[r][c]);
      if (s0 + D < KS) {
#pragma unroll
        for (int c = 0; c < 2; ++c) bq[d][c] = bp[((size_t)c * KS + s + D) * 64];
      }
    }
  }
  next();
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int col = (wave * 2 + c) * 32 + l32;
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        buf[(32 * t + 8 * (r >> 2) + 4 * g + (r & 3)) * SS + col] = head_bf16::bits(fmaxf(acc[t][c][r] + bc[c], 0.f));
  }
  __syncthreads();
}

template <int H2, int HH, int RT>
constexpr size_t head_smem() {
  return sizeof(unsigned short) * 32 * RT * ((2 * H2 > HH ? 2 * H2 : HH) + 8) + sizeof(float) * 4 * 32 * RT * 8;
}

template <int H2, int HH, int RT>
__global__ __launch_bounds__(HH, RT == 1 ? 2 : 4) void head_bf16_kernel(HeadBf16Args A) {
  constexpr int T = 32 * RT, NW = HH / 64, KS3 = HH / 16;
  constexpr int ZS = (2 * H2 > HH ? 2 * H2 : HH) + 8;
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned short* z = reinterpret_cast<unsigned short*>(smem);
  float* y = reinterpret_cast<float*>(z + T * ZS);  // [quarter][row][8]
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_index(), g = lane >> 5, l32 = lane & 31;
  const int p0 = blockIdx.x * T;
  const int P = pair_count(A.n_pairs, A.n_pairs_dev, A.dev_base);
  if (p0 >= P) return;  // uniform
  const int n = P - p0 < T ? P - p0 : T;
  constexpr int D = RT == 1 ? 8 : 4;
  u16x8 bq[D][2];
  prefetch<2 * H2, D>(A.h1p, bq);
  for (int e = tid; e < T * (2 * H2 / 8); e += HH) {
    const int i = e / (2 * H2 / 8), k = e % (2 * H2 / 8);
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (i < n) v = reinterpret_cast<const uint4*>(A.z16 + (size_t)(p0 + i) * A.z_stride)[k];
    *reinterpret_cast<uint4*>(z + i * ZS + 8 * k) = v;
  }
  __syncthreads();
  layer_in_place<2 * H2, ZS, RT, D>(A.h1p, A.c1, z, bq, [&] { prefetch<HH, D>(A.h2p, bq); });
  layer_in_place<HH, ZS, RT, D>(A.h2p, A.c2, z, bq, [] {});
  // layer 3 (8 outputs, padded to 32 columns): a quarter of the reduction of a row tile per task
  const u16x8* bp = reinterpret_cast<const u16x8*>(A.h3p) + lane;
  for (int task = wave; task < 4 * RT; task += NW) {
    const int q = task & 3, t = task >> 2;
    const unsigned short* arow = z + (32 * t + l32) * ZS + 8 * g;
    f32x16 acc = f32x16{};
#pragma unroll
    for (int s = 0; s < KS3 / 4; ++s)
      acc = head_bf16::mfma(*reinterpret_cast<const u16x8*>(arow + 16 * (q * (KS3 / 4) + s)),
                            bp[(size_t)(q * (KS3 / 4) + s) * 64], acc);
    if (l32 < 8)
#pragma unroll
      for (int r = 0; r < 16; ++r) y[(q * T + 32 * t + 8 * (r >> 2) + 4 * g + (r & 3)) * 8 + l32] = acc[r];
  }
  __syncthreads();
  for (int e = tid; e < T * 8; e += HH) {
    const int j = e & 7;
    y[e] = ((y[e] + y[T * 8 + e]) + y[2 * T * 8 + e]) + y[3 * T * 8 + e] + A.c3[j];
  }
  __syncthreads();
  for (int i = tid; i < n; i += HH) {
    const PairMeta mt = A.meta[p0 + i];
    post_contact(A.objs, mt.a, mt.swapped, y + 8 * i, A.out, A.y_dbg, p0 + i);
  }
}

template <int H2, int HH, int RT>
hipError_t run(const HeadBf16Args& a, hipStream_t s) {
  constexpr size_t smem = head_smem<H2, HH, RT>();
  static_assert(smem <= 160 * 1024, "LDS");
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&head_bf16_kernel<H2, HH, RT>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (e != hipSuccess) return e;
  kernel_launch((head_bf16_kernel<H2, HH, RT>), dim3((a.n_pairs + 32 * RT - 1) / (32 * RT)), dim3(HH), smem, s, a);
  return hipGetLastError();
}

template <int H2, int HH>
hipError_t pick(const HeadBf16Args& a, int n_cu, hipStream_t s) {
  // the whole step with one tile and with two: 5,000 pairs 104.5 and 110.1 us, 8,000 138.7 and 143.6, 12,000 196.1 and 193.5
  return a.n_pairs <= 32 * n_cu ? run<H2, HH, 1>(a, s) : run<H2, HH, 2>(a, s);
}

}  // namespace

hipError_t launch_head_bf16(const HeadBf16Args& a, int h2, int hh, int n_cu, hipStream_t s) {
  if (a.n_pairs <= 0) return hipSuccess;
  if (h2 == 256 && hh == 512) return pick<256, 512>(a, n_cu, s);
  return hipErrorInvalidValue;
}

}  // namespace locc
