// Spatial clusters of every shape's points, built once when a library is uploaded: the leaves of a kd-tree that halves
// the number of clusters along the widest axis.  One workgroup per shape; a level of the tree is one bitonic sort in
// LDS of (segment, coordinate on the segment's widest axis, stored index), so that a segment's lower half precedes its
// upper half.  A shape of 4,096 points takes 6 levels; built on the host, 128 of them took 37 ms.
#include "geometry.h"

namespace locc {
namespace {

constexpr int kMaxClusters = kMaxShapePoints / kClusterPoints;
constexpr int kClusterThreads = 1024;

// unsigned integers in the order of the (finite) floats, and back
__device__ __forceinline__ unsigned float_key(float f) {
  const unsigned b = __float_as_uint(f);
  return b & 0x80000000u ? ~b : b | 0x80000000u;
}
__device__ __forceinline__ float key_float(unsigned k) {
  return __uint_as_float(k & 0x80000000u ? k & 0x7fffffffu : ~k);
}

struct ClusterShared {
  unsigned lo[kMaxClusters][3], hi[kMaxClusters][3];  // box of the segment that starts at this cluster
  uint16_t start[kMaxClusters], len[kMaxClusters];    // each cluster's segment: first cluster, clusters
  uint16_t axis[kMaxClusters];                        // a segment's widest axis
};

__global__ __launch_bounds__(kClusterThreads) void cluster_kernel(const ShapeDesc* __restrict__ shapes,
                                                                  const float* __restrict__ xyz, int64_t n_points,
                                                                  float4* __restrict__ boxes,
                                                                  char* __restrict__ clusters) {
  __shared__ ClusterShared S;
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned long long* key = reinterpret_cast<unsigned long long*>(smem);
  const int s = blockIdx.x, tid = threadIdx.x, NT = kClusterThreads;
  const int n = shapes[s].n, off = shapes[s].off;
  const int nc = (n + kClusterPoints - 1) / kClusterPoints;
  int n2 = kClusterPoints;
  while (n2 < n) n2 *= 2;
  auto axis_of = [&](int p, int k) { return xyz[(size_t)k * n_points + off + p]; };

  for (int i = tid; i < n2; i += NT) key[i] = i < n ? (unsigned long long)i : ~0ull;
  for (int c = tid; c < nc; c += NT) {
    S.start[c] = 0;
    S.len[c] = (uint16_t)nc;
  }
  for (int most = nc; most > 1; most = (most + 1) / 2) {  // clusters in the largest segment
    for (int c = tid; c < nc; c += NT)
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        S.lo[c][k] = ~0u;
        S.hi[c][k] = 0u;
      }
    __syncthreads();
    for (int i = tid; i < n; i += NT) {
      const int st = S.start[i / kClusterPoints];
      const int p = (int)(key[i] & 0x3fff);
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const unsigned x = float_key(axis_of(p, k));
        atomicMin(&S.lo[st][k], x);
        atomicMax(&S.hi[st][k], x);
      }
    }
    __syncthreads();
    for (int c = tid; c < nc; c += NT) {
      if (S.start[c] != c) continue;
      float w[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) w[k] = key_float(S.hi[c][k]) - key_float(S.lo[c][k]);
      int axis = 0;
      if (w[1] > w[0]) axis = 1;
      if (w[2] > w[axis]) axis = 2;
      S.axis[c] = (uint16_t)axis;
    }
    __syncthreads();
    for (int i = tid; i < n; i += NT) {
      const int st = S.start[i / kClusterPoints];
      const int p = (int)(key[i] & 0x3fff);
      key[i] = (unsigned long long)st << 46 | (unsigned long long)float_key(axis_of(p, S.axis[st])) << 14 |
               (unsigned long long)p;
    }
    __syncthreads();
    for (int size = 2; size <= n2; size *= 2)
      for (int step = size / 2; step > 0; step /= 2) {
        for (int e = tid; e < n2 / 2; e += NT) {
          const int i = 2 * e - (e & (step - 1)), j = i + step;
          const unsigned long long a = key[i], b = key[j];
          if ((a > b) == ((i & size) == 0)) {
            key[i] = b;
            key[j] = a;
          }
        }
        __syncthreads();
      }
    for (int c = tid; c < nc; c += NT) {
      const int st = S.start[c], len = S.len[c], left = len / 2;
      if (len > 1) {
        S.start[c] = (uint16_t)(c < st + left ? st : st + left);
        S.len[c] = (uint16_t)(c < st + left ? left : len - left);
      }
    }
  }
  __syncthreads();

  const size_t first = (size_t)(off / kClusterPoints) + s;
  const int lane = tid & 63;
  for (int c = wave_index(); c < nc; c += NT / 64) {
    const int i = c * kClusterPoints + lane;
    const int p = (int)(key[i < n ? i : c * kClusterPoints] & 0x3fff);
    float x[3];
    char* dst = clusters + (first + c) * kClusterBytes;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      x[k] = axis_of(p, k);
      reinterpret_cast<float*>(dst)[64 * k + lane] = x[k];
    }
    reinterpret_cast<uint16_t*>(dst + 768)[lane] = (uint16_t)(i < n ? p : kNoPoint);
    float lo[3], hi[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      lo[k] = hi[k] = x[k];
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        lo[k] = fminf(lo[k], __shfl_xor(lo[k], d, 64));
        hi[k] = fmaxf(hi[k], __shfl_xor(hi[k], d, 64));
      }
    }
    if (lane == 0) {
      boxes[2 * (first + c)] = make_float4(lo[0], lo[1], lo[2], 0.f);
      boxes[2 * (first + c) + 1] = make_float4(hi[0], hi[1], hi[2], 0.f);
    }
  }
}

__global__ __launch_bounds__(256) void rows_kernel(const float* __restrict__ points, int64_t n_points,
                                                   float4* __restrict__ rows) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n_points) return;
  const float* n = points + 3 * n_points + 3 * i;
  rows[2 * i] = make_float4(points[i], points[n_points + i], points[2 * n_points + i], n[0]);
  rows[2 * i + 1] = make_float4(n[1], n[2], 0.f, 0.f);
}

}  // namespace

hipError_t launch_rows(const float* points, int64_t n_points, float4* rows, hipStream_t s) {
  if (n_points <= 0) return hipErrorInvalidValue;
  kernel_launch(rows_kernel, dim3((unsigned)((n_points + 255) / 256)), dim3(256), 0, s, points, n_points, rows);
  return hipGetLastError();
}

hipError_t launch_clusters(const ShapeDesc* shapes, int n_shapes, int max_points, const float* xyz, int64_t n_points,
                           float4* boxes, char* clusters, hipStream_t s) {
  if (n_shapes <= 0 || max_points <= 0 || max_points > kMaxShapePoints) return hipErrorInvalidValue;
  size_t n2 = kClusterPoints;
  while (n2 < (size_t)max_points) n2 *= 2;
  const size_t smem = n2 * sizeof(unsigned long long);
  static_assert(kMaxShapePoints * sizeof(unsigned long long) + sizeof(ClusterShared) <= 160 * 1024, "LDS");
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&cluster_kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (e != hipSuccess) return e;
  kernel_launch(cluster_kernel, dim3(n_shapes), dim3(kClusterThreads), smem, s, shapes, xyz, n_points, boxes,
                clusters);
  return hipGetLastError();
}

}  // namespace locc
