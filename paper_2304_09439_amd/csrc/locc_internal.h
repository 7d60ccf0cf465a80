// Internal declarations shared by the library's translation units.
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "locc.h"
#include "pack.h"

namespace locc {

// Per-kernel timing without marker packets: while a profiled step is being
// enqueued on this host thread, its first kernel records `start` as its
// dispatch begins and every kernel records `stop` as it ends (events attached
// to the dispatches themselves, so the timing adds no work between kernels).
struct LaunchTiming {
  hipEvent_t start = nullptr;
  hipEvent_t stop = nullptr;
};
extern thread_local LaunchTiming g_launch_timing;

// Every kernel of the library is launched through this.
template <class F, class... Args>
inline void kernel_launch(F kernel, const dim3& grid, const dim3& block, uint32_t shmem, hipStream_t s,
                          Args... args) {
  LaunchTiming& t = g_launch_timing;
  if (!t.stop) {
    hipLaunchKernelGGL(kernel, grid, block, shmem, s, args...);
    return;
  }
  hipExtLaunchKernelGGL(kernel, grid, block, shmem, s, t.start, t.stop, 0u, args...);
  t.start = nullptr;
}

// Per-shape descriptor in device memory: rows [off, off + n) of the SoA point
// arrays, and the axis-aligned box of the stored xyz (min / max).  32 bytes.
struct ShapeDesc {
  int32_t off;
  int32_t n;
  float lo[3];
  float hi[3];
};
static_assert(sizeof(ShapeDesc) == 32, "ShapeDesc layout");

// Per-pair record written by the crop step and read by the network steps.
//   a        canonical first object (min(i, j)), or -1 for an invalid pair
//   swapped  1 if the caller gave (b, a)
//   m_a, m_b number of valid encoder rows (min(count, K)) per object
struct PairMeta {
  int32_t a;
  int32_t swapped;
  int32_t m_a;
  int32_t m_b;
};
static_assert(sizeof(PairMeta) == 16, "PairMeta layout");

// Largest point count per shape (the crop step keeps one 64-bit membership
// mask per 64 points of each object in LDS).
constexpr int kMaxShapePoints = 16384;
constexpr int kMaxK = 256;
// Encoder input rows: 8 floats (x, y, z, nx, ny, nz, 1, 0) stored in the
// order (e0, e2, e4, e6, e1, e3, e5, e7) so that each half-wave of a 32x32x2
// MFMA operand load reads one float4.  e7, which layer 1 gives a zero weight,
// is in the rows of an object the power of two, at most 1, that takes all their
// normals, and coordinates in the library's unit, into [-1, 1] (0: none does),
// for the products of halves.
constexpr int kRowFloats = 8;

struct DeviceLibrary {
  const ShapeDesc* shapes;
  int32_t n_shapes;
  float per_unit;          // a power of two: most shapes' coordinates times it lie in [-1/2, 1/2]
  const float* points;     // x, y and z, each n_points floats, then the normals
  int64_t n_points;
  const float4* rows;      // or null: the same once more, two a point: x, y, z, nx | ny, nz, 0, 0, for gathers
  // spatial clusters (clusters.hip), or null: the box of cluster c in boxes[2 c] (lo) and boxes[2 c + 1] (hi), its
  // points at points + c * kClusterBytes
  const float4* boxes;
  const char* clusters;

  __device__ const float* coordinate(int k) const { return points + k * n_points; }
  __device__ const float3* normals() const { return reinterpret_cast<const float3*>(coordinate(3)); }
};

// A shape's points once more, as clusters of 64 close to each other (the last one padded by copies of a point with
// index kNoPoint): 64 x, 64 y, 64 z, 64 16-bit indices into the shape's stored points.  Cluster k of shape s, whose
// stored points begin at off, is number off / 64 + s + k.
constexpr int kClusterPoints = 64;
constexpr size_t kClusterBytes = 64 * (3 * 4 + 2);
constexpr unsigned kNoPoint = 0xffff;
inline size_t cluster_count(int64_t n_points, int n_shapes) { return (size_t)(n_points / 64) + n_shapes + 1; }
// The clusters of every shape of a library from its coordinates (finite; xyz: all x, all y, all z); boxes and clusters
// of cluster_count().
hipError_t launch_clusters(const ShapeDesc* shapes, int n_shapes, int max_points, const float* xyz, int64_t n_points,
                           float4* boxes, char* clusters, hipStream_t s);

// DeviceLibrary::rows from the coordinates and normals.
hipError_t launch_rows(const float* points, int64_t n_points, float4* rows, hipStream_t s);

// Pair count of a launch: n_pairs is the capacity (grid sizing); when
// n_pairs_dev is set the kernels read the actual count from device memory
// (clamped to the capacity), so one captured graph serves steps whose pair
// counts differ.  A launch over a chunk that starts at pair `base` of the
// step sees *dev - base pairs, clamped to [0, capacity].
__device__ __forceinline__ int pair_count(int capacity, const int32_t* dev, int base = 0) {
  if (!dev) return capacity;
  const int n = *dev - base;
  return n < 0 ? 0 : (n < capacity ? n : capacity);
}

struct CropArgs {
  const locc_object* objs;
  int32_t n_objs;
  const int32_t* pairs;
  int32_t n_pairs;
  const int32_t* n_pairs_dev;  // or null
  DeviceLibrary lib;
  int32_t K;
  double pad;
  int32_t* idx_out;      // [P][2][K] caller order, may be null
  int32_t* counts_out;   // [P][2] caller order, may be null
  PairMeta* meta;        // [P], may be null
  float* rows;           // [P][2K][8], may be null
  unsigned short* rows_bf16;  // [P][2K][8] bf16 (x, y, z, nx, ny, nz, 1, 0), rows up to the next
                              // multiple of 32 of each object's count written, may be null
  unsigned long long* err_counter;
  void* setup;           // [P] records of kPairSetupBytes (library workspace), required
  int32_t dev_base;      // first pair of this launch within the step (device count mode)
  int32_t cluster_min;   // set by launch_crop: shapes of more points are scanned by clusters where that is less work
};
// Read from host memory at every launch: a fourth line of 64 bytes makes a small batch 0.3 to 0.5 us longer (10 pairs at
// 64 / 128 14.6 us, 14.1 without).
static_assert(sizeof(CropArgs) <= 192, "crop arguments");

// Bytes of the per-pair record (pose, box, screening constants, canonical
// order) the pair set-up kernel writes for the crop kernel.
constexpr size_t kPairSetupBytes = 320;

// Pair set-up (one thread per pair), then the crop (one wave per object of a
// pair, the two waves of a pair in one workgroup).  unroll (2, 4 or 8): a
// wave issues the loads of max(1, unroll / 4) blocks of 256 points together.
hipError_t launch_crop(const CropArgs& args, hipStream_t s, int unroll = 8);

// Broad phase over environments: world boxes, then every overlapping pair
// i < j of objects of the same environment (see broad_phase.hip).
struct BroadArgs {
  const locc_object* objs;
  int32_t n_objs;
  const int32_t* env_offsets;  // [n_envs + 1]
  int32_t n_envs;
  DeviceLibrary lib;
  double* boxes;               // [n_objs][6] lo xyz, hi xyz (scratch)
  long long* env_count;        // [n_envs] overlapping pairs per environment (scratch)
  long long* env_start;        // [n_envs] first output position per environment (scratch)
  int32_t* pairs;              // [capacity][2], may be null when capacity is 0
  int32_t capacity;
  int32_t* count;              // [2]: pairs written, total (saturated)
};

// Scratch bytes of a broad phase over n_objs objects and n_envs environments.
size_t broad_phase_scratch_bytes(int n_objs, int n_envs);
// Carves the scratch at `base` into a.boxes / env_count / env_start.
void broad_phase_carve(void* base, int n_objs, int n_envs, BroadArgs& a);
// Four launches on s: world boxes, per-environment counts, the scan (which
// writes count), the ordered write of the pairs.
hipError_t launch_broad_phase(const BroadArgs& a, hipStream_t s);

// FP32 network weights packed in MFMA fragment order, for net_split.hip.
struct Fp32Net {
  int h1, h2, hh;
  const float* w1pack;  // [h1/32][4][64]
  const float* w2pack;  // [4 waves][h2/128][h1/2][64]
  const float* b2;      // [h2]
  const float* h1pack;  // [hh/32][h2][64]   (k-steps = 2*h2 / 2)
  const float* c1;      // [hh]
  const float* h2pack;  // [hh/32][hh/2][64]
  const float* c2;      // [hh]
  const float* h3;      // [8][hh] plain row-major
  const float* c3;      // [8]
  // both halves of every weight of W2, H1 and H2 in 32x32x16 B operand order, rows times powers of two, and the
  // factors that undo them (net_split.hip)
  const float* w1s;           // w1pack, rows times powers of two
  const float* w1c;           // [h1][8]: W1's rows, bias, 0, in the order of layer 2's reduction
  const float* w2c;           // [h1][h2]: W2^T in that order
  const unsigned short* w2s;  // [2][h2/32][h1/16][64][8]
  const unsigned short* h1s;  // [2][hh/32][2 h2/16][64][8]
  const unsigned short* h2s;  // [2][hh/32][hh/16][64][8]
  const unsigned short* h3s;  // [2][hh/16][64][8] (8 rows, zero to 32)
  const float* unscale2;      // [h2]
  const float* unscale_h1;    // [hh]
  const float* unscale_h2;    // [hh]
  const float* unscale_h3;    // [8]
  const int32_t* split_bad;   // not 0: a weight is not finite, or a row has too many short of bits: no halves
};

struct NetArgs {
  const float* rows;      // [P][2K][8]
  const PairMeta* meta;   // [P]
  const locc_object* objs;
  int32_t n_pairs;
  const int32_t* n_pairs_dev;  // or null
  int32_t K;
  float* z;               // [P][2 h2] workspace (always written)
  float* y_dbg;           // [P][8] or null
  locc_contact* out;      // [P]
  uint8_t* amax;          // [P][2][h2] row of the largest raw layer-2 sum per channel (first on ties), or null
  unsigned int* queue;    // launch_encoder_split: [2], 0 between launches, or null (static order)
  uint32_t* doubt;        // [P][2][h2/32]: with amax, a bit per channel whose row is not certain
};

// The encoder, layer 2 as products of halves: the pooled features (z, may be
// null with amax) and, with amax, the argmax rows and which are in doubt.
hipError_t launch_encoder_split(const Fp32Net& w, const NetArgs& a, int n_cu, hipStream_t s);

// From those rows the features of one FP32 chain per sum, and the rows in doubt
// decided by it.
hipError_t launch_chain_features(const Fp32Net& w, const NetArgs& a, hipStream_t s);

// The head on the features in z (products of halves).
hipError_t launch_head_split(const Fp32Net& w, const NetArgs& a, int n_cu, hipStream_t s);

// Largest finite half: a float up to it has finite halves.
constexpr float kSplitLimit = 65504.f;

// Chunks of pairs a workgroup of the split encoder claims: level l holds
// claims[l] chunks of size[l] pairs from pair base[l] on (the last level as
// many as it takes).
constexpr int kSplitChunk = 32;
struct SplitChunks {
  static constexpr int kLevels = 8;
  int32_t grid;
  int32_t size[kLevels], base[kLevels], claims[kLevels];
};
__host__ __device__ inline void split_chunk(const SplitChunks& c, int claim, int& base, int& n) {
  int l = 0;
#pragma unroll
  for (int k = 0; k + 1 < SplitChunks::kLevels; ++k)
    if (l == k && claim >= c.claims[k]) {
      claim -= c.claims[k];
      l = k + 1;
    }
  base = 0x7fffffff;
  n = 0;
#pragma unroll
  for (int k = 0; k < SplitChunks::kLevels; ++k)
    if (l == k) {
      n = c.size[k];
      const long long at = c.base[k] + (long long)claim * n;
      if (at < base) base = (int)at;
    }
}

// Device views of the halves (split_layout() in pack.h at base).
void split_bind(Fp32Net& w, const char* base);

// Repacking on the device from the flat weights raw: pack[i] = raw[pack_idx[i]]
// (0 where the index is negative), the head's matrices in the gradient
// kernels' order at frag (H1 [hh][2 h2], H2 [hh][hh], H2^T, H1^T), and the
// halves and their rows' factors at split (its flag word zero before).
struct RepackArgs {
  const float* raw;
  int32_t h1, h2, hh;
  float* pack;
  const int32_t* pack_idx;
  int32_t pack_n;
  float* frag;
  char* split;
  float unit;  // of the library's coordinates (1 / DeviceLibrary::per_unit)
};
hipError_t launch_repack(const RepackArgs& a, hipStream_t s);

// Device views of the FP32 weights packed by fp32_pack (pack.h).
Fp32Net fp32_view(const float* dev_base, int h1, int h2, int hh);

}  // namespace locc
