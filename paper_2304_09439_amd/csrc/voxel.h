// Internal declarations of the voxel-embedding variant (voxel.hip, voxel_capi.cpp).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "locc_voxel.h"

namespace locc {
namespace vox {

constexpr int kM = 6;              // grid cells per axis
constexpr int kCells = kM * kM * kM;
constexpr int kH = 256;            // point MLP width
constexpr int kC = 128;            // U-Net channels
constexpr int kB = 4 * 4 * 4;      // bottleneck cells
constexpr int kF = 16;             // embedding width
constexpr int kHP = 128;           // predictor width
constexpr int kIn = kF + 12;       // predictor input per object
constexpr int kMaxPoints = 65536;  // per shape
constexpr size_t kWeightCount = 5534609;

// Per-shape record: rows [off, off + n) of the SoA xyz, and the box of the stored xyz.
struct Shape {
  int32_t off;
  int32_t n;
  float lo[3];
  float hi[3];
};
static_assert(sizeof(Shape) == 32, "Shape layout");

// Device pointers to every weight array: the flat vector as uploaded, except
// the point MLP's layers 2-3, used transposed to [in][out] (a coalesced row
// of outputs per input), and the U-Net's weights, used as
// [27 taps][in / 8][2][out][4] (input channel 8 q + 2 v + g at [q][g][.][v]),
// both from a second, packed buffer.
struct PackedNet {
  const float *P1, *p1, *P2t, *p2, *P3t, *p3;  // point MLP
  const unsigned short *P2s, *P3s;             // layers 2-3 as halves (halves_kernel), with their rows'
  const float *u2, *u3;                        // inverse scales
  const unsigned short *As[3], *Bs[3];         // the predictor's MLPs as halves, with their rows' inverse scales
  const float* us[6];
  const float *C[4], *k[4], *D[4], *e[4];      // U-Net convs, transposed convs (C, D: [27][in / 8][2][128][4])
  const float *L, *l;                          // embedding map [16][384]
  const float *A[3], *a[3];                    // per-object MLP [128][28], [128][128] x 2 (row-major)
  const float *Bw[3], *b[4], *B4;              // pair MLP [128][128] x 3, output row [128], b[3] = its bias
};
size_t packed_floats();
// Whether the point MLP's layers 2 and 3, and the predictor's hidden layers, can be products of halves (host weights).
bool point_halves(const float* flat);
bool pair_halves(const float* flat);
// The halves of the point MLP and of the predictor, from the uploaded weights into the packed buffer.
hipError_t launch_halves(const float* d_raw, float* d_packed, hipStream_t s);
// Host-side transposition of the flat weights into dst (packed_floats() floats).
void pack_transposed(const float* flat, float* dst);
PackedNet packed_view(const float* d_raw, const float* d_packed);

struct EncoderBuffers {
  int32_t* order; // [n_points]: per shape, its point indices sorted by grid cell
  uint8_t* cell;  // [n_points]: the grid cell of each entry of order
  // activations, [position][channel / 8][channel % 2][S][(channel % 8) / 2]
  float* grid;    // 216 positions, 256 channels: cell max of the point features
  float* c[4];    // 64 positions, 128 channels
  float* d[3];    // 64 positions, 128 channels
  float* d4;      // 216 positions, 128 channels
  float* glob;    // [S][256]
};
constexpr int kEncodeShapes = 4096;
size_t encoder_scratch_floats(int n_shapes, int64_t n_points);
EncoderBuffers encoder_carve(float* base, int n_shapes, int64_t n_points);

// Shape encoder over n_shapes <= kEncodeShapes shapes; grid must be zero (the cell max starts at 0).
// fp32: the point MLP's layers 2 and 3 as FP32 products, not as products of halves.
hipError_t launch_encoder(const PackedNet& w, const Shape* shapes, int n_shapes, int max_points, const float* xyz,
                          int64_t n_points, const EncoderBuffers& b, float* emb, double* consts,
                          bool fp32, hipStream_t s);

struct PairArgs {
  const locc_object* objs;
  int32_t n_objs;
  const int32_t* pairs;
  int32_t n_pairs;
  const Shape* shapes;
  int32_t n_shapes;
  const double* consts;   // [S][4]: cell size s_0, s_1, s_2 and the margin eps (float64)
  const float* emb;       // [S][216][16]
  PackedNet w;
  float* out;             // [P][2]
  int32_t* counts;        // [P][2] or null
  float* pooled;          // [P][2][16] or null
  unsigned long long* err;
  int32_t fp32;           // 1: the predictor's layers as FP32 products, not as products of halves
  float* z;               // workspace [P][2][28]: per-object predictor inputs (canonical order)
  int32_t* valid;         // workspace [P]
};
// Workspace bytes of a launch over n_pairs pairs.
size_t pair_workspace_bytes(int n_pairs);
// Carves the workspace at base into a.z / a.valid.
void pair_workspace_carve(void* base, int n_pairs, PairArgs& a);
// Two launches: cell selection and mean embeddings (one wave per pair), then
// the predictor MLPs (32 pairs per workgroup).
hipError_t launch_pairs(const PairArgs& a, hipStream_t s);

}  // namespace vox
}  // namespace locc
