// Crop step: a set-up kernel with one thread per pair validates the pair,
// puts it in canonical order and computes its float64 relative pose, crop box
// and float32 screening constants (geometry.h), so that this work is done
// once per pair instead of once per wave (in small batches the waves do it
// themselves); then one wave per object of every
// pair runs the membership scan (by spatial clusters, clusters.hip, or in
// stored order) and the ordered first-K selection, and
// writes counts, the optional index sets, the per-pair records and the
// encoder input rows (float32 for the FP32 path, bf16 for BF16 / FP8).
#include <type_traits>

#include "geometry.h"

namespace locc {
namespace {

// one thread per pair, 64 per workgroup: a batch of 16384 pairs spreads over
// 256 workgroups, one per compute unit, for this latency-bound float64 work
constexpr int kThreads = 64;
constexpr int kInlinePairs = 2048;
constexpr int kCropWaves = 2;  // object waves per workgroup of the crop kernel (1, 2, 4, 8 measured: 2 fastest)

__device__ __forceinline__ PairSetup pair_setup(const CropArgs& A, int p) {
  PairSetup r{};
  locc_object oa, ob;
  ShapeDesc da, db;
  int a = -1, swapped = 0;
  r.valid = geo_fetch(A.objs, A.n_objs, A.pairs, p, A.lib, a, swapped, oa, ob, da, db);
  if (r.valid) {
    geo_pair(oa, ob, da, db, A.pad, r.g);
    geo_screen_values(r.g, db, r.sc);
    r.a = a;
    r.swapped = swapped;
    r.off_a = da.off;
    r.n_a = da.n;
    r.off_b = db.off;
    r.n_b = db.n;
    r.cl_a = da.off / kClusterPoints + oa.shape;
    r.cl_b = db.off / kClusterPoints + ob.shape;
  }
  return r;
}

__global__ __launch_bounds__(kThreads) void pair_setup_kernel(CropArgs A) {
  const int p = blockIdx.x * kThreads + threadIdx.x;
  if (p >= pair_count(A.n_pairs, A.n_pairs_dev, A.dev_base)) return;
  *reinterpret_cast<PairSetup*>(static_cast<char*>(A.setup) + (size_t)p * kPairSetupBytes) = pair_setup(A, p);
}

// One wave per object of a pair: wave item = 2p + side scans, selects and
// gathers object `side` of pair p on its own (no barrier; the two objects of
// a pair never wait for each other), so many more pairs are in flight per
// compute unit than with a workgroup per pair.  W independent waves share a
// workgroup (each with its own LDS), so that the compute unit's limit on
// resident workgroups does not cap the resident waves.
struct ObjectShared {
  int32_t sel[kMaxK];
  uint32_t member[kMaxShapePoints / 32];                // cluster path: a bit per stored point
  uint16_t alive[kMaxShapePoints / kClusterPoints + 1];  // clusters that may hold members
};

// LDS written by some lanes of a wave and then read by others of the same
// wave: the wave's LDS operations are performed in order, so it suffices that
// the compiler keeps them in order and waits for the writes (workgroup-scope
// fences); no other wave takes part.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Raw buffer view of n floats at p: a load at a byte offset >= 4n returns 0
// and reads no memory (the buffer unit's range check), so lanes past a
// shape's last point need no branch of their own.  Word 3 is the gfx9
// raw-buffer format word (32-bit data, no swizzle, no index stride).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t crop_view(const float* p, int n) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), (short)0, n * 4, 0x00020000);
}
__device__ __forceinline__ float crop_load(__amdgpu_buffer_rsrc_t v, int byte_offset) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(v, byte_offset, 0, 0));
}
__device__ __forceinline__ float4 crop_load4(__amdgpu_buffer_rsrc_t v, int byte_offset) {
  return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(v, byte_offset, 0, 0));
}
// A wave-uniform float copied once into a vector register, so that an fma
// taking it with a scalar coefficient needs no copy per use (one scalar
// operand per vector instruction).
__device__ __forceinline__ float crop_to_vgpr(float s) {
  float v;
  asm("v_mov_b32 %0, %1" : "=v"(v) : "s"(s));
  return v;
}

// Membership scan of one object (B: the transformed object b) by one wave,
// over blocks of 256 stored points: lane l holds points 4l .. 4l + 3 of a
// block, fetched by one 16-byte load per coordinate (a quarter of the
// address-unit work of one load per point), QU blocks' loads in flight
// together.  The wave tests the blocks in stored order and keeps the number of
// members before each block (a scalar), so a member's ordered position is that
// number, plus the members of the lanes below it (one ballot per point slot),
// plus its own members before it: the first K members are placed during the
// scan.  Without `full` the scan stops at the first block after which K
// members are known.  Returns the members found (all of them when full, else
// at least min(K, members)).
template <int QU, bool B>
__device__ __forceinline__ int crop_scan(const PairSetup* __restrict__ rec, const PairScreen& sc, const float* px,
                                         const float* py, const float* pz, int n, int K, bool full, int lane,
                                         ObjectShared& S) {
  const int nblk = (n + 255) >> 8;
  int scanned = 0, found = 0;  // wave-uniform
  while (scanned < nblk && (full || found < K)) {
    const int base = scanned << 8;
    const int rem = n - base;  // > 0 points from base on
    const __amdgpu_buffer_rsrc_t vx = crop_view(px + base, rem), vy = crop_view(py + base, rem),
                                 vz = crop_view(pz + base, rem);
    float4 X[QU], Y[QU], Z[QU];
#pragma unroll
    for (int u = 0; u < QU; ++u) {
      const int o = (256 * u + 4 * lane) * 4;
      X[u] = crop_load4(vx, o);
      Y[u] = crop_load4(vy, o);
      Z[u] = crop_load4(vz, o);
    }
#pragma unroll
    for (int u = 0; u < QU; ++u) {
      if (scanned + u < nblk && (full || found < K)) {  // uniform
        const int j0 = 256 * u + 4 * lane;  // this lane's first point: base + j0
        const int left = rem - j0;          // of its four points, those below n
        float x[4] = {X[u].x, X[u].y, X[u].z, X[u].w};
        float y[4] = {Y[u].x, Y[u].y, Y[u].z, Y[u].w};
        float z[4] = {Z[u].x, Z[u].y, Z[u].z, Z[u].w};
        if (left > 0 && left < 4) {  // the shape's last, partial four: point by point
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            x[k] = crop_load(vx, (j0 + k) * 4);
            y[k] = crop_load(vy, (j0 + k) * 4);
            z[k] = crop_load(vz, (j0 + k) * 4);
          }
        }
        bool in[4];
        unsigned long long m[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          in[k] = (B ? geo_member_b(&rec->g, sc, x[k], y[k], z[k]) : geo_member_a(sc, x[k], y[k], z[k])) & (k < left);
          m[k] = __ballot(in[k]);
        }
        unsigned pos = (unsigned)found;
#pragma unroll
        for (int k = 0; k < 4; ++k)
          pos = __builtin_amdgcn_mbcnt_hi((unsigned)(m[k] >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m[k], pos));
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (in[k] && (int)pos < K) S.sel[pos] = base + j0 + k;
          pos += in[k] ? 1u : 0u;
        }
        found += __popcll(m[0]) + __popcll(m[1]) + __popcll(m[2]) + __popcll(m[3]);
      }
    }
    scanned = scanned + QU < nblk ? scanned + QU : nblk;
  }
  return found;
}

// The power of two that takes magnitudes up to top (at least 1) to at most 1; 0 for NaN and past 2^100.
__device__ __forceinline__ float row_power(float top) {
  const unsigned e = (__float_as_uint(top) + 0x007fffffu) >> 23;  // 127 + ceil(log2 top)
  return top <= 0x1p100f ? __uint_as_float((254u - e) << 23) : 0.f;
}

// The clusters of an object that may hold members, listed in S.alive; returns their number.  An a point lies in the box
// iff its coordinates lie between the float bounds, so a cluster whose box ends before a bound holds none.  A b cluster
// is tested in the screen's normalised coordinates: its box maps to an interval u = R' c + t' +- |R'| e (c, e: centre
// and half-widths of the box), and members have |u| <= 1 up to the error that M bounds (geometry.h): with
// 2^-21 S' for the map itself, the sums here add less than 2^-21 S', and M is at least 2^-19 S'.  A NaN anywhere keeps
// the cluster.
template <bool B>
__device__ __forceinline__ int crop_alive(const PairScreen& sc, const float4* __restrict__ boxes, int nc, int lane,
                                          ObjectShared& S) {
  int alive = 0;  // wave-uniform
  for (int c0 = 0; c0 < nc; c0 += 64) {
    const int c = c0 + lane;
    bool keep = false;
    if (c < nc) {
      const float4 lo = boxes[2 * c], hi = boxes[2 * c + 1];
      if constexpr (B) {
        const float cx = 0.5f * (lo.x + hi.x), cy = 0.5f * (lo.y + hi.y), cz = 0.5f * (lo.z + hi.z);
        const float ex = fmaxf(hi.x - cx, cx - lo.x), ey = fmaxf(hi.y - cy, cy - lo.y), ez = fmaxf(hi.z - cz, cz - lo.z);
        bool out = false;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          const float* R = sc.R + 3 * i;
          const float u = __builtin_fmaf(R[2], cz, __builtin_fmaf(R[1], cy, __builtin_fmaf(R[0], cx, sc.t[i])));
          const float r = __builtin_fmaf(fabsf(R[2]), ez, __builtin_fmaf(fabsf(R[1]), ey, fabsf(R[0]) * ex));
          out |= fabsf(u) - r > sc.thr_out;
        }
        keep = !out;
      } else {
        keep = !((lo.x > sc.ahi[0]) | (hi.x < sc.alo[0]) | (lo.y > sc.ahi[1]) | (hi.y < sc.alo[1]) |
                 (lo.z > sc.ahi[2]) | (hi.z < sc.alo[2]) | (sc.alo[0] > sc.ahi[0]) | (sc.alo[1] > sc.ahi[1]) |
                 (sc.alo[2] > sc.ahi[2]));
      }
    }
    const unsigned long long m = __ballot(keep);
    if (keep)
      S.alive[__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, (unsigned)alive))] =
          (uint16_t)c;
    alive += __popcll(m);
  }
  return alive;
}

// Members of one object from its alive clusters: 16 lanes a cluster, four points a lane; a member sets its stored
// index' bit in LDS, and the first K bits in order are the selection.  Returns all members found.
template <bool B>
__device__ __forceinline__ int crop_clusters(const PairSetup* __restrict__ rec, const PairScreen& sc,
                                             const char* __restrict__ clusters, int alive, int n, int K, int lane,
                                             ObjectShared& S) {
  const int words = (n + 31) >> 5;
  for (int w = lane; w < words; w += 64) S.member[w] = 0u;
  wave_lds_sync();  // the list of clusters and the cleared bits
  int found = 0;
  for (int i0 = 0; i0 < alive; i0 += 4) {
    const int i = i0 + (lane >> 4);
    const char* c = clusters + (size_t)S.alive[i < alive ? i : i0] * kClusterBytes;
    const float4 X = reinterpret_cast<const float4*>(c)[lane & 15];
    const float4 Y = reinterpret_cast<const float4*>(c + 256)[lane & 15];
    const float4 Z = reinterpret_cast<const float4*>(c + 512)[lane & 15];
    const uint2 I = reinterpret_cast<const uint2*>(c + 768)[lane & 15];
    const float x[4] = {X.x, X.y, X.z, X.w}, y[4] = {Y.x, Y.y, Y.z, Y.w}, z[4] = {Z.x, Z.y, Z.z, Z.w};
    const unsigned id[4] = {I.x & 0xffffu, I.x >> 16, I.y & 0xffffu, I.y >> 16};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const bool in = (B ? geo_member_b(&rec->g, sc, x[k], y[k], z[k]) : geo_member_a(sc, x[k], y[k], z[k])) &
                      (i < alive) & (id[k] != kNoPoint);
      if (in) atomicOr(&S.member[id[k] >> 5], 1u << (id[k] & 31u));
      found += __popcll(__ballot(in));
    }
  }
  wave_lds_sync();
  int before = 0;  // members of the words before
  for (int w0 = 0; w0 < words && before < K; w0 += 64) {
    unsigned word = w0 + lane < words ? S.member[w0 + lane] : 0u;
    const int upto = geo_wave_inclusive_scan(__popc(word), lane);
    int pos = before + upto - __popc(word);
    while (word && pos < K) {
      S.sel[pos++] = 32 * (w0 + lane) + __builtin_ctz(word);
      word &= word - 1;
    }
    before += __builtin_amdgcn_readlane(upto, 63);
  }
  return found;
}

// Whether the alive clusters are scanned rather than the stored points in order, which ends once K members are known:
// at about K n / (32 alive) points, as an alive cluster holds half its points on average.  The clusters cost their own
// points, and the selection from the bits about as much as 256.  (Half or twice the 32 cost the same to 0.5%; always
// the clusters: 16,384 pairs of 2,048 points 267.5 us instead of 253.5.)
__device__ __forceinline__ bool crop_by_clusters(int alive, int n, int K, bool full) {
  const float scan = full ? (float)n : fminf((float)n, (float)K * (float)n / (float)(32 * alive));
  return (float)(64 * alive + 256) <= scan;
}

// Bound by latency (a wave's chain of dependent loads: record, cluster boxes, points, rows) and, with the chip full,
// by vector issue (half of it used); 80 registers keep six waves per SIMD (84 and five: 1,987 us instead of 1,941 for
// a step of 210,040 pairs).  The clusters skip most points: half of that step's objects have no member and tested
// 2,048 points each, now mostly none (crop 616 us before, 330 with them).
//
// INLINE: the pair's set-up is done here, by both of its waves, instead of by a kernel of its own.
// ROWS: the selected points are gathered from the library's rows.
template <int U, int W, bool INLINE, bool ROWS>
__global__ __launch_bounds__(64 * W, INLINE ? 4 : 6) void crop_kernel(CropArgs A) {
  __shared__ ObjectShared SW[W];
  __shared__ PairSetup RW[INLINE ? W : 1];
  const int wave = W == 1 ? 0 : wave_index();
  ObjectShared& S = SW[wave];
  const int item = blockIdx.x * W + wave;
  const int p = item >> 1;
  const int side = item & 1;
  const int lane = threadIdx.x & 63;
  const int K = A.K;
  if (p >= pair_count(A.n_pairs, A.n_pairs_dev, A.dev_base)) return;  // uniform

  // the pair's record: the same address for the whole wave (scalar loads)
  const PairSetup* __restrict__ rec =
      reinterpret_cast<const PairSetup*>(static_cast<const char*>(A.setup) + (size_t)p * kPairSetupBytes);
  if constexpr (INLINE) {
    const PairSetup r = pair_setup(A, p);
    if (lane == 0) RW[wave] = r;
    wave_lds_sync();
    rec = &RW[wave];
  }
  auto uniform = [](int v) -> int { return INLINE ? __builtin_amdgcn_readfirstlane(v) : v; };
  if (!uniform(rec->valid)) {  // uniform; object 0's wave reports the pair
    if (side == 0) {
      if (A.idx_out)
        for (int e = lane; e < 2 * K; e += 64) A.idx_out[(size_t)p * 2 * K + e] = -1;
      if (lane == 0) {
        if (A.counts_out) {
          A.counts_out[2 * p] = -1;
          A.counts_out[2 * p + 1] = -1;
        }
        if (A.meta) A.meta[p] = PairMeta{-1, 0, 0, 0};
        atomicAdd(A.err_counter, 1ull);
      }
    }
    return;
  }
  const int swapped = uniform(rec->swapped);
  const int n = uniform(side ? rec->n_b : rec->n_a);
  const int off = uniform(side ? rec->off_b : rec->off_a);
  PairScreen sc = rec->sc;
  if constexpr (INLINE) {  // wave-uniform: scalar registers
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      sc.alo[i] = geo_uniform(sc.alo[i]);
      sc.ahi[i] = geo_uniform(sc.ahi[i]);
      sc.t[i] = geo_uniform(sc.t[i]);
    }
#pragma unroll
    for (int k = 0; k < 9; ++k) sc.R[k] = geo_uniform(sc.R[k]);
    sc.thr_in = geo_uniform(sc.thr_in);
    sc.thr_out = geo_uniform(sc.thr_out);
  }
  const bool full = A.counts_out != nullptr;  // else stop once K members are known
  const float* __restrict__ px = A.lib.coordinate(0) + off;
  const float* __restrict__ py = A.lib.coordinate(1) + off;
  const float* __restrict__ pz = A.lib.coordinate(2) + off;
  const int cl = uniform(side ? rec->cl_b : rec->cl_a), nc = (n + kClusterPoints - 1) / kClusterPoints;
  const float4* boxes = A.lib.boxes && n > A.cluster_min ? A.lib.boxes + 2 * (size_t)cl : nullptr;
  const char* clusters = A.lib.clusters + (size_t)cl * kClusterBytes;
  int found, alive = 0;
  if (side) {
#pragma unroll
    for (int i = 0; i < 3; ++i) sc.t[i] = crop_to_vgpr(sc.t[i]);
    if (boxes) alive = crop_alive<true>(sc, boxes, nc, lane, S);
    if (boxes && crop_by_clusters(alive, n, K, full))
      found = crop_clusters<true>(rec, sc, clusters, alive, n, K, lane, S);
    else
      found = crop_scan<(U >= 8 ? 2 : 1), true>(rec, sc, px, py, pz, n, K, full, lane, S);
  } else {
    if (boxes) alive = crop_alive<false>(sc, boxes, nc, lane, S);
    if (boxes && crop_by_clusters(alive, n, K, full))
      found = crop_clusters<false>(rec, sc, clusters, alive, n, K, lane, S);
    else
      found = crop_scan<(U >= 8 ? 2 : 1), false>(rec, sc, px, py, pz, n, K, full, lane, S);
  }
  // found: every member when full, else at least min(K, members)
  wave_lds_sync();  // the selected indices are read by other lanes
  const int m = found < K ? found : K;
  const int caller = side ^ swapped;  // position of this object in the caller's pair
  if (lane == 0) {
    if (A.counts_out) A.counts_out[2 * p + caller] = found;
    if (A.meta) {
      if (side == 0) {
        A.meta[p].a = rec->a;
        A.meta[p].swapped = swapped;
        A.meta[p].m_a = m;
      } else {
        A.meta[p].m_b = m;
      }
    }
  }
  if (A.idx_out)
    for (int r = lane; r < K; r += 64) A.idx_out[((size_t)p * 2 + caller) * K + r] = r < m ? S.sel[r] : -1;
  if (A.rows) {
    // rows (x, y, z, nx, ny, nz, 1, 0) stored permuted as (e0, e2, e4, e6, e1, e3, e5, e7);
    // zero rows past the valid count; e7 is the object's power of two
    const PairGeom g = rec->g;
    float top = 0.f, top_n = 1.f;  // the largest coordinate and normal component in this lane's rows
    for (int r = lane; r < K; r += 64) {
      float4 lo4 = make_float4(0.f, 0.f, 0.f, 0.f), hi4 = lo4;
      if (r < m) {
        float v[6];
        geo_row<ROWS>(g, A.lib, off + S.sel[r], side, v);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          top = __builtin_elementwise_maximum(top, fabsf(v[k]));
          top_n = __builtin_elementwise_maximum(top_n, fabsf(v[3 + k]));
        }
        lo4 = make_float4(v[0], v[2], v[4], 1.0f);
        hi4 = make_float4(v[1], v[3], v[5], 1.0f);
      }
      float4* dst = reinterpret_cast<float4*>(A.rows + ((size_t)p * 2 * K + side * K + r) * kRowFloats);
      dst[0] = lo4;
      dst[1] = hi4;
    }
    top = __builtin_elementwise_maximum(top * A.lib.per_unit, top_n);
    if (__ballot(!(top <= 1.f)) != 0) {  // a coordinate past the unit, or a normal longer than 1
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) top = __builtin_elementwise_maximum(top, __shfl_xor(top, d, 64));
      const float power = row_power(top);
      for (int r = lane; r < m; r += 64)  // (each lane's own rows: behind its stores above)
        A.rows[((size_t)p * 2 * K + side * K + r) * kRowFloats + kRowFloats - 1] = power;
    }
  }
  if (A.rows_bf16) {
    // bf16 rows (x, y, z, nx, ny, nz, 1, 0), zero-padded to a multiple of 32
    const PairGeom g = rec->g;
    const int rm = (m + 31) & ~31;
    for (int r = lane; r < rm; r += 64) {
      unsigned short row[8] = {0, 0, 0, 0, 0, 0, 0, 0};
      if (r < m) {
        float v[6];
        geo_row<ROWS>(g, A.lib, off + S.sel[r], side, v);
#pragma unroll
        for (int k = 0; k < 6; ++k) row[k] = __builtin_bit_cast(unsigned short, (__bf16)v[k]);
        row[6] = 0x3f80;  // 1.0
      }
      uint4 packed;
      packed.x = row[0] | ((unsigned)row[1] << 16);
      packed.y = row[2] | ((unsigned)row[3] << 16);
      packed.z = row[4] | ((unsigned)row[5] << 16);
      packed.w = row[6] | ((unsigned)row[7] << 16);
      *reinterpret_cast<uint4*>(A.rows_bf16 + ((size_t)p * 2 * K + side * K + r) * 8) = packed;
    }
  }
}

}  // namespace

hipError_t launch_crop(const CropArgs& args, hipStream_t s, int unroll) {
  CropArgs a = args;
  if (a.n_pairs <= 0) return hipSuccess;
  // A few blocks of stored points take a lone wave no longer than the cluster boxes and the selection, and more of them
  // where it needs every member and may load ahead (80 pairs with counts: of 1,024 points 26.7 us in stored order, 27.5 by
  // clusters; of 2,048 28.7 and 30.1; of 3,072 30.7 and 32.1; 2,000 pairs: 46.1 and 47.2, 49.6 and 53.0, 54.9 and 55.8; of
  // 4,096 59.5 and 58.5) than where it stops at K (80 pairs: 26.6 and 26.9, 28.3 and 28.5, 30.5 and 27.1).  With the chip
  // full the points skipped count (a step of 210,040 pairs of 1,024 points: 1,847 and 1,782 us; of 512 points: 1,831
  // and 1,850).
  a.cluster_min = a.n_pairs >= 4096 ? 512 : (a.counts_out && a.n_pairs <= kInlinePairs ? 3072 : 1024);
  if (!a.setup || (unroll != 2 && unroll != 4 && unroll != 8)) return hipErrorInvalidValue;
  constexpr int W = kCropWaves;
  const dim3 grid((2 * a.n_pairs + W - 1) / W), block(64 * W);
  // A small batch saves the set-up kernel's launch (8 pairs: 29.7 us with it, 27.7 without; 1,500: 52.1, 50.0; 2,000: 58.5,
  // 57.3); in a larger one the float64 set-up of every wave costs more (3,000: 79.3, 80.5; 16,384: 249.7, 261.7).
  const bool inline_setup = a.n_pairs <= kInlinePairs;
  if (!inline_setup)
    kernel_launch(pair_setup_kernel, dim3((a.n_pairs + kThreads - 1) / kThreads), dim3(kThreads), 0, s, a);
  // Without the rows 22 pairs take 18.8 us and not 18.6, 400 pairs 31.9 and 31.7.
  auto run = [&](auto u) {
    constexpr int U = decltype(u)::value;
    if (inline_setup && a.lib.rows)
      kernel_launch((crop_kernel<U, W, true, true>), grid, block, 0, s, a);
    else if (inline_setup)
      kernel_launch((crop_kernel<U, W, true, false>), grid, block, 0, s, a);
    else if (a.lib.rows)
      kernel_launch((crop_kernel<U, W, false, true>), grid, block, 0, s, a);
    else
      kernel_launch((crop_kernel<U, W, false, false>), grid, block, 0, s, a);
  };
  if (unroll == 2)
    run(std::integral_constant<int, 2>{});
  else if (unroll == 4)
    run(std::integral_constant<int, 4>{});
  else
    run(std::integral_constant<int, 8>{});
  return hipGetLastError();
}

}  // namespace locc
