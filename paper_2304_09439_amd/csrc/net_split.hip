// FP32 per-point encoder with per-object max-pool, and the FP32 head, on the
// half-precision matrix cores.
//
//   h1 = ReLU(W1 r + b1), h2 = ReLU(W2 h1 + b2), f = max over the valid rows
// of each object (0 when none; Sec. III, appendix).  Layer 1 runs on the FP32
// matrix cores.  Layer 2, 97% of the work, runs on 16-bit ones: a float x is
// the sum of two halves, x0 = half(x) and x1 = half(x - x0), to 2^-23 of x
// (three floats in four exactly), and of the four products of two such sums all
// but x1 y1 (at most 2^-22 of the product) are accumulated in FP32.  x0 y0 has a
// sum of its own, so that the large partial sums round 8 times per output where a
// chain of FP32 multiply-adds rounds 128 times; the result is as near the 64-bit
// one as that chain's.  Three 32x32x16 products take 96 cycles for the 1024 that
// 16 reduction steps of 32x32x2 FP32 products take.  16,384 pairs of 2048-point
// shapes at K = 128, widths 128 / 256: 0.57 ms, 1.77 ms on the FP32 matrix cores
// (error of the whole path against 64 bits 5.8e-7, 7.9e-7 before).  The
// matrix cores are busy 0.59 of its cycles and draw enough power that the
// clock falls to about 1.9 GHz.  Six products of three bf16 parts (no scales
// needed) took 0.98 ms.
//
// Two halves keep all their bits from 2^-2 to 2^16, so everything is multiplied
// by powers of two, and the pooled sums divided by them (all exact): an object's
// rows by the one, at most 1, that takes them into [-1, 1] (the crop finds it; the
// coordinates in a unit of about most shapes' size, so that it is mostly 1);
// a hidden unit's weights and bias by one that then keeps its outputs below 2^15,
// the weights that read it by the inverse; W2's rows by one that puts their
// largest weight at 2^14 to 2^15.  So neither a wide margin, a large shape elsewhere
// in the library, a unit far from the others nor training costs bits.  What falls
// below 2^-2 all the same (by chance 2e-5 of the outputs) matters only where it is
// not beside larger ones: a step with a row that has too many such outputs in a tile
// of 32 units (halves_short), an object whose rows have no power of two, and every
// step when a row of W2 has too many or a weight is not finite, is computed as an
// FP32 chain.
//
// A persistent workgroup of h2 / 32 waves takes chunks of pairs from a queue
// (chunk sizes fall from 32 to 1 towards the end of the batch, so that the
// last chunks even out the unequal row counts) and walks their objects in
// steps of 64 rows.  Wave w owns 32 of layer 2's columns, its W2 fragments of
// both parts in registers; layer 1 of the next step is computed one 32 x 32
// tile per wave, split, and written to the other of two LDS buffers while
// layer 2 of the current step runs (one barrier per step).
#include "halves.h"
#include "locc_internal.h"
#include "post.h"

namespace locc {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float vmax(float a, float b) { return __builtin_elementwise_maximum(a, b); }
__device__ __forceinline__ f32x16 mfma32x32x2(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 mfma_k16(u32x4 a, u32x4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0,
                                                0);
}
__device__ __forceinline__ int perm_feature(int ft, int g, int r) { return 32 * ft + 8 * (r / 4) + 4 * g + r % 4; }

constexpr int kStepRows = 64;
constexpr int kMaxSteps = kSplitChunk * 2 * (kMaxK / kStepRows);
static_assert(kSplitChunk == 32, "one lane per object of a chunk");

template <int H1, int H2>
struct SplitSmem {
  static constexpr int HS = H1 + 8;  // halves per row: 16 bytes past a multiple of 64 or 128, for the banks
  alignas(16) unsigned short h[2][2][kStepRows * HS];  // layer-1 outputs of a step: [buffer][part][row][permuted feature]
  int32_t step[kMaxSteps];       // object of the chunk (0-63) | row block << 8
  int32_t m[2 * kSplitChunk];    // rows per object; -1: invalid pair
  int32_t n_steps;
  int32_t claim;
  int32_t bad[2];                // per buffer: the step whose layer-1 outputs are short of bits
};

// ARGMAX: also the row of each channel's largest sum (the first on ties), and which channels' choice is in doubt: where
// the second largest sum lies within 2^-24 of the largest magnitude a sum of the object's rows can have and the feature
// is not surely 0.  That margin is about ten times the usual rounding error of an FP32 chain here (whose terms are a
// tenth of their bounds and of both signs), not a bound of it (which is over a hundred times as large): a chain that
// rounds worse than that may have its maximum in another row.  0.3% of the channels of 16,384 pairs.
template <int H1, int H2, bool ARGMAX>
__global__ __launch_bounds__(2 * H2, 2) void encoder_split_kernel(Fp32Net W, NetArgs A, SplitChunks C) {
  using S_t = SplitSmem<H1, H2>;
  constexpr int HS = S_t::HS;
  constexpr int FT = H1 / 32;        // layer-1 feature tiles
  constexpr int NW = H2 / 32;        // waves, one layer-2 column tile each
  constexpr int KS = H1 / 16;        // layer-2 k-steps
  static_assert(2 * FT == NW, "one layer-1 tile of a step per wave");
  __shared__ S_t S;
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ft1 = wave % FT, rt1 = wave / FT;  // this wave's layer-1 tile of a step
  const int K = A.K;
  const int P = pair_count(A.n_pairs, A.n_pairs_dev);
  const bool slow = *W.split_bad != 0;

  u32x4 w2f[2][KS];
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int s = 0; s < KS; ++s)
      w2f[q][s] = reinterpret_cast<const u32x4*>(W.w2s)[((size_t)(q * NW + wave) * KS + s) * 64 + lane];
  float w1f[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) w1f[s] = W.w1s[(ft1 * 4 + s) * 64 + lane];
  const float bias2 = W.b2[wave * 32 + l32], unscale2 = W.unscale2[wave * 32 + l32];
  if (tid < 2) S.bad[tid] = -1;
  float doubt = 0.f;  // ARGMAX: 2^-24 times this column's absolute weights times 2^15, unscaled
  if constexpr (ARGMAX) {
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const f16x8 w = __builtin_bit_cast(f16x8, w2f[0][s]);
#pragma unroll
      for (int e = 0; e < 8; ++e) doubt += __builtin_fabsf((float)w[e]);
    }
    doubt = (doubt + __shfl_xor(doubt, 32, 64)) * unscale2 * 0x1p-9f;
  }

  int gstep = 0;  // steps this workgroup has started (tags S.bad)
  // The first claim is the workgroup's index; the queue has those past the grid's, so that a batch of one claim a
  // workgroup does without its atomics: hundreds at once on one address (500 pairs of 64 + 64 points at 64 / 128 with
  // counts 49.0 -> 36.2 us, 80 pairs 29.6 -> 26.9).  A caller without a queue (the no-allocation detect) has the
  // claims in static order.
  int claim = blockIdx.x, queued_base, queued_n;
  split_chunk(C, gridDim.x, queued_base, queued_n);
  const bool queued = A.queue && queued_base < P;
  for (int iter = 0;; ++iter) {
    if (iter > 0) {
      if (A.queue) {
        if (!queued) break;
        if (tid == 0) S.claim = (int)(gridDim.x + atomicAdd(A.queue, 1u));
        __syncthreads();
        claim = S.claim;
      } else {
        claim += gridDim.x;
      }
    }
    int base, n;
    split_chunk(C, claim, base, n);
    if (base >= P) break;  // uniform
    if (base + n > P) n = P - base;
    // the chunk's steps: a lane per object, prefix of the step counts
    if (wave == 0) {
      int m = 0;
      if (lane < 2 * n) {
        const PairMeta mt = A.meta[base + (lane >> 1)];
        m = mt.a < 0 ? -1 : (lane & 1 ? mt.m_b : mt.m_a);
      }
      S.m[lane] = m;
      const int ns = m > 0 ? (m + kStepRows - 1) / kStepRows : 0;
      int at = ns;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int o = __shfl_up(at, d, 64);
        if (lane >= d) at += o;
      }
      if (lane == 63) S.n_steps = at;
      at -= ns;
      for (int b = 0; b < ns; ++b) S.step[at + b] = lane | (b << 8);
    }
    __syncthreads();
    const int ns = S.n_steps;
    // objects without rows: f = 0; both objects of an invalid pair: NaN
    for (int o = wave; o < 2 * n; o += NW) {
      const int m = S.m[o];  // uniform
      if (m > 0) continue;
      if constexpr (ARGMAX) {
        if (lane < H2 / 4) reinterpret_cast<int32_t*>(A.amax + ((size_t)base * 2 + o) * H2)[lane] = -1;  // 255
        if (lane < NW) A.doubt[((size_t)base * 2 + o) * NW + lane] = 0;
      }
      const float v = m < 0 ? __builtin_nanf("") : 0.f;
      if (lane < H2 / 4 && A.z)
        reinterpret_cast<float4*>(A.z + ((size_t)base * 2 + o) * H2)[lane] = make_float4(v, v, v, v);
    }

    // a step's layer-1 input in this lane (rows past the object's count are zeros), and how many rows of the wave's row
    // tile the object has; a wave whose tile it does not reach has the step's first tile again, whose outputs are not read
    struct Input {
      float4 x;
      int live;
    };
    auto load_rows = [&](int k) __attribute__((always_inline)) -> Input {
      const int e = __builtin_amdgcn_readfirstlane(S.step[k]);
      const int o = e & 0xff, r0 = (e >> 8) * kStepRows + 32 * rt1;
      const int live = __builtin_amdgcn_readfirstlane(S.m[o]) - r0;
      const size_t row = ((size_t)base * 2 + o) * K + (live > 0 ? r0 : r0 - 32 * rt1) + l32;
      return Input{*reinterpret_cast<const float4*>(A.rows + row * kRowFloats + 4 * g), live};
    };
    f32x16 acc1 = f32x16{};
    // issues layer 1 and returns the rows' power of two, which comes with the tile's first row
    auto layer1_issue = [&](const float4& x) __attribute__((always_inline)) -> float {
      const float up = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x.w), 32));
      acc1 = mfma32x32x2(w1f[0], x.x * up, f32x16{});
      acc1 = mfma32x32x2(w1f[1], x.y * up, acc1);
      acc1 = mfma32x32x2(w1f[2], x.z * up, acc1);
      acc1 = mfma32x32x2(w1f[3], x.w * up, acc1);
      return up;
    };
    // One of the eight pairs of layer-1 outputs of this lane to their parts (h = pair / 4, e = pair % 4); the
    // fourth of a half writes the half's 16 bytes of each part.
    u32x4 q0, q1;
    unsigned least = ~0u;  // bits of the smallest output that is not negative (of a live row: 0 is rare)
    auto layer1_pair = [&](int pair, int buf) __attribute__((always_inline)) {
      const int hf = pair >> 2, e = pair & 3;
      float a = vmax(acc1[2 * pair], 0.f), b = vmax(acc1[2 * pair + 1], 0.f);
      least = min(least, min(__float_as_uint(acc1[2 * pair]), __float_as_uint(acc1[2 * pair + 1])));
      q0[e] = split_part(a, b);
      q1[e] = last_part(a, b);
      if (e == 3) {
        unsigned short* dst = &S.h[buf][0][(32 * rt1 + l32) * HS + 32 * ft1 + 8 * g + 16 * hf];
        *reinterpret_cast<u32x4*>(dst) = q0;
        *reinterpret_cast<u32x4*>(dst + kStepRows * HS) = q1;
      }
    };
    // Whether a row of the step has too many outputs short of bits in this wave's 32 units (both lanes of a row).
    auto layer1_check = [&](int buf, int tag, int live) __attribute__((always_inline)) {
      if (__ballot((least < __float_as_uint(kHalvesLeast)) & (l32 < live)) != 0) {  // a step in five, in one of its waves
        int some = 0, lost = 0;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          some += acc1[r] > 0.f;
          lost += acc1[r] > 0.f && acc1[r] < kHalvesLeast;
        }
        int count = some << 16 | lost;
        count += __shfl_xor(count, 32, 64);
        if (__ballot(halves_short(count, kShortActivations) & (l32 < live)) != 0 && lane == 0) S.bad[buf] = tag;
      }
      least = ~0u;
    };

    float up = 1.f;  // of the current step
    if (ns > 0) {
      const Input in = load_rows(0);
      up = layer1_issue(in.x);
#pragma unroll
      for (int q = 0; q < 8; ++q) layer1_pair(q, 0);
      layer1_check(0, gstep, in.live);
    }
    Input next{make_float4(0.f, 0.f, 0.f, 0.f), 0};
    if (ns > 1) next = load_rows(1);
    __syncthreads();
    float run = -__builtin_inff(), run2 = -__builtin_inff();  // the largest and (ARGMAX) second largest sum so far
    int arg = 255, chains = 0;                                // its row; bit 0: a step of halves, bit 1: a chain
    for (int k = 0; k < ns; ++k, ++gstep) {
      const int e = __builtin_amdgcn_readfirstlane(S.step[k]);
      const int o = e & 0xff, r0 = (e >> 8) * kStepRows;
      const int m = __builtin_amdgcn_readfirstlane(S.m[o]);
      const bool more = k + 1 < ns;
      const int buf = k & 1;
      const bool chain = slow || up == 0.f || __builtin_amdgcn_readfirstlane(S.bad[buf]) == gstep;
      const int live = next.live;
      float next_up = 1.f;
      if (more) next_up = layer1_issue(next.x);
      if (k + 2 < ns) next = load_rows(k + 2);
      // max of a row tile's raw sums (bias and ReLU once per column afterwards: rounding is monotone)
      float best = -__builtin_inff(), best2 = -__builtin_inff();
      int at = 255 - 4 * g;
      auto keep = [&](float v, int row0, int r) __attribute__((always_inline)) {
        // a lane's rows ascend: strict > keeps the first maximum; best2 <= best, so the median of three is the second
        const bool more_than = v > best;
        best2 = __builtin_amdgcn_fmed3f(v, best, best2);
        at = more_than ? row0 + 8 * (r >> 2) + (r & 3) : at;
        best = more_than ? v : best;
      };
      auto pool = [&](const f32x16& v, int row0) __attribute__((always_inline)) {
        if constexpr (ARGMAX) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int row = row0 + 8 * (r >> 2) + 4 * g + (r & 3);
            keep(row < m ? v[r] : -__builtin_inff(), row0, r);
          }
        } else if (row0 + 32 <= m) {
#pragma unroll
          for (int r = 0; r < 16; r += 2) best = vmax(vmax(best, v[r]), v[r + 1]);
        } else {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int row = row0 + 8 * (r >> 2) + 4 * g + (r & 3);
            if (row < m) best = vmax(best, v[r]);
          }
        }
      };
      // the products of row tile rt; between(s) is issued among those of k-step s
      f32x16 hi, lo;
      auto layer2 = [&](int rt, auto between) __attribute__((always_inline)) {
        const unsigned short* src = &S.h[buf][0][(32 * rt + l32) * HS + 8 * g];
        auto part = [&](int q, int s) __attribute__((always_inline)) {
          return *reinterpret_cast<const u32x4*>(src + q * kStepRows * HS + 16 * s);
        };
        hi = lo = f32x16{};
        u32x4 a0 = part(0, 0), a1 = part(1, 0);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          u32x4 n0, n1;
          if (s + 1 < KS) {
            n0 = part(0, s + 1);
            n1 = part(1, s + 1);
          }
          lo = mfma_k16(a1, w2f[0][s], lo);
          hi = mfma_k16(a0, w2f[0][s], hi);
          lo = mfma_k16(a0, w2f[1][s], lo);
          between(s);
          if (s + 1 < KS) {
            a0 = n0;
            a1 = n1;
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      if (!chain) {
        // (after the chunk's last step the parts of stale values go to the buffer that nobody reads again)
        layer2(0, [&](int s) __attribute__((always_inline)) {
          if (KS == 8) {
            if (s > 0) layer1_pair(s - 1, buf ^ 1);
            if (s == 7) layer1_pair(7, buf ^ 1);
          } else {
            if (s > 0) {
              layer1_pair(2 * s - 2, buf ^ 1);
              layer1_pair(2 * s - 1, buf ^ 1);
            }
            if (s == 3) {
              layer1_pair(6, buf ^ 1);
              layer1_pair(7, buf ^ 1);
            }
          }
        });
        if (r0 + 32 < m) {
          const f32x16 v = hi + lo;
          layer2(1, [&](int s) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 16 / KS * s; r < 16 / KS * (s + 1); r += 2) {
              if constexpr (ARGMAX) {
                keep(v[r], r0, r);
                keep(v[r + 1], r0, r + 1);
              } else {
                best = vmax(vmax(best, v[r]), v[r + 1]);
              }
            }
          });
          pool(hi + lo, r0 + 32);
        } else {
          pool(hi + lo, r0);
        }
      } else {  // uniform over the workgroup
        for (int rt = 0; rt < 2 && r0 + 32 * rt < m; ++rt) {
          const float4 x = *reinterpret_cast<const float4*>(
              A.rows + (((size_t)base * 2 + o) * K + r0 + 32 * rt + l32) * kRowFloats + 4 * g);
          f32x16 acc2 = f32x16{};
#pragma unroll 1
          for (int ft = 0; ft < FT; ++ft) {
            const float* w1 = W.w1pack + (size_t)ft * 4 * 64 + lane;
            const float* w2 = W.w2pack + ((size_t)wave * (H1 / 2) + 16 * ft) * 64 + lane;
            f32x16 h = mfma32x32x2(w1[0], x.x, f32x16{});
            h = mfma32x32x2(w1[64], x.y, h);
            h = mfma32x32x2(w1[128], x.z, h);
            h = mfma32x32x2(w1[192], x.w, h);
#pragma unroll
            for (int r = 0; r < 16; ++r) acc2 = mfma32x32x2(vmax(h[r], 0.f), w2[r * 64], acc2);
          }
          pool(acc2, r0 + 32 * rt);
        }
      }
      if (more) {
        if (chain)
#pragma unroll
          for (int q = 0; q < 8; ++q) layer1_pair(q, buf ^ 1);
        layer1_check(buf ^ 1, gstep + 1, live);
      }
      least = ~0u;
      const float down = halves_unscale(up);
      up = next_up;
      if (!chain) {
        best = best * unscale2 * down;
        best2 = best2 * unscale2 * down;
      }
      if constexpr (ARGMAX) {
        arg = best > run ? at + 4 * g : arg;
        run2 = vmax(vmax(run2, best2), fminf(run, best));
        chains |= chain ? 2 : 1;
      }
      run = vmax(run, best);
      if (r0 + kStepRows >= m) {  // the object's last step
        const float other = __shfl_xor(run, 32, 64);
        const size_t at0 = ((size_t)base * 2 + o) * H2 + wave * 32;
        if (lane < 32 && A.z) A.z[at0 + lane] = fmaxf(fmaxf(run, other) + bias2, 0.f);
        if constexpr (ARGMAX) {
          // the two half-waves hold rows 4g + ... of every tile: the larger value wins, the lower row on ties
          const int other_arg = __shfl_xor(arg, 32, 64);
          const float other2 = __shfl_xor(run2, 32, 64);
          const bool take = other > run || (other == run && other_arg < arg);
          const float second = vmax(vmax(run2, other2), fminf(run, other));
          const float first = vmax(run, other);
          const float margin = doubt * down;
          const bool sure = chains == 2 || first - second > margin || first + bias2 < -margin;
          if (lane < 32) A.amax[at0 + lane] = (uint8_t)(take ? other_arg : arg);
          const unsigned long long unsure = __ballot(!sure);
          if (lane == 0) A.doubt[((size_t)base * 2 + o) * NW + wave] = (uint32_t)unsure;
          run2 = -__builtin_inff();
          arg = 255;
          chains = 0;
        }
        run = -__builtin_inff();
      }
      __syncthreads();
    }
  }
  if (queued && tid == 0) {
    __threadfence();
    if (atomicAdd(A.queue + 1, 1u) == gridDim.x - 1) {  // last workgroup out resets the queue
      atomicExch(A.queue, 0u);
      atomicExch(A.queue + 1, 0u);
    }
  }
}

// ------------------------------------------------------- features as a chain
//
// The pooled features of the pose gradients and of training, whose ReLU and
// argmax decisions are those of one chain of FP32 multiply-adds per sum (in the
// order of a 32x32x2 matrix product: layer 1 over (x, y, z, nx, ny, nz, 1),
// layer 2 over layer 1's permuted features): from the row the split encoder
// found for each channel, that row's chain gives the feature; a channel whose
// row is in doubt takes the largest chain over all rows, the first on ties, 64
// rows at a time by its wave.  (A row that is not in doubt is taken as found, which
// is the chain's own choice unless that chain rounds worse than the margin of doubt
// allows: it did not on the networks and scenes tried.)  A thread per channel and
// four objects, so that a weight is read once for four; W1 is read by scalar loads.
// Bound by its vector instructions: 9 per channel, hidden unit and object, 0.27 ms
// for 16,384 pairs at 128 / 256, and with the split encoder's 0.70 ms about half of
// the 1.94 ms of the whole encoder on the FP32 matrix cores.

// Four objects a workgroup read W2 once for four; up to 2,048 pairs the chip has room for every object alone, and the
// chain of one is the shorter one (pose gradients of 40 pairs at 64 / 128 81.3 -> 76.1 us, 150 pairs at 128 / 256
// 232.5 -> 223.5; 3,000 pairs go the other way, 411.8 against 418.6).
constexpr int kChainLonePairs = 2048;
constexpr int kChainObjects = 4;

template <int H1>
__device__ __forceinline__ float chain_sum(const float* __restrict__ w1c, const float* __restrict__ w2c, int H2,
                                           const float (&x)[6]) {
  float acc = 0.f;
#pragma unroll 4
  for (int s = 0; s < H1; ++s) {
    const float* w = w1c + 8 * s;
    float h = w[0] * x[0];
#pragma unroll
    for (int c = 1; c < 6; ++c) h = __builtin_fmaf(w[c], x[c], h);
    acc = __builtin_fmaf(vmax(h + w[6], 0.f), w2c[(size_t)s * H2], acc);
  }
  return acc;
}

template <int H1, int H2, int NO>
__global__ __launch_bounds__(H2) void chain_features_kernel(Fp32Net W, NetArgs A) {
  constexpr int NW = H2 / 32;
  const int c = threadIdx.x, lane = c & 63;
  const int wave = __builtin_amdgcn_readfirstlane(c >> 6);
  const int P = pair_count(A.n_pairs, A.n_pairs_dev);
  const int K = A.K;
  const float* __restrict__ w1c = W.w1c;
  const float* __restrict__ w2c = W.w2c + c;
  const size_t o0 = (size_t)blockIdx.x * NO;  // object = 2 pair + side
  int m[NO], row[NO];
  float x[NO][6], acc[NO];
#pragma unroll
  for (int i = 0; i < NO; ++i) {
    m[i] = -2;  // no object
    if (o0 + i < 2 * (size_t)P) {
      const PairMeta mt = A.meta[(o0 + i) >> 1];
      m[i] = mt.a < 0 ? -1 : ((o0 + i) & 1 ? mt.m_b : mt.m_a);
    }
    row[i] = m[i] > 0 ? A.amax[(o0 + i) * H2 + c] : 0;
    if (row[i] >= m[i]) row[i] = 0;  // (no row above -inf: the sum is not used)
#pragma unroll
    for (int q = 0; q < 6; ++q) x[i][q] = 0.f;
    if (m[i] > 0) {
      // stored (x, z, ny, 1 | y, nx, nz, 0)
      const float4* r = reinterpret_cast<const float4*>(A.rows + ((o0 + i) * K + row[i]) * kRowFloats);
      const float4 lo = r[0], hi = r[1];
      x[i][0] = lo.x;
      x[i][1] = hi.x;
      x[i][2] = lo.y;
      x[i][3] = hi.y;
      x[i][4] = lo.z;
      x[i][5] = hi.z;
    }
    acc[i] = 0.f;
  }
#pragma unroll 2
  for (int s = 0; s < H1; ++s) {
    const float* w = w1c + 8 * s;
    const float w2 = w2c[(size_t)s * H2];
#pragma unroll
    for (int i = 0; i < NO; ++i) {
      float h = w[0] * x[i][0];
#pragma unroll
      for (int q = 1; q < 6; ++q) h = __builtin_fmaf(w[q], x[i][q], h);
      acc[i] = __builtin_fmaf(vmax(h + w[6], 0.f), w2, acc[i]);
    }
  }
#pragma unroll
  for (int i = 0; i < NO; ++i) {
    if (m[i] == -2) continue;  // uniform, like every m
    const size_t o = o0 + i;
    float best = acc[i];
    if (m[i] > 0) {
      if (A.amax[o * H2 + c] >= m[i]) best = -__builtin_inff();
      // the wave's 64 channels in doubt, one after the other
      unsigned long long todo = A.doubt[o * NW + 2 * wave] | ((unsigned long long)A.doubt[o * NW + 2 * wave + 1] << 32);
      while (todo) {  // uniform
        const int l = __builtin_ctzll(todo);
        todo &= todo - 1;
        float top = -__builtin_inff();
        int at = 255;
        for (int r0 = 0; r0 < m[i]; r0 += 64) {
          if (r0 + lane < m[i]) {
            const float4* r = reinterpret_cast<const float4*>(A.rows + (o * K + r0 + lane) * kRowFloats);
            const float4 lo = r[0], hi = r[1];
            const float y[6] = {lo.x, hi.x, lo.y, hi.y, lo.z, hi.z};
            const float v = chain_sum<H1>(w1c, W.w2c + 64 * wave + l, H2, y);
            if (v > top) {
              top = v;
              at = r0 + lane;
            }
          }
        }
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
          const float ot = __shfl_xor(top, d, 64);
          const int oa = __shfl_xor(at, d, 64);
          if (ot > top || (ot == top && oa < at)) {
            top = ot;
            at = oa;
          }
        }
        if (lane == l) {
          best = top;
          A.amax[o * H2 + c] = (uint8_t)at;
        }
      }
    } else {
      best = -__builtin_inff();
    }
    A.z[o * H2 + c] = m[i] < 0 ? __builtin_nanf("") : fmaxf(best + W.b2[c], 0.f);
  }
}

// ----------------------------------------------------------------------- head
//
// y = H3 ReLU(H2 ReLU(H1 [f_a, f_b] + c1) + c2) + c3 on RT tiles of 32 pairs
// per workgroup of eight waves, as products of halves like the encoder's layer
// 2.  The activations stay in LDS as halves (one buffer: a layer's outputs
// overwrite its inputs once every wave has read them); each wave owns HH / 8
// columns of layers 1 and 2 and streams their weight halves from L2 two steps
// ahead, each fragment serving all row tiles; layer 3 splits its reduction
// over the waves.  A pair's row is scaled by the power of two that puts its
// largest input at 2^14 to 2^15, in every layer (a bound of it through the layers
// would leave the bits to one unit with a large bias or large weights).  The
// weights are the products' first operand, so that a lane's outputs belong to one
// pair.  16,384 pairs at width 512: 55 us (0.350 ms as FP32 products, 32 pairs and
// four waves per workgroup), 1,000: 30 us; 80 pairs at width 256: 12.4 us (40 us).
// Bound by the 2 MB of weights each workgroup streams from L2 (RT = 1), or by the
// matrix cores (RT = 2).  Left to itself the compiler moves those loads to their
// use (42 us at 1,000 pairs).
// A pair with a value out of range, or with too many inputs of a layer so far below its
// largest that their halves are short of bits, gets the FP32 chain's result instead.

template <int Z, int HH, int RT>
struct HeadSmem {
  static constexpr int T = 32 * RT;
  static constexpr int W = (Z > HH ? Z : HH);
  static constexpr int AS = W + 8;      // halves per row
  static constexpr int LZ = W + 1;      // floats per row of the chain's tiles (odd: conflict-free column reads)
  union {
    alignas(16) unsigned short a[2][T * AS];   // activations: [part][row][feature]
    float chain[2][32 * LZ];                   // the FP32 chain's input and output of a layer, 32 pairs
  } u;
  float unscale[T];               // per row: undoes the scale of the current input
  float top[8][T];                // per wave and row: a layer's largest output
  float part[8][T][8];            // layer 3: each wave's part
  int32_t bad[T];                 // per row: a value out of range
  int32_t any_bad;
};

// acc[c][t] = the wave's column tile c times the rows of tile t, over KDIM inputs: a lane has 16 outputs of row l32
template <int KDIM, int AS, int CT, int RT>
__device__ __forceinline__ void head_products(const unsigned short* __restrict__ pack, size_t part_stride,
                                              const unsigned short* a, size_t a_part, int wave, int lane,
                                              f32x16 (&acc)[CT][RT]) {
  constexpr int KS = KDIM / 16, D = 2;
  static_assert(KS % D == 0, "k-steps");
  const int g = lane >> 5, l32 = lane & 31;
  const u32x4* b0 = reinterpret_cast<const u32x4*>(pack) + (size_t)wave * CT * KS * 64 + lane;
  const u32x4* b1 = reinterpret_cast<const u32x4*>(pack + part_stride) + (size_t)wave * CT * KS * 64 + lane;
  const unsigned short* row = a + l32 * AS + 8 * g;
  // sums of the small products: apart where the registers allow it (by the width alone, so that a pair's result does
  // not depend on the tiles of its batch)
  constexpr bool APART = CT == 1;
  f32x16 low[APART ? CT : 1][APART ? RT : 1];
#pragma unroll
  for (int c = 0; c < CT; ++c)
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      acc[c][t] = f32x16{};
      if constexpr (APART) low[c][t] = f32x16{};
    }
  auto lo = [&](int c, int t) __attribute__((always_inline)) -> f32x16& {
    if constexpr (APART)
      return low[c][t];
    else
      return acc[c][t];
  };
  u32x4 q0[D][CT], q1[D][CT];
#pragma unroll
  for (int d = 0; d < D; ++d)
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      q0[d][c] = b0[(c * KS + d) * 64];
      q1[d][c] = b1[(c * KS + d) * 64];
    }
#pragma unroll 1
  for (int s0 = 0; s0 < KS; s0 += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int s = s0 + d;
      u32x4 x0[RT], x1[RT];
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        x0[t] = *reinterpret_cast<const u32x4*>(row + 32 * t * AS + 16 * s);
        x1[t] = *reinterpret_cast<const u32x4*>(row + a_part + 32 * t * AS + 16 * s);
      }
#pragma unroll
      for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int t = 0; t < RT; ++t) {
          lo(c, t) = mfma_k16(q0[d][c], x1[t], lo(c, t));
          lo(c, t) = mfma_k16(q1[d][c], x0[t], lo(c, t));
          acc[c][t] = mfma_k16(q0[d][c], x0[t], acc[c][t]);
        }
      const int n = s + D < KS ? s + D : s;  // (past the end: a repeated load that nothing uses)
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        q0[d][c] = b0[(c * KS + n) * 64];
        q1[d][c] = b1[(c * KS + n) * 64];
      }
      __builtin_amdgcn_sched_barrier(0);  // the loads stay here, D steps ahead of their use
    }
  }
  if constexpr (APART)
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int t = 0; t < RT; ++t) acc[c][t] = acc[c][t] + low[c][t];
}

// The head as a chain of FP32 products for the pairs of a tile with a value or weight out of the halves' range: 32 at
// a time, by the first four waves of the workgroup (all of it enters); zt and gt are [32][ld] tiles, ys receives the
// raw outputs of the marked rows of T.
template <int Z, int HH>
__device__ __forceinline__ void head_chain(const Fp32Net& W, const NetArgs& A, int p0, int P, int T, float* zt, float* gt,
                                           int ld, const int32_t* bad, float (*ys)[8]) {
  constexpr int CT = HH / 128;
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int r0 = 0; r0 < T; r0 += 32) {
    __syncthreads();
    for (int e = tid; e < 32 * Z; e += 512) {
      const int i = e / Z, k = e - i * Z, p = p0 + r0 + i;
      const float v = p < P ? A.z[(size_t)p * Z + k] : 0.f;
      zt[i * ld + k] = v == v ? v : 0.f;
    }
    __syncthreads();
    for (int layer = 0; layer < 2; ++layer) {
      const float* src = layer ? gt : zt;
      float* dst = layer ? zt : gt;
      const int KS = (layer ? HH : Z) / 2;
      const float* pack = layer ? W.h2pack : W.h1pack;
      const float* bias = layer ? W.c2 : W.c1;
      f32x16 acc[CT];
#pragma unroll
      for (int c = 0; c < CT; ++c) acc[c] = f32x16{};
      if (wave < 4)
#pragma unroll 1
        for (int s = 0; s < KS; ++s) {
          const float av = src[l32 * ld + 2 * s + g];
#pragma unroll
          for (int c = 0; c < CT; ++c)
            acc[c] = mfma32x32x2(av, pack[((size_t)(wave * CT + c) * KS + s) * 64 + lane], acc[c]);
        }
      __syncthreads();
      if (wave < 4)
#pragma unroll
        for (int c = 0; c < CT; ++c) {
          const int col = (wave * CT + c) * 32 + l32;
#pragma unroll
          for (int r = 0; r < 16; ++r) dst[(8 * (r >> 2) + 4 * g + (r & 3)) * ld + col] = fmaxf(acc[c][r] + bias[col], 0.f);
        }
      __syncthreads();
    }
    if (tid < 256 && bad[r0 + (tid >> 3)]) {
      const int i = tid >> 3, o = tid & 7;
      float y = 0.f;
      for (int k = 0; k < HH; ++k) y += zt[i * ld + k] * W.h3[(size_t)o * HH + k];
      ys[r0 + i][o] = y + W.c3[o];
    }
  }
  __syncthreads();
}

template <int Z, int HH, int RT>
__global__ __launch_bounds__(512, 2) void head_split_kernel(Fp32Net W, NetArgs A) {
  using S_t = HeadSmem<Z, HH, RT>;
  constexpr int T = S_t::T, AS = S_t::AS, CT = HH / 256, KS3 = HH / 16;
  constexpr size_t AP = (size_t)T * AS;
  extern __shared__ __align__(16) unsigned char smem[];
  S_t& S = *reinterpret_cast<S_t*>(smem);
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int p0 = blockIdx.x * T;
  const int P = pair_count(A.n_pairs, A.n_pairs_dev);
  if (p0 >= P) return;  // uniform
  const int weights_bad = *W.split_bad;
  if (tid < T) S.bad[tid] = weights_bad;
  if (tid == 0) S.any_bad = weights_bad;
  __syncthreads();

  // the features of a pair per wave at a time: 4 consecutive ones per lane and load
  constexpr int NL = (Z + 255) / 256;
#pragma unroll 4
  for (int i = 0; i < T / 8; ++i) {
    const int r = wave + 8 * i, p = p0 + r;
    float4 v[NL];
    float mx = 0.f;
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      v[k] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (p < P) v[k] = *reinterpret_cast<const float4*>(A.z + (size_t)p * Z + 256 * k + 4 * lane);
      // an invalid pair's NaN features: its outputs are NaN-ed in the epilogue
      v[k].x = v[k].x == v[k].x ? v[k].x : 0.f;
      v[k].y = v[k].y == v[k].y ? v[k].y : 0.f;
      v[k].z = v[k].z == v[k].z ? v[k].z : 0.f;
      v[k].w = v[k].w == v[k].w ? v[k].w : 0.f;
      mx = fmaxf(mx, fmaxf(fmaxf(fabsf(v[k].x), fabsf(v[k].y)), fmaxf(fabsf(v[k].z), fabsf(v[k].w))));
    }
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) mx = fmaxf(mx, __shfl_xor(mx, d, 64));
    const float sc = halves_scale(mx), short_below = kHalvesLeast * halves_unscale(sc);
    unsigned least = ~0u;  // bits of the smallest feature that is not 0, minus 1 (a 0: the largest)
#pragma unroll
    for (int k = 0; k < NL; ++k)
      least = min(min(least, min(__float_as_uint(v[k].x) - 1u, __float_as_uint(v[k].y) - 1u)),
                  min(__float_as_uint(v[k].z) - 1u, __float_as_uint(v[k].w) - 1u));
    bool bad = !(mx <= 0x1p100f);
    if (__ballot(least < __float_as_uint(short_below) - 1u) != 0) {  // rare
      int some = 0, lost = 0;
#pragma unroll
      for (int k = 0; k < NL; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float x = e == 0 ? v[k].x : (e == 1 ? v[k].y : (e == 2 ? v[k].z : v[k].w));
          some += __popcll(__ballot(x > 0.f));
          lost += __popcll(__ballot((x > 0.f) & (x < short_below)));
        }
      bad |= halves_short(some << 16 | lost, kShortActivations);
    }
    if (lane == 0) {
      S.unscale[r] = halves_unscale(sc);
      if (bad) S.bad[r] = S.any_bad = 1;
    }
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      float a = v[k].x * sc, b = v[k].y * sc, c = v[k].z * sc, d = v[k].w * sc;
      uint2 h, l;
      h.x = split_part(a, b);
      h.y = split_part(c, d);
      l.x = last_part(a, b);
      l.y = last_part(c, d);
      unsigned short* dst = &S.u.a[0][r * AS + 256 * k + 4 * lane];
      *reinterpret_cast<uint2*>(dst) = h;
      *reinterpret_cast<uint2*>(dst + AP) = l;
    }
  }
  __syncthreads();

  f32x16 acc[CT][RT];
  float down[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) down[t] = S.unscale[32 * t + l32];
#pragma unroll
  for (int layer = 0; layer < 2; ++layer) {
    const float* bias = (layer ? W.c2 : W.c1) + wave * CT * 32 + 4 * g;
    const float* un = (layer ? W.unscale_h2 : W.unscale_h1) + wave * CT * 32 + 4 * g;
    float4 u4[CT][4], b4[CT][4];
    auto load_scales = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          u4[c][q] = *reinterpret_cast<const float4*>(un + 32 * c + 8 * q);
          b4[c][q] = *reinterpret_cast<const float4*>(bias + 32 * c + 8 * q);
        }
    };
    if (RT > 1) load_scales();
    if (layer == 0)
      head_products<Z, AS, CT, RT>(W.h1s, (size_t)HH * Z, S.u.a[0], AP, wave, lane, acc);
    else
      head_products<HH, AS, CT, RT>(W.h2s, (size_t)HH * HH, S.u.a[0], AP, wave, lane, acc);
    if (RT == 1) load_scales();
    float top[RT];
    unsigned least[RT];  // bits of the smallest output that is not negative
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      top[t] = 0.f;
      least[t] = ~0u;
    }
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float u[4] = {u4[c][q].x, u4[c][q].y, u4[c][q].z, u4[c][q].w};
        const float b[4] = {b4[c][q].x, b4[c][q].y, b4[c][q].z, b4[c][q].w};
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float v = __builtin_fmaf(acc[c][t][4 * q + e], down[t] * u[e], b[e]);
            acc[c][t][4 * q + e] = v;
            top[t] = vmax(top[t], v);
            least[t] = min(least[t], __float_as_uint(v));
          }
      }
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      top[t] = vmax(top[t], __shfl_xor(top[t], 32, 64));
      if (lane < 32) S.top[wave][32 * t + lane] = top[t];
    }
    __syncthreads();  // every wave has read the layer's inputs
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const int row = 32 * t + l32;
      float mx = 0.f;
#pragma unroll
      for (int w = 0; w < 8; ++w) mx = vmax(mx, S.top[w][row]);
      const float sc = halves_scale(mx);
      down[t] = halves_unscale(sc);
      if (tid < 32) {
        S.unscale[row] = down[t];
        if (!(mx <= 0x1p100f)) S.bad[row] = S.any_bad = 1;
      }
      const float short_below = kHalvesLeast * down[t];
      if (__ballot((least[t] < __float_as_uint(short_below)) & (mx > 0.f)) != 0) {  // rare: in the wave's columns
        int some = 0, lost = 0;
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            some += acc[c][t][r] > 0.f;
            lost += acc[c][t][r] > 0.f && acc[c][t][r] < short_below;
          }
        int count = some << 16 | lost;
        count += __shfl_xor(count, 32, 64);
        if (lane < 32 && halves_short(count, kShortActivations)) S.bad[row] = S.any_bad = 1;
      }
#pragma unroll
      for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = vmax(acc[c][t][4 * q + e], 0.f) * sc;
          uint2 h, l;
          h.x = split_part(v[0], v[1]);
          h.y = split_part(v[2], v[3]);
          l.x = last_part(v[0], v[1]);
          l.y = last_part(v[2], v[3]);
          unsigned short* dst = &S.u.a[0][row * AS + (wave * CT + c) * 32 + 8 * q + 4 * g];
          *reinterpret_cast<uint2*>(dst) = h;
          *reinterpret_cast<uint2*>(dst + AP) = l;
        }
    }
    __syncthreads();
  }

  // layer 3: 8 outputs padded to 32 columns, the reduction split over the waves
  {
    constexpr int KW = KS3 / 8;
    const u32x4* b0 = reinterpret_cast<const u32x4*>(W.h3s) + lane;
    const u32x4* b1 = b0 + KS3 * 64;
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      f32x16 hi = f32x16{}, lo = f32x16{};
      const unsigned short* row = &S.u.a[0][(32 * t + l32) * AS + 8 * g];
#pragma unroll
      for (int s = wave * KW; s < (wave + 1) * KW; ++s) {
        const u32x4 x0 = *reinterpret_cast<const u32x4*>(row + 16 * s);
        const u32x4 x1 = *reinterpret_cast<const u32x4*>(row + AP + 16 * s);
        const u32x4 w0 = b0[s * 64], w1 = b1[s * 64];
        lo = mfma_k16(x1, w0, lo);
        hi = mfma_k16(x0, w0, hi);
        lo = mfma_k16(x0, w1, lo);
      }
      if (l32 < 8)
#pragma unroll
        for (int r = 0; r < 16; ++r) S.part[wave][32 * t + 8 * (r >> 2) + 4 * g + (r & 3)][l32] = hi[r] + lo[r];
    }
  }
  __syncthreads();
  for (int i = tid; i < T * 8; i += 512) {
    const int r = i >> 3, j = i & 7;
    float y = 0.f;
#pragma unroll
    for (int w = 0; w < 8; ++w) y += S.part[w][r][j];
    S.part[0][r][j] = __builtin_fmaf(y, S.unscale[r] * W.unscale_h3[j], W.c3[j]);
  }
  __syncthreads();
  if (S.any_bad)  // uniform
    head_chain<Z, HH>(W, A, p0, P, T, S.u.chain[0], S.u.chain[1], S_t::LZ, S.bad, S.part[0]);
  if (tid < T && p0 + tid < P) {
    const PairMeta mt = A.meta[p0 + tid];
    post_contact(A.objs, mt.a, mt.swapped, S.part[0][tid], A.out, A.y_dbg, p0 + tid);
  }
}

// ------------------------------------------------------------- weights, launch

// Repacking.  The first workgroups, an element per thread: the gather, layer 1 and W2^T for the chains, the head's
// operands of the gradient kernels, and layer 1's operand times its factor.  The others, eight inputs of a row per
// thread: the halves of W2, H1, H2 and H3 (8 rows, zero to 32) in the B operand order of 32x32x16 products (W2's
// reduction index in layer 1's output order), each row times the power of two that puts its largest weight at 2^14 to
// 2^15, found here by the row's threads, and W2's columns times what undoes the powers of two of layer 1's units, so
// that the halves follow the weights through training.  A weight 2^-16 of its row's largest or less keeps fewer bits
// than a float.  A few in a row do not matter beside the others; where they are more than a 64th of the row's and one (as
// when the largest weight is that of a unit which is always 0), or a weight is not finite, the flag word becomes 1 and
// every pair takes the FP32 chains.  One launch: training runs it every step.

// A hidden unit's largest output for normals in [-1, 1] and coordinates in the library's unit in [-1, 1] is its weights'
// and bias' absolute sum (the coordinates' times the unit); unit_power is the power of two that takes it to (2^14, 2^15]
// (of a sum of at least 2^-100; 0 for a unit without weights; NaN past 2^100 and for weights that are not finite).
__device__ __forceinline__ float unit_power(const float* __restrict__ raw, int h1, float unit, int f) {
  float sum = __builtin_fabsf(raw[6 * h1 + f]);
#pragma unroll
  for (int c = 0; c < 6; ++c) sum += __builtin_fabsf(raw[6 * f + c]) * (c < 3 ? unit : 1.f);
  if (!(sum <= 0x1p100f)) return __builtin_nanf("");
  const int e = (int)((__float_as_uint(fmaxf(sum, 0x1p-100f)) + 0x007fffffu) >> 23) - 127;  // ceil(log2 sum)
  return sum == 0.f ? 0.f : __uint_as_float((unsigned)(127 + 15 - e) << 23);
}

struct RepackSizes {
  int pack, w1, w1c, w2c, frag;  // elements, in this order
  int halves[4];                 // rows' eighths of W2, H1, H2, H3: multiples of 256
  __host__ __device__ int elements() const { return pack + w1 + w1c + w2c + frag; }
  __host__ __device__ int element_blocks() const { return (elements() + 255) / 256; }
};
RepackSizes repack_sizes(int pack_n, int h1, int h2, int hh) {
  return RepackSizes{pack_n,
                     8 * h1,
                     8 * h1,
                     h2 * h1,
                     2 * (hh * 2 * h2 + hh * hh),
                     {h2 * h1 / 8, hh * 2 * h2 / 8, hh * hh / 8, 32 * hh / 8}};
}

__device__ __forceinline__ void repack_halves(const RepackArgs& A, const SplitLayout& L, const RepackSizes& Z, int i) {
  int mat = 0;
#pragma unroll
  for (int k = 0; k < 3; ++k)
    if (mat == k && i >= Z.halves[k]) {
      i -= Z.halves[k];
      mat = k + 1;
    }
  char* const base = A.split;
  const int in = mat == 0 ? L.h1 : (mat == 1 ? 2 * L.h2 : L.hh), lanes = in / 8;  // 8 to 64 lanes of a wave a row
  const int row = i / lanes, j = i % lanes, s = j >> 1, g = j & 1;
  __shared__ float unit[128];  // W2's inputs: what undoes their units' powers of two
  if (mat == 0) {              // uniform
    for (int f = threadIdx.x; f < in; f += 256) {
      const float up = unit_power(A.raw, L.h1, A.unit, f);
      unit[f] = up > 0.f ? 1.f / up : 0.f;
    }
    __syncthreads();
  }
  const int oW2 = 7 * L.h1, oH1 = oW2 + L.h2 * L.h1 + L.h2, oH2 = oH1 + L.hh * 2 * L.h2 + L.hh,
            oH3 = oH2 + L.hh * L.hh + L.hh;
  const float* W = A.raw + (mat == 0 ? oW2 : (mat == 1 ? oH1 : (mat == 2 ? oH2 : oH3)));
  const bool zero = mat == 3 && row >= 8;
  float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (!zero) {
    const float* src = W + (size_t)row * in + 16 * s + (mat == 0 ? 4 : 8) * g;
    const float4 a = *reinterpret_cast<const float4*>(src), b = *reinterpret_cast<const float4*>(src + (mat == 0 ? 8 : 4));
    v[0] = a.x, v[1] = a.y, v[2] = a.z, v[3] = a.w, v[4] = b.x, v[5] = b.y, v[6] = b.z, v[7] = b.w;
    if (mat == 0)
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] *= unit[16 * s + 4 * g + e + (e < 4 ? 0 : 4)];
  }
  float mx = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) mx = fmaxf(mx, __builtin_fabsf(v[e]));
  for (int d = 1; d < lanes; d <<= 1) mx = fmaxf(mx, __shfl_xor(mx, d, 64));
  const float up = halves_scale(mx);
  int lost = 0, some = 0;
  bool bad = false;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const bool any = v[e] != 0.f;
    v[e] *= up;
    some += any;
    lost += any && __builtin_fabsf(v[e]) < kHalvesLeast;
    bad |= !(__builtin_fabsf(v[e]) <= kSplitLimit);
  }
  int count = some << 16 | lost;
  for (int d = 1; d < lanes; d <<= 1) count += __shfl_xor(count, d, 64);
  if (bad || halves_short(count, kShortWeights)) *reinterpret_cast<int32_t*>(base) = 1;
  u32x4 part[2];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    part[0][e] = split_part(v[2 * e], v[2 * e + 1]);
    part[1][e] = last_part(v[2 * e], v[2 * e + 1]);
  }
  const size_t at = ((size_t)(row / 32) * (in / 16) + s) * 64 + row % 32 + 32 * g;
  const size_t stride = (size_t)(mat == 0 ? Z.halves[0] : (mat == 1 ? Z.halves[1] : (mat == 2 ? Z.halves[2] : Z.halves[3])));
  u32x4* dst = reinterpret_cast<u32x4*>(base + (mat == 0 ? L.w2 : (mat == 1 ? L.H1 : (mat == 2 ? L.H2 : L.H3)))) + at;
  dst[0] = part[0];
  dst[stride] = part[1];
  if (j == 0 && !zero)
    reinterpret_cast<float*>(base + L.scale)[(mat == 0 ? 0 : (mat == 1 ? L.h2 : L.h2 + (mat - 1) * L.hh)) + row] = 1.f / up;
}

__global__ __launch_bounds__(256) void repack_kernel(RepackArgs A, SplitLayout L, RepackSizes Z) {
  char* const base = A.split;
  int i = blockIdx.x * 256 + threadIdx.x;
  if ((int)blockIdx.x >= Z.element_blocks()) {
    repack_halves(A, L, Z, i - Z.element_blocks() * 256);
    return;
  }
  if (i < Z.pack) {
    const int32_t k = A.pack_idx[i];
    A.pack[i] = k >= 0 ? A.raw[k] : 0.f;
    return;
  }
  i -= Z.pack;
  const float* raw = A.raw;
  if (i < Z.w1) {  // [W1 | b1 | 0][f][c], f = 32 ft + l % 32, c = 2 s + l / 32, at (4 ft + s) 64 + l
    const int l = i & 63, f = 32 * (i >> 8) + l % 32, c = 2 * ((i >> 6) & 3) + l / 32;
    const float up = unit_power(raw, L.h1, A.unit, f), w = c < 6 ? raw[6 * f + c] : (c == 6 ? raw[6 * L.h1 + f] : 0.f);
    const float v = up == 0.f && c == 6 ? -1.f : w * up;  // (a unit without weights, which W2 does not read: below 0)
    if (!(__builtin_fabsf(v) <= 0x1p126f)) *reinterpret_cast<int32_t*>(base) = 1;
    reinterpret_cast<float*>(base + L.w1)[i] = v;
    return;
  }
  i -= Z.w1;
  // layer 1's rows (w0 .. w5, b, 0) and W2^T in the order of layer 2's reduction: step s is feature
  // F(s / 32, s % 2, (s / 2) % 16)
  if (i < Z.w1c + Z.w2c) {
    const bool first = i < Z.w1c;
    const int at = first ? i : i - Z.w1c, s = first ? at >> 3 : at / L.h2, c = first ? at & 7 : at % L.h2;
    const int f = perm_feature(s / 32, s % 2, (s / 2) % 16);
    if (first)
      reinterpret_cast<float*>(base + L.w1c)[at] = c < 6 ? raw[6 * f + c] : (c == 6 ? raw[6 * L.h1 + f] : 0.f);
    else
      reinterpret_cast<float*>(base + L.w2c)[at] = raw[7 * L.h1 + (size_t)c * L.h1 + f];
    return;
  }
  i -= Z.w1c + Z.w2c;
  // H1, H2, H2^T and H1^T [out][in] as operands of 16x16x4 products: lane l of step u of column tile ct holds
  // M[16 ct + l % 16][16 u + 4 (l / 16) .. + 3]
  if (i >= Z.frag) return;
  const int f1 = L.hh * 2 * L.h2, f2 = L.hh * L.hh, offH1 = 7 * L.h1 + L.h2 * L.h1 + L.h2, offH2 = offH1 + f1 + L.hh;
  const int mat = i < f1 ? 0 : (i < f1 + f2 ? 1 : (i < f1 + 2 * f2 ? 2 : 3));
  const int at = i - (mat == 0 ? 0 : (mat == 1 ? f1 : (mat == 2 ? f1 + f2 : f1 + 2 * f2)));
  const int steps = (mat == 0 ? 2 * L.h2 : L.hh) / 16, l = (at >> 2) & 63;
  const int row = 16 * ((at >> 8) / steps) + l % 16, k = 16 * ((at >> 8) % steps) + 4 * (l / 16) + (at & 3);
  A.frag[i] = raw[mat == 0   ? offH1 + row * 2 * L.h2 + k
                  : mat == 1 ? offH2 + row * L.hh + k
                  : mat == 2 ? offH2 + k * L.hh + row
                             : offH1 + k * 2 * L.h2 + row];
}

// Chunk sizes: half of what is left over the grid, 32 to 1. A batch of up to `lone` pairs a workgroup is dealt out
// evenly in one claim each, without the queue: the pairs of a call cost nearly the same, and the halving levels' claims
// cost more than the even split loses. At 64 / 128 (two workgroups a CU, grid 512) 2,000 pairs 61.5 -> 45.3 us, 8,000
// 110.0 -> 100.0, 12,000 147.2 -> 140.9, but with the argmax 16,000 380.6 -> 387.0; at 128 / 256 (grid 256), whose
// pairs are four times as long, 1,000 pairs 91.9 -> 87.8, but 1,400 106.4 -> 108.3. A batch whose length the device
// holds may be far shorter than n_pairs, and one claim of its capacity's share would leave workgroups without work.
SplitChunks split_chunks(int n_pairs, int grid, int lone) {
  SplitChunks c{};
  c.grid = grid;
  int left = n_pairs, base = 0;
  for (int l = 0; l < SplitChunks::kLevels; ++l) {
    int size = left / (2 * grid);
    int claims = grid;
    if (size >= kSplitChunk) {
      size = kSplitChunk;
      claims = (left - 2 * grid * kSplitChunk) / kSplitChunk + grid;
    }
    if (l == 0 && n_pairs <= (long long)lone * grid) size = (n_pairs + grid - 1) / grid;
    if (size < 1) size = 1;
    c.size[l] = size;
    c.base[l] = base;
    c.claims[l] = claims;
    base += size * claims;
    left -= size * claims;
    if (left < 0) left = 0;
  }
  return c;
}

template <int H1, int H2>
hipError_t run_split(const Fp32Net& w, const NetArgs& a, int n_cu, hipStream_t s) {
  const int slots = n_cu * (H2 >= 256 ? 1 : 2);  // workgroups the register file holds at once (four spill: 98 -> 166 us)
  const int grid = a.n_pairs < slots ? a.n_pairs : slots;
  const int lone = a.n_pairs_dev ? 0 : (H2 >= 256 ? 4 : 24);
  if (a.amax)
    kernel_launch((encoder_split_kernel<H1, H2, true>), dim3(grid), dim3(2 * H2), 0, s, w, a,
                  split_chunks(a.n_pairs, grid, lone));
  else
    kernel_launch((encoder_split_kernel<H1, H2, false>), dim3(grid), dim3(2 * H2), 0, s, w, a,
                  split_chunks(a.n_pairs, grid, lone));
  return hipGetLastError();
}

template <int H1, int H2>
hipError_t run_chain(const Fp32Net& w, const NetArgs& a, hipStream_t s) {
  const size_t objects = 2 * (size_t)a.n_pairs;
  if (a.n_pairs <= kChainLonePairs)
    kernel_launch((chain_features_kernel<H1, H2, 1>), dim3((unsigned)objects), dim3(H2), 0, s, w, a);
  else
    kernel_launch((chain_features_kernel<H1, H2, kChainObjects>),
                  dim3((unsigned)((objects + kChainObjects - 1) / kChainObjects)), dim3(H2), 0, s, w, a);
  return hipGetLastError();
}

template <int Z, int HH, int RT>
hipError_t run_head(const Fp32Net& w, const NetArgs& a, hipStream_t s) {
  constexpr size_t smem = sizeof(HeadSmem<Z, HH, RT>);
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&head_split_kernel<Z, HH, RT>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (e != hipSuccess) return e;
  kernel_launch((head_split_kernel<Z, HH, RT>), dim3((a.n_pairs + 32 * RT - 1) / (32 * RT)), dim3(512), smem, s, w, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_head_split(const Fp32Net& w, const NetArgs& a, int n_cu, hipStream_t s) {
  if (a.n_pairs <= 0) return hipSuccess;
  if (!w.h1s || !w.split_bad) return hipErrorInvalidValue;
  // One tile per workgroup while every workgroup has a compute unit of its own (the weight stream is the same, the
  // matrix work half); from there on two tiles halve the streams (8,192 pairs at width 512: 368 us with one, 380 with two;
  // 9,000: 424, 411).
  const bool two = a.n_pairs > 32 * n_cu;
  if (w.h2 == 128 && w.hh == 256) return two ? run_head<256, 256, 2>(w, a, s) : run_head<256, 256, 1>(w, a, s);
  if (w.h2 == 256 && w.hh == 512) return two ? run_head<512, 512, 2>(w, a, s) : run_head<512, 512, 1>(w, a, s);
  return hipErrorInvalidValue;
}

hipError_t launch_encoder_split(const Fp32Net& w, const NetArgs& a, int n_cu, hipStream_t s) {
  if (a.n_pairs <= 0) return hipSuccess;
  if (!w.w2s || !w.split_bad || (a.amax ? !a.doubt : !a.z)) return hipErrorInvalidValue;
  if (w.h1 == 64 && w.h2 == 128) return run_split<64, 128>(w, a, n_cu, s);
  if (w.h1 == 128 && w.h2 == 256) return run_split<128, 256>(w, a, n_cu, s);
  return hipErrorInvalidValue;
}

Fp32Net fp32_view(const float* base, int h1, int h2, int hh) {
  const Fp32Layout L = fp32_layout(h1, h2, hh);
  Fp32Net w{};
  w.h1 = h1;
  w.h2 = h2;
  w.hh = hh;
  w.w1pack = base + L.w1;
  w.w2pack = base + L.w2;
  w.b2 = base + L.b2;
  w.h1pack = base + L.h1;
  w.c1 = base + L.c1;
  w.h2pack = base + L.h2;
  w.c2 = base + L.c2;
  w.h3 = base + L.h3;
  w.c3 = base + L.c3;
  return w;
}

void split_bind(Fp32Net& w, const char* base) {
  const SplitLayout L = split_layout(w.h1, w.h2, w.hh);
  w.split_bad = reinterpret_cast<const int32_t*>(base);
  const float* scale = reinterpret_cast<const float*>(base + L.scale);
  w.unscale2 = scale;
  w.unscale_h1 = w.unscale2 + L.h2;
  w.unscale_h2 = w.unscale_h1 + L.hh;
  w.unscale_h3 = w.unscale_h2 + L.hh;
  w.w1c = reinterpret_cast<const float*>(base + L.w1c);
  w.w2c = reinterpret_cast<const float*>(base + L.w2c);
  w.w1s = reinterpret_cast<const float*>(base + L.w1);
  w.w2s = reinterpret_cast<const unsigned short*>(base + L.w2);
  w.h1s = reinterpret_cast<const unsigned short*>(base + L.H1);
  w.h2s = reinterpret_cast<const unsigned short*>(base + L.H2);
  w.h3s = reinterpret_cast<const unsigned short*>(base + L.H3);
}

hipError_t launch_chain_features(const Fp32Net& w, const NetArgs& a, hipStream_t s) {
  if (a.n_pairs <= 0) return hipSuccess;
  if (!w.w2c || !a.z || !a.amax || !a.doubt) return hipErrorInvalidValue;
  if (w.h1 == 64 && w.h2 == 128) return run_chain<64, 128>(w, a, s);
  if (w.h1 == 128 && w.h2 == 256) return run_chain<128, 256>(w, a, s);
  return hipErrorInvalidValue;
}

hipError_t launch_repack(const RepackArgs& a, hipStream_t s) {
  const RepackSizes z = repack_sizes(a.pack_n, a.h1, a.h2, a.hh);
  const int halves = (z.halves[0] + z.halves[1] + z.halves[2] + z.halves[3]) / 256;
  kernel_launch(repack_kernel, dim3(z.element_blocks() + halves), dim3(256), 0, s, a, split_layout(a.h1, a.h2, a.hh), z);
  return hipGetLastError();
}

}  // namespace locc
