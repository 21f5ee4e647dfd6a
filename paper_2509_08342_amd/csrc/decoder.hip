// Kernels of the decoder loop around the split-expert MoE layer (Sec. 2.1:
// an attention module, Eq. (1), then the MoE module, Eq. (2), per layer;
// the head after the last layer): dense projections, rotary embedding with
// the key/value cache append, causal grouped-query attention, greedy token
// choice and the embedding gather.  Stateless entry points: every buffer is
// the caller's, every call is enqueued on the caller's stream.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "device.h"
#include "kernels.h"
#include "moesplit.h"

namespace {

constexpr int kDenseThreads = 256;
constexpr int kDenseRows = 8;        // output rows per work-group (two per wave)
constexpr int kAttThreads = 256;
constexpr int kAttWideThreads = 1024;  // single-token steps
constexpr int kAttMaxScores = 16000;  // floats of queries and scores a work-group keeps in LDS (< 64 KiB)

__device__ __forceinline__ void bf16x8_to_f32(uint4 v, float (&o)[8]) {
  o[0] = __uint_as_float(v.x << 16);
  o[1] = __uint_as_float(v.x & 0xffff0000u);
  o[2] = __uint_as_float(v.y << 16);
  o[3] = __uint_as_float(v.y & 0xffff0000u);
  o[4] = __uint_as_float(v.z << 16);
  o[5] = __uint_as_float(v.z & 0xffff0000u);
  o[6] = __uint_as_float(v.w << 16);
  o[7] = __uint_as_float(v.w & 0xffff0000u);
}

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float(static_cast<uint32_t>(b) << 16); }

__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  const uint32_t u = __float_as_uint(f);
  return static_cast<uint16_t>((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

// ------------------------------------------------------------------ dense
//
// y[t][o] = sum_i x[t][i] W[o][i] (+ add[t][o]): W [n_out][n_in] bf16 rows
// (the nn.Linear layout), x bf16, y fp32.  A work-group takes 8 output rows,
// two per wave; lanes stride over the row in 16-byte pieces with every
// piece of a row requested before use; NT tokens of x sit in LDS per pass.
template <int NT, int PJ>
__global__ __launch_bounds__(kDenseThreads) void dense_kernel(const uint16_t* __restrict__ x,
                                                              const uint16_t* __restrict__ w,
                                                              const float* __restrict__ add, float* __restrict__ y,
                                                              int T, int n_in, int n_out) {
  extern __shared__ __align__(16) uint16_t xs[];  // [NT][n_in]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row0 = blockIdx.x * kDenseRows + 2 * wave;
  const int pieces = n_in / 8;
  constexpr int PMAX = PJ;  // pieces per lane at the largest n_in of this variant
  for (int t0 = 0; t0 < T; t0 += NT) {
    const int nt = min(NT, T - t0);
    __syncthreads();  // the previous tile's readers are done
    for (int i = tid; i < NT * pieces; i += kDenseThreads) {
      const int t = i / pieces, p = i - t * pieces;
      uint4 v = make_uint4(0, 0, 0, 0);
      if (t < nt) v = *reinterpret_cast<const uint4*>(x + static_cast<size_t>(t0 + t) * n_in + 8 * p);
      *reinterpret_cast<uint4*>(xs + static_cast<size_t>(t) * n_in + 8 * p) = v;
    }
    __syncthreads();
    float acc[2][NT];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[r][t] = 0.0f;
    uint4 wv[2][PMAX];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int row = min(row0 + r, n_out - 1);  // clamped: rows past n_out are not stored
#pragma unroll
      for (int j = 0; j < PMAX; ++j) {
        const int p = lane + 64 * j;
        if (p < pieces) wv[r][j] = *reinterpret_cast<const uint4*>(w + static_cast<size_t>(row) * n_in + 8 * p);
      }
    }
#pragma unroll
    for (int j = 0; j < PMAX; ++j) {
      const int p = lane + 64 * j;
      if (p < pieces) {
        float wf[2][8];
        bf16x8_to_f32(wv[0][j], wf[0]);
        bf16x8_to_f32(wv[1][j], wf[1]);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          float xf[8];
          bf16x8_to_f32(*reinterpret_cast<const uint4*>(xs + static_cast<size_t>(t) * n_in + 8 * p), xf);
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            acc[0][t] = fmaf(wf[0][e], xf[e], acc[0][t]);
            acc[1][t] = fmaf(wf[1][e], xf[e], acc[1][t]);
          }
        }
      }
    }
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int t = 0; t < NT; ++t) {
#pragma unroll
        for (int s = 32; s >= 1; s >>= 1) acc[r][t] += __shfl_xor(acc[r][t], s, 64);
      }
    if (lane == 0) {
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int row = row0 + r;
        if (row < n_out) {
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            if (t < nt) {
              const size_t o = static_cast<size_t>(t0 + t) * n_out + row;
              y[o] = acc[r][t] + (add ? add[o] : 0.0f);
            }
          }
        }
      }
    }
  }
}

// ------------------------------------------------------ rotary + KV append
//
// Heads [0, Hq) are query heads (rotated into q_out), [Hq, Hq + Hkv) key
// heads (rotated into the key cache at position pos0 + t), [Hq + Hkv, Hq + 2
// Hkv) value heads (copied into the value cache).  The pair (i, i + D/2) turns
// by the angle p * base^(-2 i / D), computed in double precision.  Block (t,
// y) computes the token's angles once (LDS) and takes every gridDim.y-th slice
// of its pairs, V consecutive pairs per thread (4 where the rows allow
// 16-byte loads).  Every head's own angles bound the kernel before: 2048
// tokens of 32 + 2 x 8 heads of 128, 30.8 -> 13.9 us for 76 MB moved.
//
// Heads up to 128 wide of calls that the GPU takes at once (kRopeFewRows
// heads of all tokens) or of tokens with too few heads to share much take
// rope_kv_few_kernel, block (t, head), whose threads turn their pairs by angles
// of their own: one barrier and LDS round trip less.  So do heads whose angles
// do not fit, and more tokens than the larger blocks can count.  Shared | own
// angles: 1 / 16 tokens of 48 heads of 128 2.7 | 2.3 / 2.9 | 2.4 us, 64 of 8 heads
// of 64 2.8 | 2.3, 3000 of 3 heads of 64 5.3 | 4.3, 1000 of 4 heads of 1200 13.4 |
// 11.4; but 300 tokens of 48 heads of 128 4.0 | 6.5, 1000 of 21 heads of 6 3.2 |
// 7.3, 1000 of 5 heads of 62 3.2 | 3.5, 16 of 4 heads of 512 2.9 | 3.1.
constexpr int kRopeThreads = 256;
constexpr int64_t kRopeFewRows = 2048;
constexpr int kRopeFewHeads = 4;
constexpr int kRopeMaxHalf = 512;  // angles of a token kept in LDS

__device__ __forceinline__ void store_bf16(uint16_t* p, const float (&v)[1]) { *p = f32_to_bf16(v[0]); }
__device__ __forceinline__ void store_bf16(uint16_t* p, const float (&v)[4]) {
  *reinterpret_cast<uint2*>(p) = make_uint2(f32_to_bf16(v[0]) | static_cast<uint32_t>(f32_to_bf16(v[1])) << 16,
                                            f32_to_bf16(v[2]) | static_cast<uint32_t>(f32_to_bf16(v[3])) << 16);
}

// cosine and sine of the angle of pair i at position pos
__device__ __forceinline__ void rope_angle(int pos, int i, int D, double log2_base, float& c, float& s) {
  const double ang = static_cast<double>(pos) * exp2(-2.0 * i / D * log2_base);
  double sn, cs;
  sincos(ang, &sn, &cs);
  c = static_cast<float>(cs);
  s = static_cast<float>(sn);
}

__global__ __launch_bounds__(64) void rope_kv_few_kernel(const float* __restrict__ qkv, int Hq, int Hkv, int D, int pos0,
                                                         double log2_base, uint16_t* __restrict__ q_out,
                                                         uint16_t* __restrict__ kc, uint16_t* __restrict__ vc,
                                                         int max_ctx) {
  const int t = blockIdx.x, head = blockIdx.y, pos = pos0 + t, half = D / 2;
  const float* src = qkv + (static_cast<size_t>(t) * (Hq + 2 * Hkv) + head) * D;
  const bool value = head >= Hq + Hkv;  // stored as is
  uint16_t* dst = head < Hq ? q_out + (static_cast<size_t>(t) * Hq + head) * D
                  : value   ? vc + (static_cast<size_t>(head - Hq - Hkv) * max_ctx + pos) * D
                            : kc + (static_cast<size_t>(head - Hq) * max_ctx + pos) * D;
  for (int i = threadIdx.x; i < half; i += 64) {
    float x1 = src[i], x2 = src[i + half];
    if (!value) {
      float c, s;
      rope_angle(pos, i, D, log2_base, c, s);
      const float r1 = x1 * c - x2 * s, r2 = x2 * c + x1 * s;
      x1 = r1;
      x2 = r2;
    }
    dst[i] = f32_to_bf16(x1);
    dst[i + half] = f32_to_bf16(x2);
  }
}

template <int V>
__global__ __launch_bounds__(kRopeThreads) void rope_kv_kernel(const float* __restrict__ qkv, int Hq, int Hkv, int D,
                                                               int pos0, double log2_base,
                                                               uint16_t* __restrict__ q_out,
                                                               uint16_t* __restrict__ kc, uint16_t* __restrict__ vc,
                                                               int max_ctx) {
  __shared__ float cs_s[kRopeMaxHalf], sn_s[kRopeMaxHalf];
  const int t = blockIdx.x, pos = pos0 + t, half = D / 2, per = half / V;
  for (int i = threadIdx.x; i < half; i += kRopeThreads)  // half <= kRopeMaxHalf
    rope_angle(pos, i, D, log2_base, cs_s[i], sn_s[i]);
  __syncthreads();
  const float* row = qkv + static_cast<size_t>(t) * (Hq + 2 * Hkv) * D;
#pragma unroll 2
  for (int j = blockIdx.y * kRopeThreads + threadIdx.x; j < (Hq + 2 * Hkv) * per; j += gridDim.y * kRopeThreads) {
    const int head = j / per, i = V * (j - head * per);
    const float* src = row + static_cast<size_t>(head) * D + i;
    const bool value = head >= Hq + Hkv;  // stored as is
    uint16_t* dst = i + (head < Hq ? q_out + (static_cast<size_t>(t) * Hq + head) * D
                         : value   ? vc + (static_cast<size_t>(head - Hq - Hkv) * max_ctx + pos) * D
                                   : kc + (static_cast<size_t>(head - Hq) * max_ctx + pos) * D);
    float x1[V], x2[V];
    if constexpr (V == 4) {
      const float4 a = *reinterpret_cast<const float4*>(src), b = *reinterpret_cast<const float4*>(src + half);
      x1[0] = a.x, x1[1] = a.y, x1[2] = a.z, x1[3] = a.w;
      x2[0] = b.x, x2[1] = b.y, x2[2] = b.z, x2[3] = b.w;
    } else {
      x1[0] = src[0];
      x2[0] = src[half];
    }
    if (!value) {
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const float c = cs_s[i + v], s = sn_s[i + v];
        const float r1 = x1[v] * c - x2[v] * s, r2 = x2[v] * c + x1[v] * s;
        x1[v] = r1;
        x2[v] = r2;
      }
    }
    store_bf16(dst, x1);
    store_bf16(dst + half, x2);
  }
}

// ------------------------------------------------------------- attention
//
// Head widths other than 64 and 128, and few tokens with out over q.  Block
// (t, g): the G = Hq / Hkv query heads of key/value group g for token t, over
// positions 0 .. pos0 + t, in BLK threads (1024 for a single-token step, whose
// T x Hkv blocks alone would leave most of the GPU idle; 256 otherwise).  A
// block reads its rows of q before it writes them in out.  Scores in LDS
// ([G][n]); softmax with the row maximum subtracted; then p . V over the
// positions.
template <int BLK>
__device__ __forceinline__ float block_reduce(float v, bool is_max, float* red) {
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) {
    const float o = __shfl_xor(v, s, 64);
    v = is_max ? fmaxf(v, o) : v + o;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wave] = v;
  __syncthreads();
  float r = red[0];
  for (int w = 1; w < BLK / 64; ++w) r = is_max ? fmaxf(r, red[w]) : r + red[w];
  return r;
}

// Whether v holds in any thread of WAVES waves; flags: WAVES ints of LDS that no
// one else uses until the next barrier.  (__syncthreads_or takes LDS of its
// own beside that of the launch.)
template <int WAVES>
__device__ __forceinline__ bool any_thread(bool v, int* flags) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const bool mine = __any(v);
  if (lane == 0) flags[wave] = mine;
  __syncthreads();
  int r = 0;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) r |= flags[w];
  return r != 0;
}

// LDS floats of attention_token for n positions: wave values (16), queries
// [G][D], scores [G][n], wave sums [waves][G][D].
constexpr int kAttRed = 16;
constexpr size_t att_token_floats(int G, int waves, int D, int n) {
  return kAttRed + static_cast<size_t>(G) * ((1 + waves) * D + n);
}

// (stores the output columns [c0, c1) of every head of the group)
template <int G, int BLK>
__device__ __forceinline__ void attention_token(const uint16_t* q, const uint16_t* __restrict__ kc,
                                                const uint16_t* __restrict__ vc, int Hq, int D, int pos0, int max_ctx,
                                                uint16_t* out, int t, int g, int c0, int c1, float* smem) {
  static_assert(BLK / 64 <= kAttRed, "one value per wave");
  const int tid = threadIdx.x;
  const int n = pos0 + t + 1;
  float* red = smem;
  float* qf = smem + kAttRed;
  float* sc = qf + G * D;
  for (int i = tid; i < G * D; i += BLK)
    qf[i] = bf16_to_f32(q[(static_cast<size_t>(t) * Hq + g * G) * D + i]);
  __syncthreads();
  const float scale = 1.0f / sqrtf(static_cast<float>(D));
  const uint16_t* K = kc + static_cast<size_t>(g) * max_ctx * D;
  const uint16_t* V = vc + static_cast<size_t>(g) * max_ctx * D;
  for (int p = tid; p < n; p += BLK) {
    float s[G];
#pragma unroll
    for (int h = 0; h < G; ++h) s[h] = 0.0f;
    for (int k8 = 0; k8 < D; k8 += 8) {
      float kf[8];
      bf16x8_to_f32(*reinterpret_cast<const uint4*>(K + static_cast<size_t>(p) * D + k8), kf);
#pragma unroll
      for (int h = 0; h < G; ++h)
#pragma unroll
        for (int e = 0; e < 8; ++e) s[h] = fmaf(qf[h * D + k8 + e], kf[e], s[h]);
    }
#pragma unroll
    for (int h = 0; h < G; ++h) sc[h * n + p] = s[h] * scale;
  }
  __syncthreads();
  for (int h = 0; h < G; ++h) {
    float m = -INFINITY;
    for (int p = tid; p < n; p += BLK) m = fmaxf(m, sc[h * n + p]);
    m = block_reduce<BLK>(m, true, red);
    float sum = 0.0f;
    for (int p = tid; p < n; p += BLK) {
      const float e = expf(sc[h * n + p] - m);
      sc[h * n + p] = e;
      sum += e;
    }
    sum = block_reduce<BLK>(sum, false, red);
    __syncthreads();
    for (int p = tid; p < n; p += BLK) sc[h * n + p] /= sum;
  }
  __syncthreads();
  // p . V: thread (position lane pl, column group cg) sums 8 columns of every
  // head over positions pl, pl + PL, ... (one 16-byte V load serves all G
  // heads); the position lanes of a wave are combined with shuffles, the
  // waves' sums through LDS (after the scores, which stay in use until then)
  const int CG = D / 8, PL = BLK / CG;
  const int cg = tid % CG, pl = tid / CG;
  float acc[G][8];
#pragma unroll
  for (int h = 0; h < G; ++h)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[h][e] = 0.0f;
  if (pl < PL) {
    for (int p = pl; p < n; p += PL) {
      float vf[8];
      bf16x8_to_f32(*reinterpret_cast<const uint4*>(V + static_cast<size_t>(p) * D + 8 * cg), vf);
#pragma unroll
      for (int h = 0; h < G; ++h) {
        const float pr = sc[h * n + p];
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[h][e] = fmaf(pr, vf[e], acc[h][e]);
      }
    }
  }
  // lanes l and l ^ (CG * 2^j) hold the same columns for other positions
  for (int m = CG; m < 64; m <<= 1)
#pragma unroll
    for (int h = 0; h < G; ++h)
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[h][e] += __shfl_xor(acc[h][e], m, 64);
  float* wsum = sc + G * n;  // [waves][G][D]
  const int lane = tid & 63, wave = tid >> 6;
  if (lane < CG && CG <= 64) {
#pragma unroll
    for (int h = 0; h < G; ++h)
#pragma unroll
      for (int e = 0; e < 8; ++e) wsum[(wave * G + h) * D + 8 * cg + e] = acc[h][e];
  }
  __syncthreads();
  for (int o = tid; o < G * D; o += BLK) {
    float v = 0.0f;
    for (int w = 0; w < BLK / 64; ++w) v += wsum[w * G * D + o];
    const int h = o / D, col = o - h * D;
    if (col >= c0 && col < c1) out[(static_cast<size_t>(t) * Hq + g * G + h) * D + col] = f32_to_bf16(v);
  }
}

template <int G, int BLK>
__global__ __launch_bounds__(BLK) void attention_kernel(const uint16_t* q,
                                                        const uint16_t* __restrict__ kc,
                                                        const uint16_t* __restrict__ vc, int Hq, int D, int pos0,
                                                        int max_ctx, uint16_t* out) {
  extern __shared__ __align__(16) float att_smem[];
  attention_token<G, BLK>(q, kc, vc, Hq, D, pos0, max_ctx, out, blockIdx.x, blockIdx.y, 0, D, att_smem);
}

// ------------------------------------------- attention of prompts (MFMA)
//
// D = 64 or 128, more tokens than attention_few_kernel takes.  A work-group
// takes 64 QB rows of
// one key/value head (a row: one token and one of the head's G query heads,
// heads fastest, so that the group shares every key and value it loads), a
// wave 16 QB of them, over the keys in tiles of 64 with the softmax kept
// online: running maximum m and sum l per row, in 32 bits.
//   S^T = K Q^T: A = 16 keys, B = 16 rows, so a lane ends with the scores of
//   one row (lane % 16) and keys 16 b + 4 (lane / 16) + r of key block b;
//   O^T += V^T P^T: B = the probabilities where they are (contraction slot 4 h
//   + r of lane group g is key 16 (2 ks + h) + 4 g + r), A = V read with
//   transposing LDS reads in the same key order.  A probability enters as three
//   bf16 parts, 8 bits each: all 24 of its mantissa.
// So no value crosses lanes but the maximum of each tile, and the rescaling
// of O (when a maximum grows by more than 2^kAttGrow; until then exponents
// stay relative to the old one) is per lane.  Maxima are kept as unscaled
// scores and subtracted before scaling: the largest key gets exactly 2^0
// however large its score, where the rounding of a scaled maximum would be
// an exponent of its own (more than 128 from scores of about 2^31 on).  K and V tiles go from memory to
// LDS directly, two stages (one in flight); 16-byte piece p of key row u sits
// in slot p ^ (u % 8) (K) or p ^ 2 (u % 4) (V), free of bank conflicts.
//
// A key past a row's position has probability 0.  Its value must not reach
// the row either where it is not finite (0 x inf), and a value of infinity
// that the row does see must not meet the parts of its probability (one of
// them may be 0 or negative).  Either leaves a result that is not finite (so
// does a finite value whose sum passes the largest float): a work-group that
// ends with one computes its rows again, one token at a time, by
// attention_token, which reads no key past the token's.
//
// Bound by VALU work (exponentials, the split) beside the matrix
// cores.  Measured, 32 x 128 query and 8 key/value heads, fma chains per
// token -> now: 2048 tokens 1202 -> 81 us, 512 tokens 92 -> 16.6 us, 100
// tokens at position 1000 87 -> 31 us (the chain of one wave's tiles); with
// two bf16 parts per probability 2048 tokens took 76 us.  Work-group index ->
// key/value head by remainder (8 heads: one per XCD, whose L2 holds its keys
// and values), then the longest row blocks first and the second half shortest
// first, so that two work-groups that share a CU add up to about the same
// work.
constexpr int kAttKeys = 64;       // keys per tile
constexpr float kAttGrow = 8.0f;   // log2 of the largest unscaled probability

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

// (a, b) as three bf16 pairs whose sum is (a, b): rounded, the remainder
// rounded, and what is left (at most 8 bits)
constexpr int kAttParts = 3;
__device__ __forceinline__ void split_pair(float a, float b, uint32_t (&part)[kAttParts]) {
#pragma unroll
  for (int i = 0; i < kAttParts; ++i) {
    part[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{a, b}, bf16x2_t));
    a -= __uint_as_float(part[i] << 16);
    b -= __uint_as_float(part[i] & 0xffff0000u);
  }
}

// eight consecutive bf16 values, 16-byte aligned or not
__device__ __forceinline__ msk::bf16x8_t load_row8(const uint16_t* p, bool aligned) {
  if (aligned) return msk::as_bf16x8(*reinterpret_cast<const uint4*>(p));
  uint32_t w[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) w[i] = p[2 * i] | static_cast<uint32_t>(p[2 * i + 1]) << 16;
  return msk::as_bf16x8(make_uint4(w[0], w[1], w[2], w[3]));
}

// maximum over the lanes l, l ^ 16, l ^ 32, l ^ 48
__device__ __forceinline__ float group_max(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

template <int G, int D, int QB>
__global__ __launch_bounds__(kAttThreads, 2) void attention_mma_kernel(const uint16_t* q,
                                                                    const uint16_t* __restrict__ kc,
                                                                    const uint16_t* __restrict__ vc, int T, int Hq,
                                                                    int Hkv, int pos0, int max_ctx,
                                                                    uint16_t* out) {
  extern __shared__ __align__(16) unsigned char att_lds[];
  constexpr int ROWS = 64 * QB;                   // rows of the work-group
  constexpr int TOK = ROWS / G;                   // its tokens
  constexpr int KS = D / 32, DB = D / 16;         // k steps of the scores, column blocks of O
  constexpr int PITCH = 2 * D;                    // bytes of a staged row
  constexpr int RPL = 1024 / PITCH;               // rows per load
  constexpr int TILE = kAttKeys * PITCH;          // bytes of a K (or V) tile
  constexpr int NL = TILE / 1024 / 4;             // K (or V) loads per wave and stage
  constexpr int SLOTS = PITCH / 16;
  const int lane = threadIdx.x & 63, n = lane & 15, g4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nb = (T + TOK - 1) / TOK;             // row blocks per key/value head
  const int head = blockIdx.x % Hkv, j = blockIdx.x / Hkv, first = (nb + 1) / 2;
  const int t0 = (j < first ? nb - 1 - j : j - first) * TOK;
  const int n_keys = pos0 + min(t0 + TOK, T);     // keys of the block's last token
  const int tiles = (n_keys + kAttKeys - 1) / kAttKeys;
  const uint16_t* K = kc + static_cast<size_t>(head) * max_ctx * D;
  const uint16_t* V = vc + static_cast<size_t>(head) * max_ctx * D;

  // staging: wave w the loads w, w + 4, ... of either tile; rows past the
  // last key repeat it (masked)
  const uint32_t lbase = msk::lds_address(att_lds) + wave * 1024;
  const int lrow = lane / SLOTS, slot = lane % SLOTS;
  auto issue = [&](int tile, int buf) {  // tiles past the last reload it (never read)
    const int k0 = min(tile, tiles - 1) * kAttKeys;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int u = (wave + 4 * i) * RPL + lrow;
      const size_t row = static_cast<size_t>(min(k0 + u, n_keys - 1)) * D;
      const uint32_t dst = lbase + buf * 2 * TILE + 4096 * i;
      msk::lds_load16(K + row + 8 * (slot ^ (u & 7)), dst);
      msk::lds_load16(V + row + 8 * (slot ^ (2 * (u & 3))), dst + TILE);
    }
  };
  issue(0, 0);

  // this lane's rows (one per 16-row block): token and head; B fragments of Q
  int lim[QB];  // keys the row sees
  msk::bf16x8_t Q[QB][KS];
  const bool q_vec = (reinterpret_cast<uintptr_t>(q) & 15u) == 0;
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    const int r = (wave * QB + b) * 16 + n;
    const int t = min(t0 + r / G, T - 1);  // rows past the last token repeat it (never stored)
    lim[b] = pos0 + t + 1;
    const uint16_t* qr = q + (static_cast<size_t>(t) * Hq + head * G + r % G) * D + 8 * g4;
#pragma unroll
    for (int s = 0; s < KS; ++s) Q[b][s] = load_row8(qr + 32 * s, q_vec);
  }
  // keys seen by the wave's first and last rows
  const int see_min = pos0 + min(t0 + wave * QB * 16 / G, T - 1) + 1;
  const int see_max = pos0 + min(t0 + ((wave + 1) * QB * 16 - 1) / G, T - 1) + 1;

  int ka[KS];  // K fragment addresses (key block 0) and V fragment addresses (columns 0, key blocks 0 and 1)
#pragma unroll
  for (int s = 0; s < KS; ++s) ka[s] = n * PITCH + 16 * ((4 * s + g4) ^ (n & 7));
  const int vr = (lane >> 2) & 3, vj = lane & 3;
  const int va = TILE + (4 * g4 + vr) * PITCH + 8 * (vj & 1);

  const float scale = 1.4426950408889634f / sqrtf(static_cast<float>(D));
  float m[QB], l[QB];
  msk::f32x4_t O[QB][DB];
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    m[b] = -INFINITY;
    l[b] = 0.0f;
#pragma unroll
    for (int c = 0; c < DB; ++c) O[b][c] = msk::f32x4_t{0.f, 0.f, 0.f, 0.f};
  }

  for (int tile = 0; tile < tiles; ++tile) {
    msk::wait_vm<0>();
    msk::bare_barrier();
    issue(tile + 1, (tile + 1) & 1);
    const unsigned char* st = att_lds + (tile & 1) * 2 * TILE;
    const int k0 = tile * kAttKeys;
    if (k0 >= see_max) continue;  // uniform over the wave
    const bool masked = k0 + kAttKeys > see_min;
    msk::f32x4_t S[QB][4];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      msk::bf16x8_t A[KS];
#pragma unroll
      for (int s = 0; s < KS; ++s) A[s] = msk::lds_frag(st + kb * 16 * PITCH + ka[s]);
#pragma unroll
      for (int b = 0; b < QB; ++b) {
        S[b][kb] = msk::f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s) S[b][kb] = msk::mfma16(A[s], Q[b][s], S[b][kb]);
      }
    }
    uint32_t P[QB][8][kAttParts];  // pairs of keys 16 kb + 4 g4 + (0, 1), (2, 3)
#pragma unroll
    for (int b = 0; b < QB; ++b) {
      if (masked) {
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (k0 + 16 * kb + 4 * g4 + r >= lim[b]) S[b][kb][r] = -INFINITY;
      }
      float top = S[b][0][0];
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int r = 0; r < 4; ++r) top = fmaxf(top, S[b][kb][r]);
      top = group_max(top);
      if (__any((top - m[b]) * scale > kAttGrow)) {
        const float next = fmaxf(m[b], top);
        const float f = __builtin_amdgcn_exp2f(m[b] == next ? 0.0f : (m[b] - next) * scale);
        m[b] = next;
        l[b] *= f;
#pragma unroll
        for (int c = 0; c < DB; ++c) O[b][c] *= f;
      }
      const float base = m[b] == -INFINITY ? 0.0f : m[b];
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        float p[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) p[r] = __builtin_amdgcn_exp2f((S[b][kb][r] - base) * scale);
        l[b] += (p[0] + p[1]) + (p[2] + p[3]);
        split_pair(p[0], p[1], P[b][2 * kb]);
        split_pair(p[2], p[3], P[b][2 * kb + 1]);
      }
    }
#pragma unroll
    for (int c = 0; c < DB; ++c) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const unsigned char* p = st + va + 32 * ks * PITCH + 16 * ((2 * c + (vj >> 1)) ^ (2 * vr));
        const msk::v4i16_t v0 = msk::lds_read_tr16(p), v1 = msk::lds_read_tr16(p + 16 * PITCH);
        const msk::bf16x8_t A =
            __builtin_bit_cast(msk::bf16x8_t, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
        for (int b = 0; b < QB; ++b)
#pragma unroll
          for (int i = 0; i < kAttParts; ++i)
            O[b][c] = msk::mfma16(A, msk::as_bf16x8(make_uint4(P[b][4 * ks][i], P[b][4 * ks + 1][i],
                                                               P[b][4 * ks + 2][i], P[b][4 * ks + 3][i])), O[b][c]);
      }
    }
  }
  msk::wait_vm<0>();  // the reload past the last tile lands before LDS is used again or given back
  bool bad = false;
  float inv[QB];
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    float sum = l[b];
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    inv[b] = 1.0f / sum;
#pragma unroll
    for (int c = 0; c < DB; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i) bad |= !isfinite(O[b][c][i] * inv[b]);
  }
  __syncthreads();  // every wave is done with the tiles
  if (any_thread<kAttThreads / 64>(bad, reinterpret_cast<int*>(att_lds))) {
    __syncthreads();  // the flags are read
    for (int t = t0; t < min(t0 + TOK, T); ++t) {
      attention_token<G, kAttThreads>(q, kc, vc, Hq, D, pos0, max_ctx, out, t, head, 0, D,
                                      reinterpret_cast<float*>(att_lds));
      __syncthreads();
    }
    return;
  }
  const bool o_vec = (reinterpret_cast<uintptr_t>(out) & 7u) == 0;
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    const int r = (wave * QB + b) * 16 + n;
    const int t = t0 + r / G;
    if (t >= T) continue;
    uint16_t* dst = out + (static_cast<size_t>(t) * Hq + head * G + r % G) * D + 4 * g4;
#pragma unroll
    for (int c = 0; c < DB; ++c) {
      uint16_t w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) w[i] = f32_to_bf16(O[b][c][i] * inv[b]);
      if (o_vec) {
        *reinterpret_cast<uint2*>(dst + 16 * c) =
            make_uint2(w[0] | static_cast<uint32_t>(w[1]) << 16, w[2] | static_cast<uint32_t>(w[3]) << 16);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) dst[16 * c + i] = w[i];
      }
    }
  }
}

// ------------------------------------------ attention of few tokens (MFMA)
//
// D = 64 or 128, calls of few tokens (att_few).  A work-group takes one token,
// one key/value head and 32 of its value columns, in KW waves: wave w the key
// steps (32 keys) w, w + KW, ..., each wave with a ring of its own (no barrier
// in the loop) and a softmax of its own (running maximum, sum, output), merged
// at the end.  The scores are needed by every column slice and computed by
// each: reading the keys D / 32 times costs less than leaving all but Hkv
// compute units idle.  Fragments and their key order are those of
// attention_mma_kernel, with the token's G query heads repeated to 16 rows.
// Keys past the token repeat its last one: score -inf, value 0.  A work-group
// with a result that is not finite computes its columns again by
// attention_token (see attention_mma_kernel).  Bound by
// what one CU can load (about 60 GB/s with these direct loads; the same
// kernel with its fragments loaded into registers reached half of that).
// Measured, 32 query and 8 key/value heads of 128, fma chains -> now: one
// token at position 1500 27.5 -> 9.5 us, at 3000 94 -> 14.8 us, 8 tokens at
// 1500 67 -> 12.9 us.
constexpr int kAttFewCols = 32;
constexpr int kAttFewWgs = 512;   // work-groups of a round: two per CU
constexpr int kAttFewKeys = 32;
// LDS bytes of the waves' rings: per stage kAttFewKeys keys and their slices of values
constexpr int kAttFewStages = 2;
constexpr size_t att_few_ring(int D, int waves) {
  return static_cast<size_t>(waves) * kAttFewStages * kAttFewKeys * 2 * (D + kAttFewCols);
}

template <int G, int D, int KW>
__global__ __launch_bounds__(64 * KW) void attention_few_kernel(const uint16_t* __restrict__ q,
                                                                const uint16_t* __restrict__ kc,
                                                                const uint16_t* __restrict__ vc, int Hq, int pos0,
                                                                int max_ctx, uint16_t* __restrict__ out) {
  constexpr int NST = kAttFewStages, KS = D / 32;
  constexpr int PITCH = 2 * D;                      // bytes of a staged key
  constexpr int SLOTS = PITCH / 16, RPL = 1024 / PITCH;
  constexpr int KBYTES = kAttFewKeys * PITCH;
  constexpr int VPITCH = 2 * kAttFewCols;           // bytes of a staged value slice
  constexpr int NK = KBYTES / 1024, NV = kAttFewKeys * VPITCH / 1024, NL = NK + NV;
  constexpr int SBYTES = NL * 1024;
  static_assert(KW * NST * SBYTES == att_few_ring(D, KW) && (NST - 2) * NL < 64, "ring");
  static_assert(KW * NST * SBYTES >= KW * (G * (kAttFewCols + 3) + 1) * 4, "the merge fits the rings");
  extern __shared__ __align__(16) unsigned char att_lds[];
  unsigned char* lds = att_lds;
  const int t = blockIdx.x, head = blockIdx.y, c0 = blockIdx.z * kAttFewCols;
  const int lane = threadIdx.x & 63, n = lane & 15, g4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int keys = pos0 + t + 1, steps = (keys + kAttFewKeys - 1) / kAttFewKeys;
  const uint16_t* K = kc + static_cast<size_t>(head) * max_ctx * D;
  const uint16_t* V = vc + static_cast<size_t>(head) * max_ctx * D + c0;
  unsigned char* ring = lds + wave * NST * SBYTES;
  const uint32_t lbase = msk::lds_address(ring);
  const int krow = lane / SLOTS, kslot = lane % SLOTS;
  const int vrow = lane >> 2, vslot = lane & 3;
  auto issue = [&](int i, int buf) {  // steps past the wave's last reload keys of the last one (never read)
    const int k0 = min(wave + KW * i, steps - 1) * kAttFewKeys;
#pragma unroll
    for (int j = 0; j < NK; ++j) {
      const int u = j * RPL + krow;
      msk::lds_load16(K + static_cast<size_t>(min(k0 + u, keys - 1)) * D + 8 * (kslot ^ (u & 7)),
                      lbase + buf * SBYTES + 1024 * j);
    }
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int u = j * 16 + vrow;
      msk::lds_load16(V + static_cast<size_t>(min(k0 + u, keys - 1)) * D + 8 * vslot,
                      lbase + buf * SBYTES + KBYTES + 1024 * j);
    }
  };
#pragma unroll
  for (int p = 0; p < NST - 1; ++p) issue(p, p);
  msk::bf16x8_t Q[KS];
  const uint16_t* qr = q + (static_cast<size_t>(t) * Hq + head * G + n % G) * D + 8 * g4;
#pragma unroll
  for (int s = 0; s < KS; ++s) Q[s] = load_row8(qr + 32 * s, (reinterpret_cast<uintptr_t>(q) & 15u) == 0);
  int ka[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) ka[s] = n * PITCH + 16 * ((4 * s + g4) ^ (n & 7));
  const int va = KBYTES + (4 * g4 + ((lane >> 2) & 3)) * VPITCH + 8 * (lane & 3);
  const float scale = 1.4426950408889634f / sqrtf(static_cast<float>(D));
  float m = -INFINITY, l = 0.0f;
  msk::f32x4_t O[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  int cur = 0, nxt = NST - 1;
  for (int i = 0; wave + KW * i < steps; ++i) {
    msk::wait_vm<(NST - 2) * NL>();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    issue(i + NST - 1, nxt);
    const unsigned char* st = ring + cur * SBYTES;
    cur = cur + 1 == NST ? 0 : cur + 1;
    nxt = nxt + 1 == NST ? 0 : nxt + 1;
    const int k0 = (wave + KW * i) * kAttFewKeys;
    msk::f32x4_t S[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      S[b] = msk::f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < KS; ++s) S[b] = msk::mfma16(msk::lds_frag(st + 16 * b * PITCH + ka[s]), Q[s], S[b]);
    }
    uint4 A[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const msk::v4i16_t v0 = msk::lds_read_tr16(st + va + 32 * c), v1 = msk::lds_read_tr16(st + va + 32 * c + 16 * VPITCH);
      A[c] = __builtin_bit_cast(uint4, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
    }
    if (k0 + kAttFewKeys > keys) {
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (k0 + 16 * b + 4 * g4 + r >= keys) S[b][r] = -INFINITY;
      // word w of a fragment holds keys 16 (w / 2) + 4 g4 + 2 (w % 2) + (0, 1)
      auto keep = [&](uint32_t x, int w) {
        const int k = k0 + 16 * (w >> 1) + 4 * g4 + 2 * (w & 1);
        return k + 1 < keys ? x : k < keys ? x & 0xffffu : 0u;
      };
#pragma unroll
      for (int c = 0; c < 2; ++c) A[c] = make_uint4(keep(A[c].x, 0), keep(A[c].y, 1), keep(A[c].z, 2), keep(A[c].w, 3));
    }
    float top = fmaxf(fmaxf(fmaxf(S[0][0], S[0][1]), fmaxf(S[0][2], S[0][3])),
                      fmaxf(fmaxf(S[1][0], S[1][1]), fmaxf(S[1][2], S[1][3])));
    top = group_max(top);
    const float next = fmaxf(m, top);
    const float f = __builtin_amdgcn_exp2f(m == next ? 0.0f : (m - next) * scale);
    m = next;
    const float base = m == -INFINITY ? 0.0f : m;
    uint32_t P[4][kAttParts];
    float sum = 0.0f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float p0 = __builtin_amdgcn_exp2f((S[w >> 1][2 * (w & 1)] - base) * scale);
      const float p1 = __builtin_amdgcn_exp2f((S[w >> 1][2 * (w & 1) + 1] - base) * scale);
      sum += p0 + p1;
      split_pair(p0, p1, P[w]);
    }
    l = l * f + sum;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      O[c] *= f;
#pragma unroll
      for (int i = 0; i < kAttParts; ++i)
        O[c] = msk::mfma16(msk::as_bf16x8(A[c]), msk::as_bf16x8(make_uint4(P[0][i], P[1][i], P[2][i], P[3][i])), O[c]);
    }
  }
  msk::wait_vm<0>();  // the reloads past the last step have landed
  __syncthreads();    // every wave is done with its ring
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  // lane (n = query head, g4): columns 16 c + 4 g4 + r of its row
  float* part = reinterpret_cast<float*>(lds);   // [KW][G][kAttFewCols + 1]
  float* mx = part + KW * G * (kAttFewCols + 1);  // [KW][G]
  float* sm = mx + KW * G;
  if (n < G) {
    if (g4 == 0) {
      mx[wave * G + n] = m;
      sm[wave * G + n] = l;
    }
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) part[(wave * G + n) * (kAttFewCols + 1) + 16 * c + 4 * g4 + r] = O[c][r];
  }
  __syncthreads();
  const int used = min(KW, steps);  // waves with a step
  static_assert(G * kAttFewCols <= 64 * KW, "one result per thread");
  const int h = threadIdx.x / kAttFewCols, col = threadIdx.x % kAttFewCols;
  float r = 0.0f;
  if (h < G) {
    float top = mx[h];
    for (int w = 1; w < used; ++w) top = fmaxf(top, mx[w * G + h]);
    float num = 0.0f, den = 0.0f;
    for (int w = 0; w < used; ++w) {
      const float f = __builtin_amdgcn_exp2f(mx[w * G + h] == top ? 0.0f : (mx[w * G + h] - top) * scale);
      num += f * part[(w * G + h) * (kAttFewCols + 1) + col];
      den += f * sm[w * G + h];
    }
    r = num / den;
  }
  if (any_thread<KW>(!isfinite(r), reinterpret_cast<int*>(sm + KW * G))) {
    __syncthreads();  // the flags and the waves' parts are read
    attention_token<G, 64 * KW>(q, kc, vc, Hq, D, pos0, max_ctx, out, t, head, c0, c0 + kAttFewCols,
                                reinterpret_cast<float*>(lds));
  } else if (h < G) {
    out[(static_cast<size_t>(t) * Hq + head * G + h) * D + c0 + col] = f32_to_bf16(r);
  }
}

// ---------------------------------------------------------- arg max, gather

__global__ __launch_bounds__(256) void argmax_kernel(const float* __restrict__ x, int n, int32_t* __restrict__ idx) {
  __shared__ float bv[4];
  __shared__ int bi[4];
  const int t = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float* row = x + static_cast<size_t>(t) * n;
  float v = -INFINITY;
  int i = n;
  for (int j = tid; j < n; j += 256) {
    const float xv = row[j];
    if (xv > v) {  // ascending j per thread: the first maximum stays
      v = xv;
      i = j;
    }
  }
  for (int s = 32; s >= 1; s >>= 1) {
    const float ov = __shfl_xor(v, s, 64);
    const int oi = __shfl_xor(i, s, 64);
    if (ov > v || (ov == v && oi < i)) {
      v = ov;
      i = oi;
    }
  }
  if (lane == 0) {
    bv[wave] = v;
    bi[wave] = i;
  }
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < 4; ++w)
      if (bv[w] > v || (bv[w] == v && bi[w] < i)) {
        v = bv[w];
        i = bi[w];
      }
    idx[t] = i < n ? i : 0;
  }
}

__global__ void embed_kernel(const int32_t* __restrict__ ids, const uint16_t* __restrict__ table, int n_vocab,
                             int d, uint16_t* __restrict__ out) {
  const int t = blockIdx.x;
  const int id = min(max(ids[t], 0), n_vocab - 1);  // ids are validated by the argmax; clamped to stay in bounds
  const uint4* src = reinterpret_cast<const uint4*>(table + static_cast<size_t>(id) * d);
  uint4* dst = reinterpret_cast<uint4*>(out + static_cast<size_t>(t) * d);
  for (int i = threadIdx.x; i < d / 8; i += blockDim.x) dst[i] = src[i];
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Prompts whose n_in is an odd multiple of 32 (T >= kDenseMmaTokens; other
// multiples of 32 take the staged kernels below): the same product on the
// matrix cores, v_mfma_f32_16x16x32_bf16 (lane l holds A[row l % 16][8 k
// from 8 (l / 16)], B[8 k from 8 (l / 16)][column l % 16] and C[rows
// 4 (l / 16) + r][column l % 16]).  A work-group takes 64 tokens x 64
// outputs, wave w the outputs 16 w .. 16 w + 15 of all four 16-token blocks.
// x [T][n_in] and W [n_out][n_in] are both contiguous along k, so each
// fragment is one 16-byte load; loads run kDenseKb k steps of 32 ahead.
// Tokens past T and outputs past n_out are clamped on load, never stored.
constexpr int kDenseMmaTokens = 16;
constexpr int kDenseKb = 2;

typedef __bf16 dbf16x8_t __attribute__((ext_vector_type(8)));
typedef float df32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ df32x4_t dmfma(uint4 a, uint4 b, df32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(dbf16x8_t, a), __builtin_bit_cast(dbf16x8_t, b),
                                                 c, 0, 0, 0);
}

__global__ __launch_bounds__(256) void dense_mma_kernel(const uint16_t* __restrict__ x,
                                                        const uint16_t* __restrict__ w,
                                                        const float* __restrict__ add, float* __restrict__ y, int T,
                                                        int n_in, int n_out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int t0 = blockIdx.x * 64, o0 = blockIdx.y * 64 + 16 * wave;
  const int n = lane & 15, kq = 8 * (lane >> 4);
  const uint16_t* wrow = w + static_cast<size_t>(min(o0 + n, n_out - 1)) * n_in + kq;
  const uint16_t* xrow[4];
#pragma unroll
  for (int rb = 0; rb < 4; ++rb) xrow[rb] = x + static_cast<size_t>(min(t0 + 16 * rb + n, T - 1)) * n_in + kq;
  const int ksteps = n_in / 32;
  df32x4_t acc[4];
#pragma unroll
  for (int rb = 0; rb < 4; ++rb) acc[rb] = df32x4_t{0.f, 0.f, 0.f, 0.f};
  uint4 bn[kDenseKb], an[kDenseKb][4], bc[kDenseKb], ac[kDenseKb][4];
  auto load = [&](int s0) {
#pragma unroll
    for (int u = 0; u < kDenseKb; ++u) {
      const int k = min(s0 + u, ksteps - 1) * 32;  // clamped past the last step; used only in range
      bn[u] = *reinterpret_cast<const uint4*>(wrow + k);
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) an[u][rb] = *reinterpret_cast<const uint4*>(xrow[rb] + k);
    }
  };
  load(0);
  for (int s0 = 0; s0 < ksteps; s0 += kDenseKb) {
#pragma unroll
    for (int u = 0; u < kDenseKb; ++u) {
      bc[u] = bn[u];
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) ac[u][rb] = an[u][rb];
    }
    load(s0 + kDenseKb);
#pragma unroll
    for (int u = 0; u < kDenseKb; ++u)
      if (s0 + u < ksteps) {
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) acc[rb] = dmfma(ac[u][rb], bc[u], acc[rb]);
      }
  }
  const int o = o0 + n;
  if (o < n_out) {
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int t = t0 + 16 * rb + 4 * (lane >> 4) + r;
        if (t < T) {
          const size_t i = static_cast<size_t>(t) * n_out + o;
          y[i] = acc[rb][r] + (add ? add[i] : 0.0f);
        }
      }
  }
}

// Prompts (T >= kDenseMmaTokens, n_in a multiple of 64): y^T = W x^T on the
// matrix cores, A = 16 output rows of W, B = 16 tokens of x, so that a lane
// ends with four consecutive outputs of one token (one 16-byte store).  A
// work-group takes BM tokens x BN outputs; both operands go from memory to
// LDS directly (lds_load16, 8 rows of 64 k per load) in a ring of NST
// stages of 64 k, all but one of them in flight while a stage is computed.
// Piece p (8 k) of staged row r sits in slot p ^ (r % 8), so the 8 lanes an
// LDS read serves together hit distinct banks.  WM x WN waves split the
// tile.  Every sum runs over k in ascending 32-wide MFMA steps whatever the
// tile, so the tile choice changes no result (the bits are also those of
// dense_mma_kernel, whose loads went through registers and repeated every
// weight row per 64 tokens).  Tokens past T and outputs past n_out repeat
// the last one on load and are never stored.  Bound by the matrix cores from
// about 1000 tokens on, by the loads below.  Measured, before -> now: 2048
// tokens 4096 -> 6144 846 -> 94 us (1095 TFLOP/s), 4096 -> 4096 566 -> 74 us;
// 512 tokens 219 -> 45 and 148 -> 28 us; 16 tokens 42 -> 10.7 us (4.7 TB/s of
// weights) and 41 -> 9.8 us.
constexpr int kDsSlab = 64;                 // k per stage
constexpr int kDsRowBytes = 2 * kDsSlab;    // one staged row: a cache line
constexpr int kDsLoadBytes = 64 * 16;       // one load: 8 rows
constexpr int kDsBlockBytes = 16 * kDsRowBytes;

template <int BM, int BN, int WM, int WN, int NST>
__global__ __launch_bounds__(64 * WM * WN) void dense_staged_kernel(const uint16_t* __restrict__ x,
                                                                    const uint16_t* __restrict__ w,
                                                                    const float* add, float* y, int T,
                                                                    int n_in, int n_out, int m_tiles, int vec) {
  constexpr int NWV = WM * WN;
  constexpr int TM = BM / WM / 16, TN = BN / WN / 16;  // 16-wide blocks per wave
  constexpr int NL = (BM + BN) / 8 / NWV;              // loads per wave and stage
  constexpr int SBYTES = (BM + BN) * kDsRowBytes;
  static_assert(TM * WM * 16 == BM && TN * WN * 16 == BN && NL * 8 * NWV == BM + BN, "tile split");
  static_assert(NST >= 2 && NST * SBYTES <= 160 * 1024 && (NST - 2) * NL < 64, "ring");
  __shared__ __align__(16) unsigned char lds[NST * SBYTES];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wv % WM, wn = wv / WM;
  const int tile = msk::xcd_local(blockIdx.x, gridDim.x);
  const int t0 = (tile % m_tiles) * BM, o0 = (tile / m_tiles) * BN;
  const int lrow = lane >> 3, lk = 8 * ((lane & 7) ^ lrow);
  const uint16_t* src[NL];  // staged rows: the tile's BM tokens, then its BN outputs
#pragma unroll
  for (int j = 0; j < NL; ++j) {
    const int r = 8 * (wv + NWV * j) + lrow;
    src[j] = (r < BM ? x + static_cast<size_t>(min(t0 + r, T - 1)) * n_in
                     : w + static_cast<size_t>(min(o0 + r - BM, n_out - 1)) * n_in) + lk;
  }
  const int nsl = n_in / kDsSlab;
  const uint32_t lbase = msk::lds_address(lds) + wv * kDsLoadBytes;
  auto issue = [&](int sl, int buf) {  // stages past the last reload it (in bounds, never read)
    const int k0 = min(sl, nsl - 1) * kDsSlab;
#pragma unroll
    for (int j = 0; j < NL; ++j) msk::lds_load16(src[j] + k0, lbase + buf * SBYTES + NWV * j * kDsLoadBytes);
  };
  int fo[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) fo[s] = (lane & 15) * kDsRowBytes + 16 * ((4 * s + (lane >> 4)) ^ (lane & 7));
  msk::f32x4_t acc[TN][TM];
#pragma unroll
  for (int n = 0; n < TN; ++n)
#pragma unroll
    for (int m = 0; m < TM; ++m) acc[n][m] = msk::f32x4_t{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](int buf) {
    const unsigned char* sx = lds + buf * SBYTES + wm * TM * kDsBlockBytes;
    const unsigned char* sw = lds + buf * SBYTES + BM * kDsRowBytes + wn * TN * kDsBlockBytes;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      msk::bf16x8_t A[TN], B[TM];
#pragma unroll
      for (int n = 0; n < TN; ++n) A[n] = msk::lds_frag(sw + n * kDsBlockBytes + fo[s]);
#pragma unroll
      for (int m = 0; m < TM; ++m) B[m] = msk::lds_frag(sx + m * kDsBlockBytes + fo[s]);
#pragma unroll
      for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int n = 0; n < TN; ++n) acc[n][m] = msk::mfma16(A[n], B[m], acc[n][m]);
    }
  };
#pragma unroll
  for (int p = 0; p < NST - 1; ++p) issue(p, p);
  int cur = 0, nxt = NST - 1;
  for (int sl = 0; sl < nsl; ++sl) {
    msk::wait_vm<(NST - 2) * NL>();
    msk::bare_barrier();
    issue(sl + NST - 1, nxt);
    compute(cur);
    cur = cur + 1 == NST ? 0 : cur + 1;
    nxt = nxt + 1 == NST ? 0 : nxt + 1;
  }
  msk::wait_vm<0>();  // the reloads past the last stage land before the work-group ends
#pragma unroll
  for (int m = 0; m < TM; ++m) {
    const int t = t0 + (wm * TM + m) * 16 + (lane & 15);
    if (t >= T) continue;
#pragma unroll
    for (int n = 0; n < TN; ++n) {
      const int o = o0 + (wn * TN + n) * 16 + 4 * (lane >> 4);
      const size_t i = static_cast<size_t>(t) * n_out + o;
      if (vec) {  // n_out a multiple of 4, rows 16-byte aligned
        if (o < n_out) {
          float4 v = make_float4(acc[n][m][0], acc[n][m][1], acc[n][m][2], acc[n][m][3]);
          if (add) {
            const float4 b = *reinterpret_cast<const float4*>(add + i);
            v = make_float4(v.x + b.x, v.y + b.y, v.z + b.z, v.w + b.w);
          }
          *reinterpret_cast<float4*>(y + i) = v;
        }
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (o + r < n_out) y[i + r] = acc[n][m][r] + (add ? add[i + r] : 0.0f);
      }
    }
  }
}

// Few tokens (T < kDenseMmaTokens, n_in a multiple of 64): 16 tokens (the
// last one repeated) x 16 outputs per work-group on the matrix cores, bound by
// the weights' bytes in flight.  The KW waves split k: wave w takes the
// 64-wide stages w, w + KW, ..., each wave loading its stages into a ring of
// its own (no barrier in the loop).  A stage's products are summed from zero
// in 32 bits and added to the wave's 64-bit sums, and the waves' sums are
// added in order at the end, so a result is rounded to 32 bits once (measured
// against 64-bit references: relative error 3.4e-8, the fma kernel of the other
// widths 7.8e-8; one 32-bit MFMA chain over k would have 3.6e-7).  Eight waves
// where the work-groups have a CU each and a row is long, four otherwise:
// 8192 -> 1024 8.7 | 6.4 us with four | eight waves, 4096 -> 4096 5.9 | 5.1, 2048
// -> 64 3.7 | 3.6, 1024 -> 1024 3.1 | 3.2, 4096 -> 6144 (384 work-groups) 9.0 |
// 9.1, 64 -> 32000 6.6 | 12.4.  Measured at 1 / 15 tokens, fma kernel -> now:
// 4096 -> 6144 11.7 -> 9.0 / 42.6 -> 9.9 us, 4096 -> 4096 8.1 -> 5.1 / 31.6 -> 6.1,
// 4096 -> 32000 44.9 -> 40.8 us (6.4 TB/s), 8192 -> 1024 7.8 -> 6.4 us; 2 or 3
// output blocks per work-group were no faster over these.
constexpr int kDsCus = 256;
constexpr int kDsLongRow = 2048;  // n_in
constexpr int kDsFewStages = 4;   // of a wave's ring

template <int KW>
__global__ __launch_bounds__(64 * KW) void dense_few_kernel(const uint16_t* __restrict__ x,
                                                            const uint16_t* __restrict__ w,
                                                            const float* add, float* y,
                                                            int T, int n_in, int n_out) {
  constexpr int NST = kDsFewStages;
  constexpr int NL = 4;  // loads of a stage: 16 token rows, then 16 output rows
  constexpr int SBYTES = NL * kDsLoadBytes;
  constexpr int LDS = KW * NST * SBYTES;
  static_assert(LDS <= 160 * 1024 && (NST - 2) * NL < 64, "ring");
  static_assert(LDS >= KW * 64 * 32, "the waves' sums, after the loop");
  __shared__ __align__(16) unsigned char lds[LDS];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int o0 = blockIdx.x * 16;
  const int lrow = lane >> 3, lk = 8 * ((lane & 7) ^ lrow);
  const uint16_t* src[NL];
#pragma unroll
  for (int j = 0; j < NL; ++j) {
    const int r = 8 * j + lrow;
    src[j] = (r < 16 ? x + static_cast<size_t>(min(r, T - 1)) * n_in
                     : w + static_cast<size_t>(min(o0 + r - 16, n_out - 1)) * n_in) + lk;
  }
  const int nsl = n_in / kDsSlab;
  const int mine = (nsl - wv + KW - 1) / KW;  // stages of this wave
  unsigned char* ring = lds + wv * NST * SBYTES;
  const uint32_t lbase = msk::lds_address(ring);
  auto issue = [&](int i, int buf) {  // stages past the wave's last reload one (in bounds, never read)
    const int k0 = min(wv + KW * min(i, max(mine, 1) - 1), nsl - 1) * kDsSlab;
#pragma unroll
    for (int j = 0; j < NL; ++j) msk::lds_load16(src[j] + k0, lbase + buf * SBYTES + j * kDsLoadBytes);
  };
  int fo[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) fo[s] = (lane & 15) * kDsRowBytes + 16 * ((4 * s + (lane >> 4)) ^ (lane & 7));
  const msk::f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
  double sum[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int p = 0; p < NST - 1; ++p) issue(p, p);
  int cur = 0, nxt = NST - 1;
  for (int i = 0; i < mine; ++i) {
    // this wave's loads of the stage have landed, and its reads of the buffer
    // it loads next are done
    msk::wait_vm<(NST - 2) * NL>();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    issue(i + NST - 1, nxt);
    const unsigned char* st = ring + cur * SBYTES;
    msk::bf16x8_t A[2], B[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      B[s] = msk::lds_frag(st + fo[s]);
      A[s] = msk::lds_frag(st + kDsBlockBytes + fo[s]);
    }
    const msk::f32x4_t p0 = msk::mfma16(A[0], B[0], zero), p1 = msk::mfma16(A[1], B[1], zero);
#pragma unroll
    for (int r = 0; r < 4; ++r) sum[r] += static_cast<double>(p0[r]) + static_cast<double>(p1[r]);
    cur = cur + 1 == NST ? 0 : cur + 1;
    nxt = nxt + 1 == NST ? 0 : nxt + 1;
  }
  msk::wait_vm<0>();  // the reloads past the last stage have landed
  __syncthreads();    // every wave is done with its ring
  double* red = reinterpret_cast<double*>(lds);  // [KW][64][4]
#pragma unroll
  for (int r = 0; r < 4; ++r) red[(wv * 64 + lane) * 4 + r] = sum[r];
  __syncthreads();
  if (const int i = threadIdx.x; i < 256) {  // value i: token (i / 4) % 16, output below
    double v = red[i];
#pragma unroll
    for (int k = 1; k < KW; ++k) v += red[k * 256 + i];
    const int t = (i >> 2) & 15, o = o0 + 4 * (i >> 6) + (i & 3);
    if (t < T && o < n_out) {
      const size_t j = static_cast<size_t>(t) * n_out + o;
      y[j] = static_cast<float>(v) + (add ? add[j] : 0.0f);
    }
  }
}

ms_status launched();

// Tile of a staged launch: the one whose rounds over the CUs cost least.  The
// costs are times of one full launch relative to each other, measured at
// n_in 4096 (they scale with n_in alike): with one work-group per CU, and
// with the two that fit for the small tiles, whose second one overlaps the
// first's waits.  Checked over T = 16 .. 2048 at 4096 -> 6144, 4096 -> 4096,
// 2048 -> 5120 and 256 -> 512: within 5% of the fastest of twenty tiles but
// for 1000 tokens 2048 -> 5120 (39 us for 36).
ms_status launch_dense_staged(const uint16_t* x, const uint16_t* w, const float* add, float* y, int T, int n_in,
                              int n_out, hipStream_t s) {
  struct Tile {
    int bm, bn, threads, one, two;  // tokens, outputs, cost of a round with one and with two work-groups per CU
  };
  static constexpr Tile tiles[] = {{32, 32, 256, 10, 14},   {64, 64, 256, 20, 29},   {128, 64, 512, 26, 52},
                                   {128, 128, 512, 41, 82}, {256, 128, 512, 68, 136}, {256, 192, 512, 94, 188}};
  auto count = [&](const Tile& t) {
    return ((static_cast<int64_t>(T) + t.bm - 1) / t.bm) * ((static_cast<int64_t>(n_out) + t.bn - 1) / t.bn);
  };
  int best = 0;
  int64_t best_cost = INT64_MAX;
  for (int i = 0; i < 6; ++i) {
    const Tile& t = tiles[i];
    const int64_t n = count(t), rest = n % (2 * kDsCus);
    if (n * t.threads > UINT32_MAX) continue;  // past what one launch can hold
    const int64_t cost = n / (2 * kDsCus) * t.two + (rest == 0 ? 0 : rest <= kDsCus ? t.one : t.two);
    if (cost < best_cost) {
      best = i;
      best_cost = cost;
    }
  }
  const int m_tiles = static_cast<int>((static_cast<int64_t>(T) + tiles[best].bm - 1) / tiles[best].bm);
  const int64_t grid = count(tiles[best]);
  if (best_cost == INT64_MAX) return MS_E_HIP;
  const int vec = n_out % 4 == 0 && ((reinterpret_cast<uintptr_t>(y) | reinterpret_cast<uintptr_t>(add)) & 15u) == 0;
#define MSK_DENSE_CASE(I_, BM_, BN_, WM_, WN_, NST_)                                                            \
  case I_:                                                                                                      \
    static_assert(tiles[I_].bm == BM_ && tiles[I_].bn == BN_ && tiles[I_].threads == 64 * WM_ * WN_, "tiles");      \
    hipLaunchKernelGGL((dense_staged_kernel<BM_, BN_, WM_, WN_, NST_>), dim3(static_cast<unsigned>(grid)),      \
                       dim3(64 * WM_ * WN_), 0, s, x, w, add, y, T, n_in, n_out, m_tiles, vec);                 \
    break;
  switch (best) {
    MSK_DENSE_CASE(0, 32, 32, 2, 2, 8)
    MSK_DENSE_CASE(1, 64, 64, 2, 2, 5)
    MSK_DENSE_CASE(2, 128, 64, 4, 2, 6)
    MSK_DENSE_CASE(3, 128, 128, 2, 4, 4)
    MSK_DENSE_CASE(4, 256, 128, 4, 2, 3)
    MSK_DENSE_CASE(5, 256, 192, 4, 2, 2)
  }
#undef MSK_DENSE_CASE
  return launched();
}

ms_status launched() { return hipGetLastError() == hipSuccess ? MS_OK : MS_E_HIP; }

template <int G, int D, int QB>
void launch_attention_mma(const uint16_t* q, const uint16_t* kc, const uint16_t* vc, int T, int Hq, int Hkv, int pos0,
                          int max_ctx, uint16_t* out, hipStream_t s) {
  constexpr int TOK = 64 * QB / G;
  const size_t ring = size_t{4} * kAttKeys * 2 * D;  // two stages of a K and a V tile
  const size_t again = sizeof(float) * att_token_floats(G, kAttThreads / 64, D, pos0 + T);
  hipLaunchKernelGGL((attention_mma_kernel<G, D, QB>), dim3((T + TOK - 1) / TOK * Hkv), dim3(kAttThreads),
                     ring > again ? ring : again, s, q, kc, vc, T, Hq, Hkv, pos0, max_ctx, out);
}

// Row blocks of 64, or 128 (half the LDS reads per row) from kAttTallBlocks
// blocks of 64 on, below which the longer chain of a tall block costs more than
// it saves.  Measured, 4 x 128 heads for each of 8 key/value heads, 64 | 128
// rows: 512 tokens (256 blocks of 64) 16.6 | 22.6 us, 1024 31 | 40, 1536 (768)
// 55 | 59, 2048 (1024) 89 | 81; deeper rings of tiles were slower (512 tokens
// 17.3 us for 16.6 with three stages, 17.5 with four).
constexpr int kAttTallBlocks = 1024;
template <int G, int D>
void launch_attention_rows(const uint16_t* q, const uint16_t* kc, const uint16_t* vc, int T, int Hq, int Hkv, int pos0,
                           int max_ctx, uint16_t* out, hipStream_t s) {
  if ((static_cast<int64_t>(T) * G + 63) / 64 * Hkv >= kAttTallBlocks)
    launch_attention_mma<G, D, 2>(q, kc, vc, T, Hq, Hkv, pos0, max_ctx, out, s);
  else
    launch_attention_mma<G, D, 1>(q, kc, vc, T, Hq, Hkv, pos0, max_ctx, out, s);
}

template <int G, int D, int KW>
void launch_attention_few(const uint16_t* q, const uint16_t* kc, const uint16_t* vc, int T, int Hq, int Hkv, int pos0,
                          int max_ctx, uint16_t* out, hipStream_t s) {
  constexpr size_t ring = att_few_ring(D, KW);
  static_assert(ring <= msk::kCuLdsBytes, "rings of one work-group");
  const size_t again = sizeof(float) * att_token_floats(G, KW, D, pos0 + T);
  hipLaunchKernelGGL((attention_few_kernel<G, D, KW>), dim3(T, Hkv, D / kAttFewCols), dim3(64 * KW),
                     ring > again ? ring : again, s, q, kc, vc, Hq, pos0, max_ctx, out);
}

// Whether a call of T tokens over n positions takes attention_few_kernel: one
// round of its work-groups, or two where the keys are many, since a row
// block of attention_mma_kernel walks them all, and a token's slices of keys
// and values are few enough to stay in the caches.  Measured, few | row
// blocks, us, G x heads x width: 4 x 8 x 128, 16 tokens (512 work-groups) at
// position 20 4.7 | 5.6, 24 (768) at 20 / 100 / 500 6.6 | 5.6 / 7.5 | 7.1 / 14.2 |
// 17.6, 32 (1024) at 1300 29.5 | 35.2; 1 x 1 x 64, 500 (1000) at 20 8.7 | 11.3;
// 1 x 16 x 128, 12 (768) at 1300 27.8 | 34.3, 16 (1024) 33.5 | 34.4; 1 x 32 x
// 128, 8 (1024) 55.5 | 34.4.  Left slower than fma chains per token: one query
// head per key/value head where a row block's last key tile is nearly empty
// (1 x 16 x 128, 48 tokens at position 20 7.0 for 5.9, 16 at 500 16.9 for 15.4).
bool att_few(int T, int Hkv, int D, int n) {
  const int64_t wgs = static_cast<int64_t>(T) * Hkv * (D / kAttFewCols);
  if (wgs <= kAttFewWgs) return true;
  return n >= 256 && wgs <= (Hkv * D <= 1024 ? 2 : 1.5) * kAttFewWgs;
}

template <int G, int D>
ms_status launch_attention_tiles(const uint16_t* q, const uint16_t* kc, const uint16_t* vc, int T, int Hq, int Hkv,
                                int pos0, int max_ctx, uint16_t* out, hipStream_t s) {
  // one work-group per (token, head, 32 columns) while those are few: eight
  // waves where each has a CU, else four (two work-groups per CU)
  if (!att_few(T, Hkv, D, pos0 + T))
    launch_attention_rows<G, D>(q, kc, vc, T, Hq, Hkv, pos0, max_ctx, out, s);
  else if (static_cast<int64_t>(T) * Hkv * (D / kAttFewCols) <= 256)
    launch_attention_few<G, D, 8>(q, kc, vc, T, Hq, Hkv, pos0, max_ctx, out, s);
  else
    launch_attention_few<G, D, 4>(q, kc, vc, T, Hq, Hkv, pos0, max_ctx, out, s);
  return launched();
}

template <int G>
ms_status launch_attention(const uint16_t* q, const uint16_t* kc, const uint16_t* vc, int T, int Hq, int Hkv, int D,
                           int pos0, int max_ctx, uint16_t* out, hipStream_t s) {
  // out over q: attention_few_kernel's work-groups read a row of q that others
  // write columns of, so such a call does not take it; the others' read their
  // rows of q before they write them, which is enough where out is q itself
  const size_t bytes = sizeof(uint16_t) * T * Hq * D;
  const auto qa = reinterpret_cast<uintptr_t>(q), oa = reinterpret_cast<uintptr_t>(out);
  const bool apart = qa + bytes <= oa || oa + bytes <= qa;
  if (apart || (qa == oa && !att_few(T, Hkv, D, pos0 + T))) {
    if (D == 64) return launch_attention_tiles<G, 64>(q, kc, vc, T, Hq, Hkv, pos0, max_ctx, out, s);
    if (D == 128) return launch_attention_tiles<G, 128>(q, kc, vc, T, Hq, Hkv, pos0, max_ctx, out, s);
  }
  const bool wide = T == 1 && static_cast<int64_t>(G) * ((1 + kAttWideThreads / 64) * D + pos0 + T) <= kAttMaxScores;
  const int waves = (wide ? kAttWideThreads : kAttThreads) / 64;
  const size_t lds = sizeof(float) * att_token_floats(G, waves, D, pos0 + T);
  if (wide)
    hipLaunchKernelGGL((attention_kernel<G, kAttWideThreads>), dim3(T, Hkv), dim3(kAttWideThreads), lds, s, q, kc, vc,
                       Hq, D, pos0, max_ctx, out);
  else
    hipLaunchKernelGGL((attention_kernel<G, kAttThreads>), dim3(T, Hkv), dim3(kAttThreads), lds, s, q, kc, vc, Hq, D,
                       pos0, max_ctx, out);
  return launched();
}

}  // namespace

extern "C" {

ms_status ms_dense(const void* x, const void* w, int32_t T, int32_t n_in, int32_t n_out, float* y, const float* add,
                   void* stream) {
  if (T < 0 || n_in <= 0 || n_out <= 0) return MS_E_INVALID;
  if (T == 0) return MS_OK;
  if (!x || !w || !y || !aligned16(x) || !aligned16(w)) return MS_E_INVALID;
  if (n_in % 8 != 0 || n_in > 8192) return MS_E_UNSUPPORTED;
  const hipStream_t s = static_cast<hipStream_t>(stream);
  const dim3 grid((n_out + kDenseRows - 1) / kDenseRows);
  const auto* xp = static_cast<const uint16_t*>(x);
  const auto* wp = static_cast<const uint16_t*>(w);
  if (n_in % kDsSlab == 0) {
    if (T < kDenseMmaTokens) {
      const int wgs = (n_out - 1) / 16 + 1;
      if (wgs <= kDsCus && n_in >= kDsLongRow)
        hipLaunchKernelGGL((dense_few_kernel<8>), dim3(wgs), dim3(512), 0, s, xp, wp, add, y, T, n_in, n_out);
      else
        hipLaunchKernelGGL((dense_few_kernel<4>), dim3(wgs), dim3(256), 0, s, xp, wp, add, y, T, n_in, n_out);
      return launched();
    }
    return launch_dense_staged(xp, wp, add, y, T, n_in, n_out, s);
  }
  if (T >= kDenseMmaTokens && n_in % 32 == 0) {
    hipLaunchKernelGGL(dense_mma_kernel, dim3((T + 63) / 64, (n_out + 63) / 64), dim3(256), msk::kGuardLds, s, xp, wp,
                       add, y, T, n_in, n_out);
    return launched();
  }
  if (n_in <= 4096)
    hipLaunchKernelGGL((dense_kernel<4, 8>), grid, dim3(kDenseThreads), 4 * n_in * 2, s, xp, wp, add, y, T, n_in,
                       n_out);
  else
    hipLaunchKernelGGL((dense_kernel<2, 16>), grid, dim3(kDenseThreads), 2 * n_in * 2, s, xp, wp, add, y, T, n_in,
                       n_out);
  return launched();
}

ms_status ms_rope_kv(const float* qkv, int32_t T, int32_t Hq, int32_t Hkv, int32_t D, int32_t pos0, double base,
                     void* q_out, void* k_cache, void* v_cache, int32_t max_ctx, void* stream) {
  if (T < 0 || Hq <= 0 || Hkv <= 0 || D <= 0 || pos0 < 0 || max_ctx <= 0 || !(base > 1.0)) return MS_E_INVALID;
  if (T == 0) return MS_OK;
  if (!qkv || !q_out || !k_cache || !v_cache) return MS_E_INVALID;
  if (D % 2 != 0 || Hq % Hkv != 0) return MS_E_INVALID;
  if (static_cast<int64_t>(pos0) + T > max_ctx) return MS_E_INVALID;
  const int64_t heads = static_cast<int64_t>(Hq) + 2 * Hkv;
  if ((D <= 128 && (heads < kRopeFewHeads || heads * T <= kRopeFewRows)) || D / 2 > kRopeMaxHalf ||
      T > static_cast<int>(UINT32_MAX / kRopeThreads)) {
    hipLaunchKernelGGL(rope_kv_few_kernel, dim3(T, static_cast<unsigned>(heads)), dim3(64), msk::kGuardLds,
                       static_cast<hipStream_t>(stream), qkv, Hq, Hkv, D, pos0, log2(base),
                       static_cast<uint16_t*>(q_out), static_cast<uint16_t*>(k_cache), static_cast<uint16_t*>(v_cache),
                       max_ctx);
    return launched();
  }
  const bool wide = D % 8 == 0 && aligned16(qkv) &&
                    ((reinterpret_cast<uintptr_t>(q_out) | reinterpret_cast<uintptr_t>(k_cache) |
                      reinterpret_cast<uintptr_t>(v_cache)) & 7u) == 0;
  // blocks per token: enough work-groups to fill the GPU, at least one pass each
  const int64_t items = heads * (D / 2) / (wide ? 4 : 1);
  const int y = static_cast<int>(std::min<int64_t>((items + kRopeThreads - 1) / kRopeThreads, std::max(1, 2048 / T)));
  hipLaunchKernelGGL(wide ? rope_kv_kernel<4> : rope_kv_kernel<1>, dim3(T, y), dim3(kRopeThreads), 0,
                     static_cast<hipStream_t>(stream), qkv, Hq, Hkv, D, pos0, log2(base), static_cast<uint16_t*>(q_out),
                     static_cast<uint16_t*>(k_cache), static_cast<uint16_t*>(v_cache), max_ctx);
  return launched();
}

ms_status ms_attention(const void* q, const void* k_cache, const void* v_cache, int32_t T, int32_t Hq, int32_t Hkv,
                       int32_t D, int32_t pos0, int32_t max_ctx, void* out, void* stream) {
  if (T < 0 || Hq <= 0 || Hkv <= 0 || D <= 0 || pos0 < 0 || max_ctx <= 0) return MS_E_INVALID;
  if (T == 0) return MS_OK;
  if (!q || !k_cache || !v_cache || !out || !aligned16(k_cache) || !aligned16(v_cache)) return MS_E_INVALID;
  if (Hq % Hkv != 0 || static_cast<int64_t>(pos0) + T > max_ctx) return MS_E_INVALID;
  const int G = Hq / Hkv;
  if (D < 8 || D > 512 || (D & (D - 1)) != 0 || G > 8 || static_cast<int64_t>(G) * (5 * D + pos0 + T) > kAttMaxScores)
    return MS_E_UNSUPPORTED;
  const hipStream_t s = static_cast<hipStream_t>(stream);
  const auto* qp = static_cast<const uint16_t*>(q);
  const auto* kp = static_cast<const uint16_t*>(k_cache);
  const auto* vp = static_cast<const uint16_t*>(v_cache);
  auto* op = static_cast<uint16_t*>(out);
#define MSK_ATT_CASE(G_)                                                                                    \
  case G_: return launch_attention<G_>(qp, kp, vp, T, Hq, Hkv, D, pos0, max_ctx, op, s);
  switch (G) {
    MSK_ATT_CASE(1)
    MSK_ATT_CASE(2)
    MSK_ATT_CASE(4)
    MSK_ATT_CASE(8)
    default: return MS_E_UNSUPPORTED;
  }
#undef MSK_ATT_CASE
}

ms_status ms_argmax(const float* x, int32_t T, int32_t n, int32_t* idx_out, void* stream) {
  if (T < 0 || n <= 0) return MS_E_INVALID;
  if (T == 0) return MS_OK;
  if (!x || !idx_out) return MS_E_INVALID;
  hipLaunchKernelGGL(argmax_kernel, dim3(T), dim3(256), 0, static_cast<hipStream_t>(stream), x, n, idx_out);
  return launched();
}

ms_status ms_embed(const int32_t* ids, const void* table, int32_t n_vocab, int32_t T, int32_t d, void* out,
                   void* stream) {
  if (T < 0 || n_vocab <= 0 || d <= 0) return MS_E_INVALID;
  if (T == 0) return MS_OK;
  if (!ids || !table || !out || !aligned16(table) || !aligned16(out) || d % 8 != 0) return MS_E_INVALID;
  hipLaunchKernelGGL(embed_kernel, dim3(T), dim3(256), msk::kGuardLds, static_cast<hipStream_t>(stream), ids,
                     static_cast<const uint16_t*>(table), n_vocab, d, static_cast<uint16_t*>(out));
  return launched();
}

}  // extern "C"
