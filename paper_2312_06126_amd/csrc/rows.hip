// Row-tile update step: see rows.h for the operation list and the packed layouts.
//
// Why this shape. The layers of the narrow networks (up to a few hundred units) are bound by
// everything but the matrix cores when each is a launch of its own: 60 launches of 2 - 15 us
// a step, activations written and read back between them. Here a tile's activations stay in
// LDS and its weights, which every tile shares, stream from L2 as whole 1 KB fragments
// straight into registers (each fragment is used by one wave only, so LDS would not help).
// fp32 needs 16 bytes of weights per CU clock at 32-row tiles, far below L2's rate; bf16
// needs eight times that at 64 rows and is bound by L2.
// Measured, a step with graph replay against the layer-by-layer path: 2 x 64 fp32 at 256 rows
// 260 -> 70 us; 2 x 256 fp32 at 8192 rows 520 -> 290 us; 400-300 fp32 (TD3) at 32768 rows
// 1.89 -> 1.63 ms; 2 x 256 bf16 (376 inputs) at 16384 rows 420 -> 300 us.
#include "rows.h"

#include <atomic>

namespace spz {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <typename T> struct RowT;
template <> struct RowT<float> { static constexpr int KS = 8, VEC = 4, RG = 8; };
template <> struct RowT<bf16_t> { static constexpr int KS = 16, VEC = 8, RG = 16; };

// acc += A B^T over one KS-deep step, both operands as fragments.
template <typename T>
__device__ inline void mma(f32x16& acc, const u32x4& a, const u32x4& b) {
  if constexpr (sizeof(T) == 2) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc,
                                                  0, 0, 0);
  } else {
    const f32x4 x = __builtin_bit_cast(f32x4, a), y = __builtin_bit_cast(f32x4, b);
#pragma unroll
    for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[i], y[i], acc, 0, 0, 0);
  }
}

__device__ inline void zero(f32x16& a) {
#pragma unroll
  for (int q = 0; q < 16; ++q) a[q] = 0.0f;
}

// A 32 x 32 block in accumulator order (v: column lane % 32, rows 8 (q / 4) + 4 (lane / 32) +
// q % 4) to the packed image of a batch tensor with ncb column blocks; rt: 32-row block.
template <typename T>
__device__ inline void pack_block(void* pack, const T (&v)[16], int64_t rt, int ncb, int cb, int lane) {
  u32x4* p = static_cast<u32x4*>(pack);
  constexpr int G = 32 / RowT<T>::RG;
#pragma unroll
  for (int g = 0; g < G; ++g) {
    u32x4 o;
    if constexpr (sizeof(T) == 2) {
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (uint32_t)v[8 * g + 2 * e] | ((uint32_t)v[8 * g + 2 * e + 1] << 16);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = __builtin_bit_cast(uint32_t, v[4 * g + e]);
    }
    p[((rt * G + g) * ncb + cb) * 64 + lane] = o;
  }
}

template <typename T>
__device__ inline void unpack_block(const void* pack, T (&v)[16], int64_t rt, int ncb, int cb, int lane) {
  const u32x4* p = static_cast<const u32x4*>(pack);
  constexpr int G = 32 / RowT<T>::RG;
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const u32x4 o = p[((rt * G + g) * ncb + cb) * 64 + lane];
    if constexpr (sizeof(T) == 2) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[8 * g + 2 * e] = (T)(o[e] & 0xFFFFu);
        v[8 * g + 2 * e + 1] = (T)(o[e] >> 16);
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[4 * g + e] = __builtin_bit_cast(f32x4, o)[e];
    }
  }
}

// Row (within its 32-row block) of accumulator register q.
__device__ inline int acc_row(int q, int lane) { return 8 * (q >> 2) + 4 * (lane >> 5) + (q & 3); }

// The arguments and the operation list are uniform and constant for the launch: fields are
// read through the scalar cache where they are used. The pointers are made opaque once per
// operation, or the compiler would keep every field of both in registers across the whole
// list and spill them.
#define CONST_AS __attribute__((address_space(4)))
template <typename S>
__device__ inline const S* opaque(const CONST_AS S* p) {
  asm volatile("" : "+s"(p));
  return (const S*)p;
}

struct Lds {
  uint8_t* base;
  const RowArgs& g;
  template <typename T> __device__ inline T* x() const { return reinterpret_cast<T*>(base + g.oX); }
  template <typename T> __device__ inline T* h(int slot) const { return reinterpret_cast<T*>(base + g.oH) + slot * g.hnet; }
  __device__ inline float* z() const { return reinterpret_cast<float*>(base + g.oZ); }
  // per-row values: 0, 1 q of the two nets, 2 y, 3, 4 dq of the two nets, 5 log pi
  __device__ inline float* v(int i) const { return reinterpret_cast<float*>(base + g.oV) + i * 32 * g.tm; }
  __device__ inline uint16_t* m() const { return reinterpret_cast<uint16_t*>(base + g.oM); }
};

// One product operation on the wave's NB column blocks first, first + stride, ...
template <typename T, int TM, int MAXNB, int NB>
__device__ inline void product(const RowArgs& g, const RowOp& o, const Lds& L, int64_t tile, int net, int slot, int first,
                               int stride, int lane) {
  constexpr int KS = RowT<T>::KS, BM = 32 * TM;
  // weight fragments in flight per buffer
  constexpr int PD = (MAXNB <= 2 && TM == 1 ? 4 : 8) / NB;
  const int half = lane >> 5, c32 = lane & 31, steps = o.steps;
  const int lda = o.from_h ? g.ldh : g.ldx;
  const T* a = (o.from_h ? L.h<T>(slot) : L.x<T>()) + c32 * lda + (KS / 2) * half;
  const u32x4* w = static_cast<const u32x4*>(o.w[net - o.net0]) + first * steps * 64;
  const int ws = stride * steps * 64;
  float bias[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) bias[j] = o.bias[net - o.net0] ? o.bias[net - o.net0][(first + j * stride) * 32 + c32] : 0.0f;

  f32x16 acc[TM][NB];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) zero(acc[i][j]);

  u32x4 b0[PD][NB], b1[PD][NB];
  auto load = [&](u32x4 (&b)[PD][NB], int s0) {
#pragma unroll
    for (int i = 0; i < PD; ++i) {
      const u32x4* p = w + min(s0 + i, steps - 1) * 64;   // uniform
#pragma unroll
      for (int j = 0; j < NB; ++j) b[i][j] = (p + j * ws)[lane];
    }
  };
  auto multiply = [&](const u32x4 (&b)[PD][NB], int s0) {
#pragma unroll
    for (int i = 0; i < PD; ++i) {
      if (s0 + i >= steps) break;   // uniform
      u32x4 af[TM];
#pragma unroll
      for (int t = 0; t < TM; ++t) af[t] = *reinterpret_cast<const u32x4*>(a + t * 32 * lda + (s0 + i) * KS);
#pragma unroll
      for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int j = 0; j < NB; ++j) mma<T>(acc[t][j], af[t], b[i][j]);
    }
  };
  load(b0, 0);
  for (int s = 0; s < steps; s += 2 * PD) {
    if (s + PD < steps) load(b1, s + PD);
    multiply(b0, s);
    if (s + 2 * PD < steps) load(b0, s + 2 * PD);
    if (s + PD < steps) multiply(b1, s + PD);
  }

  if (o.from_h) __syncthreads();   // every wave is done reading H before it is overwritten
  uint16_t* mask = o.mask >= 0 ? L.m() + o.mask + (net - o.net0) * (o.nblk * TM * 64) : nullptr;
  T* H = L.h<T>(slot);
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int cb = first + j * stride, col = cb * 32 + c32;
    float sum = 0.0f;
#pragma unroll
    for (int t = 0; t < TM; ++t) {
      if (o.kind == ROW_Z || o.kind == ROW_DACT) {
        float* z = L.z() + (o.kind == ROW_DACT ? (net - 1) * BM * g.zp : 0) + t * 32 * g.zp + col;
#pragma unroll
        for (int q = 0; q < 16; ++q) z[acc_row(q, lane) * g.zp] = acc[t][j][q] + bias[j];
        continue;
      }
      T v[16];
      uint16_t* mp = mask ? mask + (cb * TM + t) * 64 + lane : nullptr;
      uint32_t bits = 0;
      if (o.kind == ROW_HIDDEN) {
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          float x = acc[t][j][q] + bias[j];
          x = x < 0.0f ? 0.0f : x;
          v[q] = from_f<T>(x);
          bits |= to_f<T>(v[q]) > 0.0f ? 1u << q : 0u;
        }
        if (mp) *mp = (uint16_t)bits;
      } else {   // ROW_DGRAD
        bits = *mp;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          v[q] = from_f<T>((bits >> q) & 1u ? acc[t][j][q] : 0.0f);
          sum += to_f<T>(v[q]);
        }
      }
#pragma unroll
      for (int q = 0; q < 16; ++q) H[(t * 32 + acc_row(q, lane)) * g.ldh + col] = v[q];
      if (o.pack[net - o.net0]) pack_block<T>(o.pack[net - o.net0], v, tile * TM + t, o.nblk, cb, lane);
    }
    if (o.part[net - o.net0]) {
      sum += __shfl_xor(sum, 32);
      if (half == 0) o.part[net - o.net0][tile * (o.nblk * 32) + col] = sum;
    }
  }
}

// Gradient of the last hidden layer from dq: H = dq w where the unit was active, with its
// packed image and column sums, and the output layer's weight-gradient sums.
template <typename T, int TM>
__device__ inline void output_backward(const RowArgs& g, const RowOp& o, const Lds& L, int64_t tile, int net, int slot,
                                       int first, int cnt, int stride, int lane) {
  const int k = net - o.net0, c32 = lane & 31;
  const uint16_t* mask = L.m() + o.mask + k * (o.nblk * TM * 64);
  const float* dq = L.v(3 + net - 1);
  T* H = L.h<T>(slot);
  for (int j = 0; j < cnt; ++j) {
    const int cb = first + j * stride, col = cb * 32 + c32;
    const float w = to_f<T>(from_f<T>(static_cast<const float*>(o.w[k])[col]));
    float sum = 0.0f, wsum = 0.0f;
#pragma unroll
    for (int t = 0; t < TM; ++t) {
      const uint32_t bits = mask[(cb * TM + t) * 64 + lane];
      T v[16], h[16];
      if (o.wpart[k]) unpack_block<T>(o.hpack[k], h, tile * TM + t, o.nblk, cb, lane);
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int r = t * 32 + acc_row(q, lane);
        const float d = dq[r];
        if (o.wpart[k]) wsum = fmaf(d, to_f<T>(h[q]), wsum);
        v[q] = from_f<T>((bits >> q) & 1u ? d * w : 0.0f);
        sum += to_f<T>(v[q]);
        H[r * g.ldh + col] = v[q];
      }
      if (o.pack[k]) pack_block<T>(o.pack[k], v, tile * TM + t, o.nblk, cb, lane);
    }
    if (o.part[k]) {
      sum += __shfl_xor(sum, 32);
      if (lane < 32) o.part[k][tile * (o.nblk * 32) + col] = sum;
    }
    if (o.wpart[k]) {
      wsum += __shfl_xor(wsum, 32);
      if (lane < 32) o.wpart[k][tile * (o.nblk * 32) + col] = wsum;
    }
  }
}

template <typename T, int TM>
__device__ inline void load_tile(const RowArgs& g, const RowOp& o, const Lds& L, int64_t tile, int tid) {
  constexpr int VEC = RowT<T>::VEC, BM = 32 * TM;
  const T* src = static_cast<const T*>(o.flags ? g.xsa : g.xs2) + tile * BM * (int64_t)g.Kc;
  T* X = L.x<T>();
  const int nv = g.Kc / VEC;
#pragma unroll 4
  for (int v = tid; v < BM * nv; v += ROW_THREADS) {
    const int r = v / nv, c = (v - r * nv) * VEC;
    *reinterpret_cast<u32x4*>(X + r * g.ldx + c) = *reinterpret_cast<const u32x4*>(src + (int64_t)v * VEC);
  }
  if (!o.pack[0]) return;
  __syncthreads();
  const int lane = tid & 63, ncb = g.Kc / 32;
  for (int u = tid >> 6; u < ncb * TM; u += ROW_WAVES) {
    const int cb = u % ncb, t = u / ncb;
    T v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = X[(t * 32 + acc_row(q, lane)) * g.ldx + cb * 32 + (lane & 31)];
    pack_block<T>(o.pack[0], v, tile * TM + t, ncb, cb, lane);
  }
}

// q[net][r] of the critic output layer: 16 lanes per row.
template <typename T, int TM>
__device__ inline void output_dot(const RowArgs& g, const RowOp& o, const Lds& L, int tid) {
  constexpr int VEC = RowT<T>::VEC, BM = 32 * TM;
  const int l = tid & 15, K = o.nblk * 32;
  for (int d = tid >> 4; d < o.nets * BM; d += ROW_THREADS / 16) {
    const int k = d / BM, r = d % BM;
    const T* h = L.h<T>(o.nets == 2 ? k : 0) + r * g.ldh;
    const float* w = static_cast<const float*>(k ? o.w[1] : o.w[0]);
    float s = 0.0f;
    for (int c = l * VEC; c < K; c += 16 * VEC) {
      const u32x4 hv = *reinterpret_cast<const u32x4*>(h + c);
#pragma unroll
      for (int e = 0; e < VEC / 4; ++e) {
        const f32x4 wv = *reinterpret_cast<const f32x4*>(w + c + 4 * e);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float hx;
          if constexpr (sizeof(T) == 2) {
            const uint32_t p = hv[2 * e + (i >> 1)];
            hx = bf2f((bf16_t)(i & 1 ? p >> 16 : p & 0xFFFFu));
          } else {
            hx = __builtin_bit_cast(f32x4, hv)[i];
          }
          s = fmaf(hx, to_f<T>(from_f<T>(wv[i])), s);
        }
      }
    }
#pragma unroll
    for (int m = 8; m > 0; m >>= 1) s += __shfl_xor(s, m);
    if (l == 0) L.v(o.net0 - 1 + k)[r] = s + *(k ? o.bias[1] : o.bias[0]);
  }
}

__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) v += __shfl_xor(v, m);
  return v;
}
__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) v += __shfl_xor(v, m);
  return v;
}

// Critic loss of the tile's rows (the first wave): dq_i = 2 (q_i - y) / B in the operand
// type, and the tile's sums of (q1 - y)^2, (q2 - y)^2, q1 and of each dq.
template <typename T, int TM>
__device__ inline void critic_loss(const RowArgs& g, const RowOp& o, const Lds& L, int64_t tile, int lane) {
  constexpr int BM = 32 * TM;
  const int64_t b = tile * BM + lane;
  float d1 = 0.0f, d2 = 0.0f;
  double e1s = 0.0, e2s = 0.0, q1s = 0.0;
  if (lane < BM) {
    if (b < g.B) {
      const float q1 = L.v(0)[lane], q2 = L.v(1)[lane], y = L.v(2)[lane];
      const float e1 = q1 - y, e2 = q2 - y;
      d1 = to_f<T>(from_f<T>(2.0f * e1 / (float)g.B));
      d2 = to_f<T>(from_f<T>(2.0f * e2 / (float)g.B));
      e1s = (double)e1 * e1;
      e2s = (double)e2 * e2;
      q1s = q1;
      g.q1[b] = q1;
      g.q2[b] = q2;
    }
    L.v(3)[lane] = d1;
    L.v(4)[lane] = d2;
  }
  e1s = wave_sum(e1s);
  e2s = wave_sum(e2s);
  q1s = wave_sum(q1s);
  d1 = wave_sum(d1);
  d2 = wave_sum(d2);
  if (lane == 0) {
    g.cpart[tile * 3 + 0] = e1s;
    g.cpart[tile * 3 + 1] = e2s;
    g.cpart[tile * 3 + 2] = q1s;
    o.part[0][tile] = d1;
    o.part[1][tile] = d2;
  }
}

// Actor loss of the tile's rows (the first wave). SAC: dq = -1 / B to the smaller critic
// (critic 1 on ties); sums of alpha log pi - min(q1, q2) and of log pi. TD3: critic 1 only,
// sum of q1.
template <typename T, int TM>
__device__ inline void actor_loss(const RowArgs& g, const Lds& L, int64_t tile, int lane) {
  constexpr int BM = 32 * TM;
  const int64_t b = tile * BM + lane;
  double l0 = 0.0, l1 = 0.0;
  if (lane < BM) {
    float g1 = 0.0f, g2 = 0.0f;
    if (b < g.B) {
      const float inv = to_f<T>(from_f<T>(-1.0f / (float)g.B));
      const float q1 = L.v(0)[lane];
      g.qp1[b] = q1;
      if (g.sac) {
        const float q2 = L.v(1)[lane], lp = L.v(5)[lane];
        const bool take1 = q1 <= q2;
        g1 = take1 ? inv : 0.0f;
        g2 = take1 ? 0.0f : inv;
        l0 = (double)expf(*g.log_alpha) * lp - (double)(take1 ? q1 : q2);
        l1 = lp;
        g.qp2[b] = q2;
      } else {
        g1 = inv;
        l0 = q1;
      }
    }
    L.v(3)[lane] = g1;
    L.v(4)[lane] = g2;
  }
  l0 = wave_sum(l0);
  l1 = wave_sum(l1);
  if (lane == 0) {
    g.apart[tile * 2 + 0] = l0;
    g.apart[tile * 2 + 1] = l1;
  }
}

// Policy head: Z -> the action columns of X. SAC: the log-density terms take the place of
// the means in Z and are added per row in action order.
template <typename T, int TM>
__device__ inline void head(const RowArgs& g, const RowOp& o, const Lds& L, int64_t tile, int tid) {
  constexpr int BM = 32 * TM;
  T* X = L.x<T>();
  float* Z = L.z();
  const bool policy = o.flags != 0;
  const uint32_t t = (uint32_t)(*g.step + 1);
  for (int e = tid; e < BM * g.A; e += ROW_THREADS) {
    const int r = e / g.A, j = e - r * g.A;
    const int64_t b = tile * BM + r;
    float* z = Z + r * g.zp;
    float a = 0.0f, term = 0.0f;
    if (b < g.B) {
      const uint64_t i = (uint64_t)b * g.A + j;
      if (g.sac) {
        const SacHeadValue v = sac_head_value(z[j], z[g.A + j], normal_at(g.seed, i, t, policy ? P_NOISE_POL : P_NOISE_TGT),
                                              g.lmin, g.lmax);
        a = v.a;
        term = v.term;
        if (policy) {
          g.th[i] = a;
          g.se[i] = v.se;
          g.lm[i] = v.lm;
        }
      } else {
        a = tanhf(z[j]);
        if (policy) g.th[i] = a;
        else a = clamp_keep_nan(a + clamp_keep_nan(g.noise * normal_at(g.seed, i, t, P_NOISE_TGT), -g.clip, g.clip), -1.0f, 1.0f);
      }
    }
    X[r * g.ldx + g.Ka + j] = from_f<T>(a);
    if (g.sac) z[j] = term;
  }
  if (!g.sac) return;
  __syncthreads();
  if (tid < BM) {
    float lp = 0.0f;
    for (int j = 0; j < g.A; ++j) lp += Z[tid * g.zp + j];
    L.v(5)[tid] = lp;
    if (policy && tile * BM + tid < g.B) g.logp[tile * BM + tid] = lp;
  }
}

// Actor head backward: the action gradients in Z (of both critics for SAC) -> the actor's
// output gradient in H, with its packed image and column sums.
template <typename T, int TM>
__device__ inline void head_backward(const RowArgs& g, const RowOp& o, const Lds& L, int64_t tile, int tid) {
  constexpr int BM = 32 * TM;
  T* H = L.h<T>(0);
  const float* D = L.z();
  const float aB = g.sac ? expf(*g.log_alpha) / (float)g.B : 0.0f;
  for (int e = tid; e < BM * g.pa; e += ROW_THREADS) {
    const int r = e / g.pa, c = e - r * g.pa;
    const int64_t b = tile * BM + r;
    const bool mean = c < g.A;
    const int j = mean ? c : c - g.A;
    float out = 0.0f;
    if (b < g.B && (mean || (g.sac && j < g.A))) {
      float da = D[r * g.zp + j];
      if (g.sac) da += D[(BM + r) * g.zp + j];
      const uint64_t i = (uint64_t)b * g.A + j;
      const float a = g.th[i];
      out = da * (1.0f - a * a);
      if (g.sac) out += aB * 2.0f * a;
      if (mean) g.da[b * g.Ap + j] = da;
      else out = (out * g.se[i] - aB) * g.lm[i];
    }
    H[r * g.ldh + c] = from_f<T>(out);
  }
  __syncthreads();
  const int lane = tid & 63;
  for (int cb = tid >> 6; cb < o.nblk; cb += ROW_WAVES) {
    float sum = 0.0f;
#pragma unroll
    for (int t = 0; t < TM; ++t) {
      T v[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        v[q] = H[(t * 32 + acc_row(q, lane)) * g.ldh + cb * 32 + (lane & 31)];
        sum += to_f<T>(v[q]);
      }
      pack_block<T>(o.pack[0], v, tile * TM + t, o.nblk, cb, lane);
    }
    sum += __shfl_xor(sum, 32);
    if (lane < 32) o.part[0][tile * (o.nblk * 32) + cb * 32 + lane] = sum;
  }
}

template <typename T, int TM, int MAXNB>
__global__ void __launch_bounds__(ROW_THREADS, MAXNB <= 2 && TM == 1 ? 4 : 2) k_rows(RowArgs args) {
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  constexpr int BM = 32 * TM;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int part = (int)blockIdx.x >= args.tiles ? 1 : 0;
  const int64_t tile = (int)blockIdx.x - part * args.tiles;
  const CONST_AS RowArgs* argp = (const CONST_AS RowArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  const CONST_AS RowOp* op = (const CONST_AS RowOp*)(uintptr_t)(args.ops + args.op0[part]);
  for (int n = args.nops[part]; n > 0; --n, ++op) {
    const RowArgs& g = *opaque(argp);
    const RowOp& o = *opaque(op);
    const Lds L{smem, g};
    // The wave's share of the operation's column blocks.
    const int wpn = o.nets == 2 ? ROW_WAVES / 2 : ROW_WAVES;
    const int k = wave / wpn, first = wave - k * wpn;
    const int net = o.net0 + k, slot = o.nets == 2 ? k : 0;
    const int cnt = o.nblk > first ? (o.nblk - 1 - first) / wpn + 1 : 0;
    switch (o.kind) {
      case ROW_HIDDEN: case ROW_Z: case ROW_DGRAD: case ROW_DACT:
        if (cnt == 1) product<T, TM, MAXNB, 1>(g, o, L, tile, net, slot, first, wpn, lane);
        else if (cnt == 2) product<T, TM, MAXNB, 2>(g, o, L, tile, net, slot, first, wpn, lane);
        else if (MAXNB > 2 && cnt == 3) product<T, TM, MAXNB, (MAXNB > 2 ? 3 : 1)>(g, o, L, tile, net, slot, first, wpn, lane);
        else if (MAXNB > 2 && cnt == 4) product<T, TM, MAXNB, (MAXNB > 2 ? 4 : 1)>(g, o, L, tile, net, slot, first, wpn, lane);
        else if (o.from_h) __syncthreads();
        break;
      case ROW_LOAD: load_tile<T, TM>(g, o, L, tile, tid); break;
      case ROW_OBS: {
        T* X = L.x<T>();
        for (int e = tid; e < BM * g.Ka; e += ROW_THREADS) {
          const int r = e / g.Ka, c = e - r * g.Ka;
          const int64_t b = tile * BM + r;
          X[r * g.ldx + c] = from_f<T>(b < g.B && c < g.O ? g.obs[b * g.O + c] : 0.0f);
        }
        break;
      }
      case ROW_DOT: output_dot<T, TM>(g, o, L, tid); break;
      case ROW_TARGET:
        if (tid < BM) {
          const int64_t b = tile * BM + tid;
          float y = 0.0f;
          if (b < g.B) {
            const float q1 = L.v(0)[tid], q2 = L.v(1)[tid];
            float m = min_keep_nan(q1, q2);
            if (g.sac) m -= expf(*g.log_alpha) * L.v(5)[tid];
            y = g.r[b] + g.gamma * (1.0f - g.d[b]) * m;
            g.y[b] = y;
          }
          L.v(2)[tid] = y;
        }
        break;
      case ROW_CLOSS: if (wave == 0) critic_loss<T, TM>(g, o, L, tile, lane); break;
      case ROW_ALOSS: if (wave == 0) actor_loss<T, TM>(g, L, tile, lane); break;
      case ROW_DZ: output_backward<T, TM>(g, o, L, tile, net, slot, first, cnt, wpn, lane); break;
      case ROW_HEAD: head<T, TM>(g, o, L, tile, tid); break;
      case ROW_HEAD_BWD: head_backward<T, TM>(g, o, L, tile, tid); break;
      case ROW_ACT:
        for (int e = tid; e < BM * g.A; e += ROW_THREADS) {
          const int r = e / g.A, j = e - r * g.A;
          const int64_t b = tile * BM + r;
          if (b >= g.B) break;
          const float* z = L.z() + r * g.zp;
          const int64_t i = b * g.A + j;
          float u = z[j];
          if (g.stochastic)
            u += expf(clamp_keep_nan(z[g.A + j], g.lmin, g.lmax)) * normal_at(g.seed, (uint64_t)(g.row0 * g.A + i), g.counter, P_ACT);
          g.act[i] = tanhf(u);
        }
        break;
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------------------ weight gradients
// One wave takes 2 x 2 blocks of a product over one slice of the batch, fragments straight
// from memory into registers: no LDS, no barriers. The four waves of a workgroup and its
// neighbours on the same XCD take neighbouring tiles of the same slice, which share fragments.
template <typename T>
__global__ void __launch_bounds__(256, 2) k_row_wgrad(RowWArgs W) {
  const int wgs = (W.tasks + 3) / 4;
  int wg = blockIdx.x;
  if (wg >= wgs) {
    __shared__ double sh[256];
    finish_step(W.fin, sh);
    return;
  }
  // Workgroup b runs on XCD b % 8: contiguous ranges of tasks per XCD.
  if (wgs % 8 == 0) wg = (wg % 8) * (wgs / 8) + wg / 8;
  const int lane = threadIdx.x & 63;
  const int task = wg * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (task >= W.tasks) return;
  int k = 0;
  for (int i = 1; i < W.n; ++i)
    if (task >= W.j[i].task0) k = i;
  const RowWJob& J = W.j[k];
  const int tn = (J.nblk + 1) / 2, tiles = (J.mblk + 1) / 2 * tn;
  const int local = task - J.task0, slice = local / tiles, tl = local - slice * tiles;
  const int m0 = tl / tn * 2, n0 = (tl - tl / tn * tn) * 2;
  const bool m2 = m0 + 1 < J.mblk, n2 = n0 + 1 < J.nblk;
  const int g0 = (int)((int64_t)W.groups * slice / J.slices), g1 = (int)((int64_t)W.groups * (slice + 1) / J.slices);
  const u32x4* a = static_cast<const u32x4*>(J.a) + (int64_t)m0 * 64 + lane;
  const u32x4* b = static_cast<const u32x4*>(J.b) + (int64_t)n0 * 64 + lane;
  const int64_t as = (int64_t)J.mblk * 64, bs = (int64_t)J.bcb * 64;
  const int am = m2 ? 64 : 0, bn = n2 ? 64 : 0;
  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 4; ++i) zero(acc[i >> 1][i & 1]);
  constexpr int PD = sizeof(T) == 2 ? 4 : 2;
  u32x4 f0[PD][4], f1[PD][4];
  auto load = [&](u32x4 (&f)[PD][4], int gr) {
#pragma unroll
    for (int i = 0; i < PD; ++i) {
      const int64_t q = min(gr + i, g1 - 1);
      f[i][0] = a[q * as];
      f[i][1] = a[q * as + am];
      f[i][2] = b[q * bs];
      f[i][3] = b[q * bs + bn];
    }
  };
  auto multiply = [&](const u32x4 (&f)[PD][4], int gr) {
#pragma unroll
    for (int i = 0; i < PD; ++i) {
      if (gr + i >= g1) break;
#pragma unroll
      for (int x = 0; x < 4; ++x) mma<T>(acc[x >> 1][x & 1], f[i][x >> 1], f[i][2 + (x & 1)]);
    }
  };
  if (g0 < g1) {
    load(f0, g0);
    for (int gr = g0; gr < g1; gr += 2 * PD) {
      if (gr + PD < g1) load(f1, gr + PD);
      multiply(f0, gr);
      if (gr + 2 * PD < g1) load(f0, gr + 2 * PD);
      if (gr + PD < g1) multiply(f1, gr + PD);
    }
  }
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    if (((x >> 1) && !m2) || ((x & 1) && !n2)) continue;
    f32x4* out = reinterpret_cast<f32x4*>(J.part) +
                 (((int64_t)slice * J.mblk + m0 + (x >> 1)) * J.nblk + n0 + (x & 1)) * 256 + lane;
    const f32x16& c = acc[x >> 1][x & 1];
#pragma unroll
    for (int g = 0; g < 4; ++g) out[g * 64] = f32x4{c[4 * g], c[4 * g + 1], c[4 * g + 2], c[4 * g + 3]};
  }
}

// ------------------------------------------------------------------------------ reduction, Adam, packed images
// Position of element (row m, column n) of a 32-row block's fragments [steps][64][KS / 2].
template <typename T>
__device__ inline int64_t frag_pos(int m, int n) {
  constexpr int KS = RowT<T>::KS, HV = KS / 2;
  return ((int64_t)(n / KS) * 64 + m + 32 * (n % KS / HV)) * HV + n % HV;
}

template <typename T>
__device__ inline void store_packed(T* f, T* t, const RowPBlk& B, int m0, int n, const float (&v)[4]) {
  // rows m0 .. m0 + 3 of column n: four places of the forward image, four consecutive
  // elements of the transposed one
#pragma unroll
  for (int j = 0; j < 4; ++j) f[B.fwd + frag_pos<T>(m0 + j, n)] = from_f<T>(v[j]);
  if (!t || B.tr < 0) return;
  T o[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) o[j] = from_f<T>(v[j]);
  T* p = t + B.tr + frag_pos<T>(n, m0);
  if constexpr (sizeof(T) == 2)
    *reinterpret_cast<uint2*>(p) = make_uint2((uint32_t)o[0] | ((uint32_t)o[1] << 16), (uint32_t)o[2] | ((uint32_t)o[3] << 16));
  else
    *reinterpret_cast<float4*>(p) = make_float4(o[0], o[1], o[2], o[3]);
}

template <typename T>
__global__ void __launch_bounds__(256) k_row_adam(RowPArgs p) {
  __shared__ float bc[4];
  __shared__ float4 sh[256];
  const AdamArgs& a = p.a;
  const RowPBlk B = p.blk[p.first + blockIdx.x];
  T* PF = static_cast<T*>(p.PF);
  T* PT = static_cast<T*>(p.PT);
  T* TF = static_cast<T*>(p.TF);
  const int tid = threadIdx.x;
  // Thread of a weight block: column n, rows m0 .. m0 + 3 (accumulator order).
  const int lane = tid & 63, n = lane & 31, m0 = 8 * (tid >> 6) + 4 * (lane >> 5);
  if (!p.update) {
    if (B.kind != 0) return;
    float v[4], u[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t i = B.off + (int64_t)(m0 + j) * B.ld + n;
      v[j] = a.P[i];
      u[j] = a.T[i];
    }
    store_packed<T>(PF, PT, B, m0, n, v);
    store_packed<T>(TF, nullptr, B, m0, n, u);
    return;
  }
  adam_corrections(a, bc);
  const bool actor = B.net == 0;
  const bool polyak = actor ? a.polyak_actor : a.polyak_critic;
  const float lr = actor ? a.lr_a : a.lr_c;
  auto element = [&](int64_t i, float g, float& t) {
    a.G[i] = g;
    float m = a.M[i], v = a.V[i];
    const float x = adam_element(a, a.P[i], m, v, g, lr, bc[actor ? 2 : 0], bc[actor ? 3 : 1]);
    a.M[i] = m;
    a.V[i] = v;
    a.P[i] = x;
    if (polyak) {
      t = (1.0f - a.tau) * a.T[i] + a.tau * x;
      a.T[i] = t;
    }
    return x;
  };
  float t;
  if (B.kind == 0) {
    const RowPJob J = p.j[B.job];
    const float4* src = reinterpret_cast<const float4*>(J.part) + (int64_t)B.blk * 256 + tid;
    const int64_t zs = J.zstride / 4;
    float4 s = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll 8
    for (int z = 0; z < J.slices; ++z) {
      const float4 v = src[z * zs];
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    __syncthreads();
    const float g[4] = {s.x, s.y, s.z, s.w};
    float v[4], u[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = element(B.off + (int64_t)(m0 + j) * B.ld + n, g[j], u[j]);
    store_packed<T>(PF, PT, B, m0, n, v);
    if (polyak) store_packed<T>(TF, nullptr, B, m0, n, u);
    return;
  }
  if (B.kind == 1) {
    // 16 columns as 4 pieces of 4, each summed by 64 threads over every 64th slice, then
    // the thread sums in order.
    const int piece = tid & 3, grp = tid >> 2;
    const float* src = B.part + 4 * piece;
    float4 s = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll 4
    for (int z = grp; z < p.vslices; z += 64) {
      const float4 v = *reinterpret_cast<const float4*>(src + (int64_t)z * B.ld);
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    sh[tid] = s;
    __syncthreads();
    if (tid >= 16) return;
    const float* f = reinterpret_cast<const float*>(sh);
    float g = 0.0f;
    for (int q = 0; q < 64; ++q) g += f[q * 16 + tid];
    element(B.off + tid, g, t);
    return;
  }
  if (B.kind == 2) {
    float* f = reinterpret_cast<float*>(sh);
    float s = 0.0f;
    for (int z = tid; z < p.vslices; z += 256) s += B.part[z];
    f[tid] = s;
    __syncthreads();
    if (tid != 0) return;
    float g = 0.0f;
    for (int q = 0; q < 256; ++q) g += f[q];
    element(B.off, g, t);
    return;
  }
  __syncthreads();
  if (tid == 0 && a.do_alpha) {   // the temperature: its gradient is already in G
    float m = a.M[B.off], v = a.V[B.off];
    a.P[B.off] = adam_element(a, a.P[B.off], m, v, a.G[B.off], a.lr_al, bc[0], bc[1]);
    a.M[B.off] = m;
    a.V[B.off] = v;
  }
}

template <typename T, int TM, int MAXNB>
hipError_t launch_rows_t(const RowArgs& g, size_t lds, hipStream_t s) {
  static std::atomic<bool> ready{false};
  if (!ready.load()) {
    const hipError_t e = hipFuncSetAttribute((const void*)(k_rows<T, TM, MAXNB>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
    ready.store(true);
  }
  (k_rows<T, TM, MAXNB>)<<<g.tiles * g.parts, ROW_THREADS, lds, s>>>(g);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_rows(bool bf16, const RowArgs& g, int max_blocks, size_t lds, hipStream_t s) {
  if (g.tiles < 1 || g.parts < 1 || g.parts > 2 || (g.tm != 1 && g.tm != 2) || max_blocks < 1 ||
      max_blocks > ROW_MAX_BLOCKS || lds > 160 * 1024 || (!bf16 && g.tm != 1) || (int64_t)g.tiles * 32 * g.tm < g.B)
    return hipErrorInvalidValue;
  if (!bf16) return max_blocks <= 2 ? launch_rows_t<float, 1, 2>(g, lds, s) : launch_rows_t<float, 1, 4>(g, lds, s);
  if (g.tm == 1) return max_blocks <= 2 ? launch_rows_t<bf16_t, 1, 2>(g, lds, s) : launch_rows_t<bf16_t, 1, 4>(g, lds, s);
  return max_blocks <= 2 ? launch_rows_t<bf16_t, 2, 2>(g, lds, s) : launch_rows_t<bf16_t, 2, 4>(g, lds, s);
}

hipError_t launch_row_wgrad(bool bf16, RowWArgs& w, hipStream_t s) {
  if (w.n < 1 || w.n > MAX_ROW_WJOBS || w.groups < 1) return hipErrorInvalidValue;
  w.tasks = 0;
  for (int i = 0; i < w.n; ++i) {
    RowWJob& j = w.j[i];
    if (j.mblk < 1 || j.nblk < 1 || j.bcb < j.nblk || j.slices < 1) return hipErrorInvalidValue;
    j.task0 = w.tasks;
    w.tasks += row_wjob_tiles(j.mblk, j.nblk) * j.slices;
  }
  const int grid = (w.tasks + 3) / 4 + (w.has_fin ? 1 : 0);
  if (bf16) k_row_wgrad<bf16_t><<<grid, 256, 0, s>>>(w);
  else k_row_wgrad<float><<<grid, 256, 0, s>>>(w);
  return hipGetLastError();
}

hipError_t launch_row_adam(bool bf16, const RowPArgs& p, hipStream_t s) {
  if (p.count < 1) return hipSuccess;
  if (bf16) k_row_adam<bf16_t><<<p.count, 256, 0, s>>>(p);
  else k_row_adam<float><<<p.count, 256, 0, s>>>(p);
  return hipGetLastError();
}

}  // namespace spz
