// Row-tile update step: see rows.h for the operation list and the packed layouts.
//
// Why this shape. The layers of the narrow networks (up to a few hundred units) are bound by
// everything but the matrix cores when each is a launch of its own: 60 launches of 2 - 15 us
// a step, activations written and read back between them. Here a tile's activations stay in
// LDS and its weights, which every tile shares, stream from L2 as whole 1 KB fragments
// straight into registers (each fragment is used by one wave only, so LDS would not help).
// fp32 is bound by the matrix cores (2 x 256 at 8192 rows: 60% of their rate in k_rows, 400-300
// at 32768 rows: 77%), bf16 by the weights' way through the vector L1 (64 bytes a clock) and by
// the fixed time of an operation, 2 - 3 thousand clocks of loads, epilogue and barriers.
// Measured, a step against the layer-by-layer path: 2 x 64 fp32 at 256 rows 260 -> 50 us; 2 x
// 256 fp32 at 8192 rows 520 -> 225 us; 400-300 fp32 (TD3) at 32768 rows 1.89 -> 1.28 ms; 2 x
// 256 bf16 (376 inputs) at 16384 rows 420 -> 188 us; TD3 2 x 256 bf16 at 4096 rows 235 -> 60 us.
#include "rows.h"

namespace spz {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
#define LDS_AS __attribute__((address_space(3)))

// KS: depth of one step of a product; VEC: elements of 16 bytes; WPB: 32-bit words of 16
// accumulator values in the operand type.
template <typename T> struct RowT;
template <> struct RowT<float> { static constexpr int KS = 8, VEC = 4, WPB = 16; };
template <> struct RowT<bf16_t> { static constexpr int KS = 16, VEC = 8, WPB = 8; };

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

// Eight float32 values of a lane (two steps' fragments), 2^24 times each, as a sum of three
// bfloat16: the rounded value, the rounded rest and the rest of that, 24 bits and exact (the last
// rest has at most 8 significant bits, and the factor keeps it a normal number down to the
// smallest normal value: without it values below 2^-109 lose bits).
constexpr float SPLIT_SCALE = 0x1p24f;
struct Split { u32x4 p[3]; };
__device__ inline Split split(const u32x4& lo, const u32x4& hi) {
  Split s;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const f32x4 v = __builtin_bit_cast(f32x4, i < 2 ? lo : hi);
    float a = SPLIT_SCALE * v[2 * (i & 1)], b = SPLIT_SCALE * v[2 * (i & 1) + 1];
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      const uint32_t w = pack_bf16x2(a, b);
      s.p[t][i] = w;
      if (t < 2) {
        a -= __builtin_bit_cast(float, w << 16);
        b -= __builtin_bit_cast(float, w & 0xFFFF0000u);
      }
    }
  }
  return s;
}

// A B^T over two float32 steps (16 deep) on the bfloat16 matrix instructions, 6 x 32 clocks where
// the float32 instructions take 8 x 64: the products of the largest parts are added to `hi`, the
// five of at most 2^-9 and at least 2^-18 of them to `lo` (the three left out are below 2^-26 of
// them). With all six on one accumulator each of them would round the running sum; apart, only
// the first does, once for 16 rows where the float32 instructions round it for every two.
// Distance from 64 bits over that of the float32 instructions (128 x 128, masked gradients and
// ReLU outputs, the sum over all elements): 0.91 at 4 rows, 0.56 at 32, 0.5 at 1000, 0.44 at 32768 and
// 131072; on one accumulator 1.13, 1.12, 1.3, 1.5 and 1.9. One and two rows: see ROW_SPLIT_ROWS.
// Weight gradients only: input gradients on split operands, 3 - 4% faster a step, put the first
// layer's bias gradient up to 1.6 times further off.
__device__ inline void mma_split(f32x16& hi, f32x16& lo, const Split& a, const Split& b) {
  constexpr int A[6] = {2, 0, 1, 1, 0, 0}, B[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    f32x16& c = i < 5 ? lo : hi;
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a.p[A[i]]),
                                                __builtin_bit_cast(bf16x8, b.p[B[i]]), c, 0, 0, 0);
  }
}

__device__ inline void zero(f32x16& a) {
#pragma unroll
  for (int q = 0; q < 16; ++q) a[q] = 0.0f;
}

// A block of a product as a lane holds it: the weight is the A operand, so lane 32 h + r has
// batch row r and the 16 output columns 8 (q / 4) + 4 h + q % 4 -- four runs of four columns,
// which go to LDS as 8 (bf16) or 16 bytes each. (The other way round a lane holds 16 rows of
// one column: 16 two-byte LDS stores and per-value masks took longer than the product itself
// in bf16.) In the operand type: WPB words, bf16 two columns a word.
template <typename T> struct Block { uint32_t w[RowT<T>::WPB]; };

__device__ inline uint32_t pk_min1(uint32_t x) {   // min(x, 1) of both halves
  uint32_t m;
  asm("v_pk_min_u16 %0, %1, %2" : "=v"(m) : "v"(x), "s"(0x00010001u));
  return m;
}

// ReLU of the accumulators, rounded to the operand type, and its mask: 16 bits, 1 where the
// stored value is not zero (fp32: above zero). bf16: the pairs' low halves in bits 7 .. 0, high
// halves in 15 .. 8. A NaN of either sign stays one, so that it reaches the loss record (the
// matrix instructions make negative ones, so the ReLU is not taken on the rounded bits).
template <typename T>
__device__ inline uint32_t relu_block(const f32x16& acc, Block<T>& b) {
  uint32_t bits = 0;
  if constexpr (sizeof(T) == 2) {
#pragma unroll
    for (int p = 0; p < 8; ++p) {
      b.w[p] = pack_bf16x2(__builtin_elementwise_maximum(acc[2 * p], 0.0f),
                           __builtin_elementwise_maximum(acc[2 * p + 1], 0.0f));
      bits = (bits << 1) | pk_min1(b.w[p]);
    }
    bits = __builtin_amdgcn_perm(0u, bits, 0x0C0C0200u);   // bytes 2, 0
  } else {
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const float x = acc[q] < 0.0f ? 0.0f : acc[q];   // keeps NaN
      b.w[q] = __builtin_bit_cast(uint32_t, x);
      bits = (bits << 1) | (x > 0.0f ? 1u : 0u);
    }
  }
  return bits;
}

// v (in the operand type) where the mask bit is set, else 0.
template <typename T>
__device__ inline void mask_block(const float (&v)[16], uint32_t bits, Block<T>& b) {
  if constexpr (sizeof(T) == 2) {
    const uint32_t m = __builtin_amdgcn_perm(0u, bits, 0x0C010C00u);   // bytes 0 and 1 to the halves
#pragma unroll
    for (int p = 0; p < 8; ++p) {
      const uint32_t one = (m >> (7 - p)) & 0x00010001u;
      b.w[p] = pack_bf16x2(v[2 * p], v[2 * p + 1]) & (one * 0xFFFFu);
    }
  } else {
#pragma unroll
    for (int q = 0; q < 16; ++q) b.w[q] = (bits >> (15 - q)) & 1u ? __builtin_bit_cast(uint32_t, v[q]) : 0u;
  }
}

// To row-major LDS: p is the lane's row at the block's first column.
template <typename T>
__device__ inline void store_block(T* p, const Block<T>& b, int half) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    if constexpr (sizeof(T) == 2)
      *reinterpret_cast<uint2*>(p + 8 * g + 4 * half) = make_uint2(b.w[2 * g], b.w[2 * g + 1]);
    else
      *reinterpret_cast<u32x4*>(p + 8 * g + 4 * half) = u32x4{b.w[4 * g], b.w[4 * g + 1], b.w[4 * g + 2], b.w[4 * g + 3]};
  }
}

// The arguments and the operation list are uniform and constant for the launch: fields are
// read through the scalar cache where they are used. The pointers are made opaque once per
// operation, or the compiler would keep every field of both in registers across the whole
// list and spill them. (The list in LDS and its fields in scalar registers from the start of
// an operation was slower: the registers spilled, 137 -> 180 us on 2 x 256 bf16, 16384 rows.)
#define CONST_AS __attribute__((address_space(4)))
template <typename S>
__device__ inline const S* opaque(const CONST_AS S* p) {
  asm volatile("" : "+s"(p));
  return (const S*)p;
}

// Element k (0 or 1) of an operation's pair, without indexed (stack) access.
template <typename V>
__device__ inline V pick(const V (&v)[2], int k) { return k ? v[1] : v[0]; }

struct Lds {
  uint8_t* base;
  const RowArgs& g;
  template <typename T> __device__ inline T* x() const { return reinterpret_cast<T*>(base + g.oX); }
  template <typename T> __device__ inline T* h(int slot) const { return reinterpret_cast<T*>(base + g.oH) + slot * g.hnet; }
  __device__ inline float* z() const { return reinterpret_cast<float*>(base + g.oZ); }
  // per-row values: 0, 1 q of the two nets, 2 y, 3, 4 r and d, then dq of the two nets, 5 log pi,
  // 6 ring rows
  __device__ inline float* v(int i) const { return reinterpret_cast<float*>(base + g.oV) + i * 32 * g.tm; }
  __device__ inline uint16_t* m() const { return reinterpret_cast<uint16_t*>(base + g.oM); }
  __device__ inline f32x4* s() const { return reinterpret_cast<f32x4*>(base + g.oS); }
};

// Packed image of one 32-column block of X or H (a lane takes a column: bf16 by transposing
// LDS reads), with its column sums (part) and sums weighted by dq (wpart) over the tile's
// rows. saved: the image is there already and gives the sums. Reads what other waves wrote
// only past a barrier; a wave may pack a block that it has just stored.
template <typename T, int TM>
__device__ inline void pack_block(const T* src, int ld, int nblk, int cb, int64_t tile, void* image, float* part,
                                  float* wpart, const float* dq, bool saved, int lane) {
  constexpr int KS = RowT<T>::KS, G = 32 * TM / KS;
  const int half = lane >> 5;
  float sum = 0.0f, wsum = 0.0f;
  u32x4* dst = static_cast<u32x4*>(image) + (tile * G * nblk + cb) * 64 + lane;
#pragma unroll
  for (int f = 0; f < G; ++f) {
    u32x4 v;
    if (saved) {
      v = dst[f * nblk * 64];
    } else if constexpr (sizeof(T) == 2) {
      const int q = lane >> 4, i = lane & 15;
      const T* p = src + (f * 16 + 8 * (q >> 1) + (i >> 2)) * ld + cb * 32 + 16 * (q & 1) + 4 * (i & 3);
      const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_AS bf16x4*)(p));
      const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_AS bf16x4*)(p + 4 * ld));
      v = __builtin_bit_cast(u32x4, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    } else {
      const T* p = src + (f * 8 + 4 * half) * ld + cb * 32 + (lane & 31);
      v = __builtin_bit_cast(u32x4, f32x4{p[0], p[ld], p[2 * ld], p[3 * ld]});
    }
    if (!saved) dst[f * nblk * 64] = v;
    if (part) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if constexpr (sizeof(T) == 2)
          sum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, (uint32_t)v[e]), (bf16x2){1.0f, 1.0f}, sum, false);
        else
          sum += __builtin_bit_cast(f32x4, v)[e];
      }
    }
    if (wpart) {
      const float* d = dq + f * KS + KS / 2 * half;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if constexpr (sizeof(T) == 2)   // dq is in the operand type already
          wsum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, (uint32_t)v[e]),
                                                 __builtin_bit_cast(bf16x2, pack_bf16x2(d[2 * e], d[2 * e + 1])), wsum, false);
        else
          wsum = fmaf(d[e], __builtin_bit_cast(f32x4, v)[e], wsum);
      }
    }
  }
  const int64_t at = tile * (nblk * 32) + cb * 32 + lane;
  if (part) {
    sum += __shfl_xor(sum, 32);
    if (half == 0) part[at] = sum;
  }
  if (wpart) {
    wsum += __shfl_xor(wsum, 32);
    if (half == 0) wpart[at] = wsum;
  }
}

// One product operation on the wave's NB column blocks first, first + stride, ... over the
// steps s0 .. s1 - 1. part > 0: the sums go to LDS for the wave with part 0 of the same block.
template <typename T, int TM, int NB>
__device__ inline void product(const RowArgs& g, const RowOp& o, const Lds& L, int64_t tile, int net, int slot, int first,
                               int stride, int part, int group, int lane) {
  constexpr int KS = RowT<T>::KS;
  // Steps of weights in flight: a ring, each slot reloaded as soon as it is used (12 or 16
  // fragments instead of 8 gain nothing, 24 cost 4% on 400-300 fp32).
  constexpr int PD = 8 / NB;
  const int half = lane >> 5, r = lane & 31, k = net - o.net0;
  const int lda = o.from_h ? g.ldh : g.ldx;
  const int s0 = o.steps * part / o.split, s1 = o.steps * (part + 1) / o.split;
  const T* a = (o.from_h ? L.h<T>(slot) : L.x<T>()) + r * lda + (KS / 2) * half;
  const u32x4* w = static_cast<const u32x4*>(pick(o.w, k)) + first * o.steps * 64;
  const int ws = stride * o.steps * 64;
  u32x4 b[PD][NB];
  auto load = [&](int i, int s) {
    const u32x4* p = w + min(s, s1 - 1) * 64;   // uniform
#pragma unroll
    for (int j = 0; j < NB; ++j) b[i][j] = (p + j * ws)[lane];
  };
  f32x16 acc[TM][NB];
  auto multiply = [&](int i, int s) {
    u32x4 x[TM];
#pragma unroll
    for (int t = 0; t < TM; ++t) x[t] = *reinterpret_cast<const u32x4*>(a + t * 32 * lda + s * KS);
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int t = 0; t < TM; ++t) mma<T>(acc[t][j], b[i][j], x[t]);
  };
  // bf16: the bias starts the accumulators. fp32 adds it last, as the layer-by-layer products
  // do: both paths' pre-activations are the same bits, and so are their ReLU decisions.
  constexpr bool BIAS_FIRST = sizeof(T) == 2;
  const float* bias = part == 0 ? pick(o.bias, k) : nullptr;
  auto bias_run = [&](int j, int q) {
    return *reinterpret_cast<const f32x4*>(bias + (first + j * stride) * 32 + 8 * q + 4 * half);
  };
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    zero(acc[0][j]);
    if (BIAS_FIRST && bias) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 v = bias_run(j, q);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[0][j][4 * q + e] = v[e];
      }
    }
  }
#pragma unroll
  for (int t = 1; t < TM; ++t)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[t][j] = acc[0][j];
#pragma unroll
  for (int i = 0; i < PD; ++i) load(i, s0 + i);
  int s = s0;
  for (; s + PD < s1; s += PD) {
#pragma unroll
    for (int i = 0; i < PD; ++i) {
      multiply(i, s + i);
      load(i, s + PD + i);
    }
  }
#pragma unroll
  for (int i = 0; i < PD; ++i) {
    if (s + i >= s1) break;   // uniform
    multiply(i, s + i);
  }

  if (!BIAS_FIRST && bias) {
    static_assert(BIAS_FIRST || TM == 1, "one row block");
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 v = bias_run(j, q);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[0][j][4 * q + e] += v[e];
      }
  }

  if (o.split > 1) {   // one block per wave
    f32x4* buf = L.s() + group * (o.split - 1) * (256 * TM) + lane;
    if (part > 0) {
#pragma unroll
      for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          buf[((part - 1) * TM + t) * 256 + q * 64] =
              f32x4{acc[t][0][4 * q], acc[t][0][4 * q + 1], acc[t][0][4 * q + 2], acc[t][0][4 * q + 3]};
    }
    __syncthreads();
    if (part > 0) return;
    for (int p = 0; p < o.split - 1; ++p)
#pragma unroll
      for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 v = buf[(p * TM + t) * 256 + q * 64];
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[t][0][4 * q + e] += v[e];
        }
  } else if (o.from_h) {
    __syncthreads();   // every wave is done reading H before it is overwritten
  }
  if (o.kind == ROW_Z || o.kind == ROW_DACT) {
    const int zp = o.kind == ROW_DACT ? g.dp : g.zp;
    float* z = L.z() + (o.kind == ROW_DACT ? (net - 1) * 32 * TM * zp : 0) + r * zp;
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<f32x4*>(z + t * 32 * zp + (first + j * stride) * 32 + 8 * q + 4 * half) =
              f32x4{acc[t][j][4 * q], acc[t][j][4 * q + 1], acc[t][j][4 * q + 2], acc[t][j][4 * q + 3]};
    return;
  }
  uint16_t* mask = L.m() + o.mask + k * (o.nblk * TM * 64) + lane;
  T* H = L.h<T>(slot) + r * g.ldh;
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int t = 0; t < TM; ++t) {
      const int cb = first + j * stride;
      uint16_t* m = mask + (cb * TM + t) * 64;
      Block<T> v;
      if (o.kind == ROW_HIDDEN) {
        const uint32_t bits = relu_block<T>(acc[t][j], v);
        if (o.mask >= 0) *m = (uint16_t)bits;
      } else {   // ROW_DGRAD
        float x[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) x[q] = acc[t][j][q];
        mask_block<T>(x, *m, v);
      }
      store_block<T>(H + t * 32 * g.ldh + cb * 32, v, half);
    }
  if (pick(o.pack, k)) {
#pragma unroll
    for (int j = 0; j < NB; ++j)
      pack_block<T, TM>(L.h<T>(slot), g.ldh, o.nblk, first + j * stride, tile, pick(o.pack, k), pick(o.part, k), nullptr,
                        nullptr, false, lane);
  }
}

// Gradient of the last hidden layer from dq: H = dq w where the unit was active. For the
// critics' own gradients its packed image and column sums, and before it is overwritten the
// packed image of H with the output layer's weight-gradient sums (saved: the image is there).
template <typename T, int TM>
__device__ inline void output_backward(const RowArgs& g, const RowOp& o, const Lds& L, int64_t tile, int net, int slot,
                                       int first, int cnt, int stride, int lane) {
  const int k = net - o.net0, half = lane >> 5, r = lane & 31;
  const uint16_t* mask = L.m() + o.mask + k * (o.nblk * TM * 64) + lane;
  const float* dq = L.v(3 + net - 1) + r;
  const T* w = static_cast<const T*>(pick(o.w, k));
  T* H = L.h<T>(slot) + r * g.ldh;
  for (int j = 0; j < cnt; ++j) {
    const int cb = first + j * stride;
    if (pick(o.hpack, k))
      pack_block<T, TM>(L.h<T>(slot), g.ldh, o.nblk, cb, tile, pick(o.hpack, k), nullptr, pick(o.wpart, k),
                        L.v(3 + net - 1), o.flags != 0, lane);
    float wf[16];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const T* p = w + cb * 32 + 8 * q + 4 * half;
      if constexpr (sizeof(T) == 2) {
        const uint2 v = *reinterpret_cast<const uint2*>(p);
        wf[4 * q] = bf2f((bf16_t)(v.x & 0xFFFFu));
        wf[4 * q + 1] = bf2f((bf16_t)(v.x >> 16));
        wf[4 * q + 2] = bf2f((bf16_t)(v.y & 0xFFFFu));
        wf[4 * q + 3] = bf2f((bf16_t)(v.y >> 16));
      } else {
        const f32x4 v = *reinterpret_cast<const f32x4*>(p);
#pragma unroll
        for (int e = 0; e < 4; ++e) wf[4 * q + e] = v[e];
      }
    }
#pragma unroll
    for (int t = 0; t < TM; ++t) {
      const float d = dq[t * 32];
      float x[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) x[q] = d * wf[q];
      Block<T> v;
      mask_block<T>(x, mask[(cb * TM + t) * 64], v);
      store_block<T>(H + t * 32 * g.ldh + cb * 32, v, half);
    }
    if (pick(o.pack, k))
      pack_block<T, TM>(L.h<T>(slot), g.ldh, o.nblk, cb, tile, pick(o.pack, k), pick(o.part, k), nullptr, nullptr, false,
                        lane);
  }
}

// The tile's rows of the replay ring, sampled by Philox as in the layer-by-layer path's gather.
// A ring row's segments start on 16 bytes and are zero past their last element, and so are
// the operand's columns past each segment. The critic part also writes the batch to global
// memory, where only debug reads look at it. A launch of its own for this wrote the batch and
// read it back; without it a step of 2 x 64 fp32 at 256 rows takes 51 us (54), 2 x 256 bf16
// at 16384 rows of 3.2 KB 188 us (198: the rows' 43 MB are 9 us of memory time either way).
template <typename T, int TM>
__device__ inline void load_tile(const RowArgs& g, const RowOp& o, const Lds& L, int64_t tile, int tid) {
  constexpr int VEC = RowT<T>::VEC, BM = 32 * TM;
  int32_t* rows = reinterpret_cast<int32_t*>(L.v(6));   // ring row, -1 past the batch
  if (o.flags != ROW_LOAD_SA) {   // the first load of a part
    if (tid < BM) {
      const int64_t b = tile * BM + tid;
      int32_t row = -1;
      if (b < g.B) {
        row = (int32_t)mulhi32(philox_word(g.seed, (uint64_t)b, (uint32_t)(*g.step + 1), P_IDX, 0u), g.size);
        if (o.flags == ROW_LOAD_NEXT) {
          const uint8_t* src = g.ring + (uint32_t)row * g.row_bytes;
          const float r = *reinterpret_cast<const float*>(src + g.off_r), d = *reinterpret_cast<const float*>(src + g.off_d);
          L.v(3)[tid] = r;
          L.v(4)[tid] = d;
          g.r[b] = r;
          g.d[b] = d;
          g.idx[b] = row;
        }
      }
      rows[tid] = row;
    }
    __syncthreads();
  }
  const bool next = o.flags == ROW_LOAD_NEXT, act = o.flags == ROW_LOAD_SA;
  const int seg = next ? g.off_s2 : 0;
  const int ns = (g.O + VEC - 1) / VEC, na = act ? (g.A + VEC - 1) / VEC : 0, nk = g.Ka / VEC, nv = g.Kc / VEC;
  T* X = L.x<T>();
  T* copy = o.flags == ROW_LOAD_S ? nullptr : static_cast<T*>(next ? g.xs2 : g.xsa) + tile * BM * (int64_t)g.Kc;
  // Four reads of random rows in flight a thread: one at a time, each pays the whole latency of the memory.
  constexpr int D = 4;
  for (int v0 = tid; v0 < BM * nv; v0 += D * ROW_THREADS) {
    u32x4 x[D];
#pragma unroll
    for (int i = 0; i < D; ++i) {
      const int v = v0 + i * ROW_THREADS, r = v < BM * nv ? v / nv : 0, c = v - r * nv;
      const int32_t row = rows[r];   // an unsigned index; -1 is past the largest ring
      const bool s = c < ns, a = c >= nk && c < nk + na;
      // what is not there reads the ring's first bytes and is zero
      const uint8_t* src = g.ring;
      const bool on = v < BM * nv && row != -1 && (s || a);
      if (on) src += (uint32_t)row * g.row_bytes + (s ? seg + c * 16 : g.off_a + (c - nk) * 16);
      x[i] = *reinterpret_cast<const u32x4*>(src);
      if (!on) x[i] = {0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int i = 0; i < D; ++i) {
      const int v = v0 + i * ROW_THREADS;
      if (v < BM * nv) {
        const int r = v / nv, c = v - r * nv;
        if (copy && rows[r] != -1) *reinterpret_cast<u32x4*>(copy + (int64_t)v * VEC) = x[i];
        *reinterpret_cast<u32x4*>(X + r * g.ldx + c * VEC) = x[i];
      }
    }
  }
}

// The tile's sampler observations, four columns and four such pieces in flight a thread: a
// call for 256 of 376 columns on 64-64 bf16 takes 10 us, 16 with a column at a time, for 8192
// on 256-256 16 and 26. Rows of four-column multiples from a 16-byte address are read whole,
// others by the element.
template <typename T, int TM>
__device__ inline void load_obs(const RowArgs& g, const Lds& L, int64_t tile, int tid) {
  constexpr int BM = 32 * TM, D = 4;
  const bool whole = g.O % 4 == 0 && (reinterpret_cast<uintptr_t>(g.obs) & 15) == 0;
  const int nv = g.Ka / 4;
  T* X = L.x<T>();
  for (int v0 = tid; v0 < BM * nv; v0 += D * ROW_THREADS) {
    float x[D][4];
#pragma unroll
    for (int i = 0; i < D; ++i) {
      const int v = v0 + i * ROW_THREADS, r = v / nv, c = 4 * (v - r * nv);
      const int64_t b = tile * BM + r;
      const bool on = v < BM * nv && b < g.B;
      const float* src = g.obs + b * g.O + c;
#pragma unroll
      for (int e = 0; e < 4; ++e) x[i][e] = 0.0f;
      if (whole) {
        if (on && c < g.O) {
          const float4 f = *reinterpret_cast<const float4*>(src);
          x[i][0] = f.x; x[i][1] = f.y; x[i][2] = f.z; x[i][3] = f.w;
        }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (on && c + e < g.O) x[i][e] = src[e];
      }
    }
#pragma unroll
    for (int i = 0; i < D; ++i) {
      const int v = v0 + i * ROW_THREADS, r = v / nv, c = 4 * (v - r * nv);
      if (v >= BM * nv) continue;
      T* dst = X + r * g.ldx + c;
      if constexpr (sizeof(T) == 2)
        *reinterpret_cast<uint2*>(dst) = make_uint2(pack_bf16x2(x[i][0], x[i][1]), pack_bf16x2(x[i][2], x[i][3]));
      else
        *reinterpret_cast<float4*>(dst) = make_float4(x[i][0], x[i][1], x[i][2], x[i][3]);
    }
  }
}

// Sum over the wave's groups of LPR lanes (every lane of a group holds its value).
template <int LPR, typename V>
__device__ inline V group_sum(V v) {
#pragma unroll
  for (int m = LPR; m < 64; m <<= 1) v += __shfl_xor(v, m);
  return v;
}

// The critic output layer, LPR lanes per row of the tile, and what follows from q per row:
//   target       y = r + gamma (1 - d) (min(q1, q2) - alpha log pi)
//   critic loss  dq_i = 2 (q_i - y) / B in the operand type; sums of (q1 - y)^2, (q2 - y)^2,
//                q1 and each dq per wave
//   actor loss   SAC: dq = -1 / B to the smaller critic (critic 1 on ties), sums of
//                alpha log pi - min(q1, q2) and log pi; TD3: critic 1 only, sum of q1
// One operation, so that neither q nor y waits for a barrier of its own.
template <typename T, int TM>
__device__ inline void output_dot(const RowArgs& g, const RowOp& o, const Lds& L, int64_t tile, int tid) {
  constexpr int VEC = RowT<T>::VEC, LPR = ROW_THREADS / (32 * TM);
  const int l = tid % LPR, r = tid / LPR, K = o.nblk * 32;
  const int64_t b = tile * (32 * TM) + r;
  const bool live = b < g.B;
  float q[2] = {0.0f, 0.0f};
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    if (k >= o.nets) break;
    const T* h = L.h<T>(k) + r * g.ldh;
    const T* w = static_cast<const T*>(k ? o.w[1] : o.w[0]);
    float s = 0.0f;
#pragma unroll 4
    for (int c = l * VEC; c < K; c += LPR * VEC) {
      const u32x4 hv = *reinterpret_cast<const u32x4*>(h + c), wv = *reinterpret_cast<const u32x4*>(w + c);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if constexpr (sizeof(T) == 2)
          s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, (uint32_t)hv[e]),
                                              __builtin_bit_cast(bf16x2, (uint32_t)wv[e]), s, false);
        else
          s = fmaf(__builtin_bit_cast(f32x4, hv)[e], __builtin_bit_cast(f32x4, wv)[e], s);
      }
    }
#pragma unroll
    for (int m = LPR / 2; m > 0; m >>= 1) s += __shfl_xor(s, m);
    q[k] = s + *(k ? o.bias[1] : o.bias[0]);
  }
  if (o.flags == ROW_DOT_ONLY) {   // critic 1 of two that run one after the other
    if (l == 0) L.v(0)[r] = q[0];
    return;
  }
  if (o.nets == 1 && o.net0 == 2) {
    q[1] = q[0];
    q[0] = L.v(0)[r];
  }
  const bool first = l == 0;
  if (o.flags == ROW_DOT_TARGET) {
    float m = min_keep_nan(q[0], q[1]);
    if (g.sac) m -= expf(*g.log_alpha) * L.v(5)[r];
    const float y = live ? L.v(3)[r] + g.gamma * (1.0f - L.v(4)[r]) * m : 0.0f;   // r, d of the load
    if (first) L.v(2)[r] = y;
    if (first && live) g.y[b] = y;
    return;
  }
  const int64_t at = tile * ROW_WAVES + (tid >> 6);
  float d1 = 0.0f, d2 = 0.0f;
  if (o.flags == ROW_DOT_CLOSS) {
    double e1s = 0.0, e2s = 0.0, q1s = 0.0;
    if (live) {
      const float y = L.v(2)[r];
      const float e1 = q[0] - y, e2 = q[1] - y;
      d1 = to_f<T>(from_f<T>(2.0f * e1 / (float)g.B));
      d2 = to_f<T>(from_f<T>(2.0f * e2 / (float)g.B));
      e1s = (double)e1 * e1;
      e2s = (double)e2 * e2;
      q1s = q[0];
    }
    if (first && live) {
      g.q1[b] = q[0];
      g.q2[b] = q[1];
    }
    if (first) {
      L.v(3)[r] = d1;
      L.v(4)[r] = d2;
    }
    e1s = group_sum<LPR>(e1s);
    e2s = group_sum<LPR>(e2s);
    q1s = group_sum<LPR>(q1s);
    d1 = group_sum<LPR>(d1);
    d2 = group_sum<LPR>(d2);
    if ((tid & 63) == 0) {
      g.cpart[at * 3 + 0] = e1s;
      g.cpart[at * 3 + 1] = e2s;
      g.cpart[at * 3 + 2] = q1s;
      o.part[0][at] = d1;
      o.part[1][at] = d2;
    }
    return;
  }
  double l0 = 0.0, l1 = 0.0;
  if (live) {
    const float inv = to_f<T>(from_f<T>(-1.0f / (float)g.B));
    if (g.sac) {
      const float lp = L.v(5)[r];
      const bool take1 = q[0] <= q[1];
      d1 = take1 ? inv : 0.0f;
      d2 = take1 ? 0.0f : inv;
      l0 = (double)expf(*g.log_alpha) * lp - (double)(take1 ? q[0] : q[1]);
      l1 = lp;
    } else {
      d1 = inv;
      l0 = q[0];
    }
  }
  if (first && live) {
    g.qp1[b] = q[0];
    if (g.sac) g.qp2[b] = q[1];
  }
  if (first) {
    L.v(3)[r] = d1;
    L.v(4)[r] = d2;
  }
  l0 = group_sum<LPR>(l0);
  l1 = group_sum<LPR>(l1);
  if ((tid & 63) == 0) {
    g.apart[at * 2 + 0] = l0;
    g.apart[at * 2 + 1] = l1;
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
// output gradient in H.
template <typename T, int TM>
__device__ inline void head_backward(const RowArgs& g, const RowOp& o, const Lds& L, int64_t tile, int tid) {
  constexpr int BM = 32 * TM;
  T* H = L.h<T>(0);
  const float* D = L.z();
  const float aB = g.sac ? expf(*g.log_alpha) / (float)g.B : 0.0f;
  // both outputs of an (row, action) element; the columns past the outputs are zero
  for (int e = tid; e < BM * g.A; e += ROW_THREADS) {
    const int r = e / g.A, j = e - r * g.A;
    const int64_t b = tile * BM + r;
    float gm = 0.0f, gl = 0.0f;
    if (b < g.B) {
      const uint64_t i = (uint64_t)b * g.A + j;
      const float a = g.th[i];
      float da = D[r * g.dp + j];
      if (g.sac) {
        const float se = g.se[i], lm = g.lm[i];
        da += D[(BM + r) * g.dp + j];
        gm = da * (1.0f - a * a) + aB * 2.0f * a;
        gl = (gm * se - aB) * lm;
      } else {
        gm = da * (1.0f - a * a);
      }
      g.da[b * g.Ap + j] = da;
    }
    H[r * g.ldh + j] = from_f<T>(gm);
    if (g.sac) H[r * g.ldh + g.A + j] = from_f<T>(gl);
  }
  const int used = g.sac ? 2 * g.A : g.A, rest = g.pa - used;
  for (int e = tid; e < BM * rest; e += ROW_THREADS) H[e / rest * g.ldh + used + e % rest] = from_f<T>(0.0f);
}

// Brings the operation list and the packed images into the L2 of the workgroup's XCD, which
// starts a launch without them: each operation would wait for its record and then for its
// weights from beyond L2. Workgroup b runs on XCD b % 8; those of an XCD share the lines, a word
// of each a lane. The loads run beside the first operation's; t holds them until it is done.
constexpr int WARM = 4;
__device__ inline void warm_l2(const RowArgs& g, int part, int tid, uint32_t (&t)[WARM + 1]) {
  const int n = max(1, (int)gridDim.x / 8), id = blockIdx.x / 8, lines = g.warm_lines;
  const int bytes = g.nops[part] * (int)sizeof(RowOp);
  t[WARM] = 0;
  if (tid * 128 < bytes) t[WARM] = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const uint8_t*>(g.ops + g.op0[part]) + tid * 128);
#pragma unroll
  for (int i = 0; i < WARM; ++i) {
    const int v = (i * n + id) * ROW_THREADS + tid;
    const int w = (v >= lines) + (v >= 2 * lines);
    t[i] = 0;
    if (id < n && v < 3 * lines) t[i] = *reinterpret_cast<const uint32_t*>(g.warm[w] + (int64_t)(v - w * lines) * 128);
  }
}

// Sampler actions from the actor's output in Z.
template <typename T, int TM>
__device__ inline void sampler_actions(const RowArgs& g, const Lds& L, int64_t tile, int tid) {
  constexpr int BM = 32 * TM;
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
}

// ACT: sampler actions, a kernel of their own so that neither's operations press on the other's
// registers (in one kernel: 24 bytes of scratch in float32, or 2% of a step of 400-300 (TD3) at 32768
// rows in other arrangements of the same code).
// 32-row tiles: 128 registers, two workgroups per CU where their LDS allows it (where it does
// not, 155 registers are slower: 400-300 fp32 1067 against 1028 us); 64-row tiles take the LDS
// of a CU.
template <typename T, int TM, bool ACT>
__global__ void __launch_bounds__(ROW_THREADS, TM == 1 ? 4 : 2) k_rows(RowArgs args) {
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int part = (int)blockIdx.x >= args.tiles ? 1 : 0;
  const int64_t tile = (int)blockIdx.x - part * args.tiles;
  const CONST_AS RowArgs* argp = (const CONST_AS RowArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  const CONST_AS RowOp* op = (const CONST_AS RowOp*)(uintptr_t)(args.ops + args.op0[part]);
  for (int n = args.nops[part]; n > 0; --n, ++op) {
    const RowArgs& g = *opaque(argp);
    const RowOp& o = *opaque(op);
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));   // (as for the pointers: no per-lane values kept across operations)
    const int lane = tid & 63;
    const Lds L{smem, g};
    // The wave's share of the operation's column blocks: blocks first, first + wpn, ... of
    // one net, or (split) a range of the steps of one block.
    const int wpn = o.nets == 2 ? ROW_WAVES / 2 : ROW_WAVES;
    const int k = wave / wpn, i = wave - k * wpn;
    const int net = o.net0 + k, slot = o.nets == 2 ? k : 0;
    // Blocks of the second net start at the other end: with few blocks both nets' waves
    // would otherwise share matrix cores (wave w runs on SIMD w % 4).
    const int turn = k ? wpn - 1 - i : i;
    int first = turn, kpart = 0;
    if (o.split > 1) {
      first = turn % o.nblk;
      kpart = turn / o.nblk;
    }
    const int cnt = o.split > 1 ? (kpart < o.split ? 1 : 0) : o.nblk > first ? (o.nblk - 1 - first) / wpn + 1 : 0;
    switch (o.kind) {
      case ROW_HIDDEN: case ROW_Z: case ROW_DGRAD: case ROW_DACT: {
        const int group = slot * o.nblk + first;
        if (cnt == 1) product<T, TM, 1>(g, o, L, tile, net, slot, first, wpn, kpart, group, lane);
        else if (cnt == 2) product<T, TM, 2>(g, o, L, tile, net, slot, first, wpn, 0, group, lane);
        else if (cnt == 3) product<T, TM, 3>(g, o, L, tile, net, slot, first, wpn, 0, group, lane);
        else if (cnt == 4) product<T, TM, 4>(g, o, L, tile, net, slot, first, wpn, 0, group, lane);
        else if (o.split > 1 || o.from_h) __syncthreads();
        break;
      }
      case ROW_LOAD:
        if constexpr (!ACT) {
          uint32_t t[WARM + 1];
          const bool warm = g.warm_lines > 0 && o.flags != ROW_LOAD_SA;
          if (warm) warm_l2(g, part, tid, t);
          load_tile<T, TM>(g, o, L, tile, tid);
          if (warm) {
#pragma unroll
            for (int i = 0; i <= WARM; ++i) asm volatile("" ::"v"(t[i]));
          }
        }
        break;
      case ROW_OBS: if constexpr (ACT) load_obs<T, TM>(g, L, tile, tid); break;
      case ROW_DOT: if constexpr (!ACT) output_dot<T, TM>(g, o, L, tile, tid); break;
      case ROW_DZ: if constexpr (!ACT) output_backward<T, TM>(g, o, L, tile, net, slot, first, cnt, wpn, lane); break;
      case ROW_PACK:
        if constexpr (!ACT)
          for (int cb = wave; cb < o.nblk; cb += ROW_WAVES)
            pack_block<T, TM>(o.from_h ? L.h<T>(0) : L.x<T>(), o.from_h ? g.ldh : g.ldx, o.nblk, cb, tile, o.pack[0],
                              o.part[0], nullptr, nullptr, false, lane);
        break;
      case ROW_HEAD: if constexpr (!ACT) head<T, TM>(g, o, L, tile, tid); break;
      case ROW_HEAD_BWD: if constexpr (!ACT) head_backward<T, TM>(g, o, L, tile, tid); break;
      case ROW_ACT: if constexpr (ACT) sampler_actions<T, TM>(g, L, tile, tid); break;
    }
    if (o.kind != ROW_PACK) __syncthreads();   // what a pack reads is overwritten only past a later barrier
  }
}

// ------------------------------------------------------------------------------ weight gradients
// One wave takes 2 x 2 blocks of a product over one slice of the batch, fragments straight
// from memory into registers: no LDS, no barriers. The four waves of a workgroup and its
// neighbours on the same XCD take neighbouring tiles of the same slice, which share fragments.
// float32 runs on split operands (from ROW_SPLIT_ROWS rows on): 400-300 (TD3) at 32768 rows 272 us
// for a launch of actor and critics and 182 for the critics' (float32 instructions 484 and 340), 2 x
// 256 at 8192 rows 40 us (48); small parts on the main accumulators took 275, 172 and 36, further from
// 64 bits than the float32 instructions (mma_split). bf16 is bound by
// L2: 46 us for 550 MB at 2 x 256 (376 inputs), 16384 rows. (4 x 2 blocks a wave, 96 instead of
// 128 bytes a block and row, is slower in both: the registers leave too little in flight.)
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
  const int pairs = W.groups / 2;   // (a multiple of 32 rows)
  const int g0 = 2 * (int)((int64_t)pairs * slice / J.slices), g1 = 2 * (int)((int64_t)pairs * (slice + 1) / J.slices);
  const u32x4* a = static_cast<const u32x4*>(J.a) + (int64_t)m0 * 64 + lane;
  const u32x4* b = static_cast<const u32x4*>(J.b) + (int64_t)n0 * 64 + lane;
  const int64_t as = (int64_t)J.mblk * 64, bs = (int64_t)J.bcb * 64;
  const int am = m2 ? 64 : 0, bn = n2 ? 64 : 0;
  f32x16 acc[2][2];
  auto clear = [&] {
#pragma unroll
    for (int i = 0; i < 4; ++i) zero(acc[i >> 1][i & 1]);
  };
  clear();
  // Row groups in flight, twice: the float32 sums on split operands need the registers.
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
  auto run = [&](auto&& multiply) {
    if (g0 >= g1) return;
    load(f0, g0);
    for (int gr = g0; gr < g1; gr += 2 * PD) {
      if (gr + PD < g1) load(f1, gr + PD);
      multiply(f0, gr);
      if (gr + 2 * PD < g1) load(f0, gr + 2 * PD);
      if (gr + PD < g1) multiply(f1, gr + PD);
    }
  };
  auto exact = [&](const u32x4 (&f)[PD][4], int gr) {
#pragma unroll
    for (int i = 0; i < PD; ++i) {
      if (gr + i >= g1) break;
#pragma unroll
      for (int x = 0; x < 4; ++x) mma<T>(acc[x >> 1][x & 1], f[i][x >> 1], f[i][2 + (x & 1)]);
    }
  };
  if (sizeof(T) == 2 || !W.split) {
    run(exact);
  } else if constexpr (sizeof(T) == 4) {
    // two row groups at a time on split operands (a slice has an even number of them)
    f32x16 lo[2][2];
#pragma unroll
    for (int x = 0; x < 4; ++x) zero(lo[x >> 1][x & 1]);
    run([&](const u32x4 (&f)[PD][4], int) {
      const Split A[2] = {split(f[0][0], f[1][0]), split(f[0][1], f[1][1])};
      const Split B[2] = {split(f[0][2], f[1][2]), split(f[0][3], f[1][3])};
#pragma unroll
      for (int x = 0; x < 4; ++x) mma_split(acc[x >> 1][x & 1], lo[x >> 1][x & 1], A[x >> 1], B[x & 1]);
    });
    float bad = 0.0f;   // NaN once a sum is an infinity or NaN
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      f32x16& c = acc[x >> 1][x & 1];
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        c[q] = (c[q] + lo[x >> 1][x & 1][q]) * (1.0f / (SPLIT_SCALE * SPLIT_SCALE));
        bad = fmaf(c[q], 0.0f, bad);
      }
    }
    if (__any(bad != bad)) {
      clear();   // infinities, NaN or sums past the scaled range: again in float32
      run(exact);
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
  __shared__ double sh[1024];
  const AdamArgs& a = p.a;
  const RowPBlk B = p.blk[p.first + blockIdx.x];
  T* PF = static_cast<T*>(p.PF);
  T* PT = static_cast<T*>(p.PT);
  T* TF = static_cast<T*>(p.TF);
  const int tid = threadIdx.x;
  // Thread of a weight block: column n, rows m0 .. m0 + 3 (accumulator order).
  const int lane = tid & 63, n = lane & 31, m0 = 8 * (tid >> 6) + 4 * (lane >> 5);
  if (!p.update) {
    if (B.kind == 1 && B.fwd >= 0 && tid < 16) {
      PF[B.fwd + tid] = from_f<T>(a.P[B.off + tid]);
      TF[B.fwd + tid] = from_f<T>(a.T[B.off + tid]);
    }
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
  // A parameter's state is read before its slices are summed: one memory latency, not two (2 x
  // 64 fp32 7.7 -> 6.7 us, 2 x 256 bf16 13.0 -> 11.7, 200-120 fp32 19.8 -> 17.0 in two launches).
  struct Old { float p, m, v, t; };
  auto old = [&](int64_t i) { return Old{a.P[i], a.M[i], a.V[i], polyak ? a.T[i] : 0.0f}; };
  auto element = [&](int64_t i, Old o, float g, float& t) {
    a.G[i] = g;
    const float x = adam_element(a, o.p, o.m, o.v, g, lr, bc[actor ? 2 : 0], bc[actor ? 3 : 1]);
    a.M[i] = o.m;
    a.V[i] = o.v;
    a.P[i] = x;
    if (polyak) {
      t = polyak_element(a, o.t, x);
      a.T[i] = t;
    }
    return x;
  };
  float t;
  if (B.kind == 0) {
    const RowPJob J = p.j[B.job];
    const float4* src = reinterpret_cast<const float4*>(J.part) + (int64_t)B.blk * 256 + tid;
    const int64_t zs = J.zstride / 4;
    Old o[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = old(B.off + (int64_t)(m0 + j) * B.ld + n);
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
    for (int j = 0; j < 4; ++j) v[j] = element(B.off + (int64_t)(m0 + j) * B.ld + n, o[j], g[j], u[j]);
    store_packed<T>(PF, PT, B, m0, n, v);
    if (polyak) store_packed<T>(TF, nullptr, B, m0, n, u);
    return;
  }
  if (B.kind == 1) {
    // 16 columns as 4 pieces of 4, each summed by 64 threads over every 64th slice, then
    // the thread sums in order; in double precision, as there may be thousands of slices.
    const int piece = tid & 3, grp = tid >> 2;
    const float* src = B.part + 4 * piece;
    Old o{};
    if (tid < 16) o = old(B.off + tid);
    double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int z = grp; z < p.vslices; z += 64) {
      const float4 v = *reinterpret_cast<const float4*>(src + (int64_t)z * B.ld);
      s[0] += v.x; s[1] += v.y; s[2] += v.z; s[3] += v.w;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) sh[grp * 16 + 4 * piece + e] = s[e];
    __syncthreads();
    if (tid >= 16) return;
    double g = 0.0;
    for (int q = 0; q < 64; ++q) g += sh[q * 16 + tid];
    const float x = element(B.off + tid, o, (float)g, t);
    if (B.fwd >= 0) {
      PF[B.fwd + tid] = from_f<T>(x);
      if (polyak) TF[B.fwd + tid] = from_f<T>(t);
    }
    return;
  }
  if (B.kind == 2) {
    double s = 0.0;
    for (int z = tid; z < p.vslices * ROW_WAVES; z += 256) s += B.part[z];
    s = block_sum<256>(s, sh);
    if (tid != 0) return;
    element(B.off, old(B.off), (float)s, t);
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

template <typename T, int TM>
hipError_t prepare_rows_t() {
  for (const void* f : {(const void*)(k_rows<T, TM, false>), (const void*)(k_rows<T, TM, true>)}) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <typename T, int TM>
hipError_t launch_rows_t(const RowArgs& g, size_t lds, hipStream_t s) {
  if (g.obs) (k_rows<T, TM, true>)<<<g.tiles * g.parts, ROW_THREADS, lds, s>>>(g);
  else (k_rows<T, TM, false>)<<<g.tiles * g.parts, ROW_THREADS, lds, s>>>(g);
  return hipGetLastError();
}

}  // namespace

hipError_t prepare_rows(bool bf16) {
  if (!bf16) return prepare_rows_t<float, 1>();
  const hipError_t e = prepare_rows_t<bf16_t, 1>();
  return e == hipSuccess ? prepare_rows_t<bf16_t, 2>() : e;
}

hipError_t launch_rows(bool bf16, const RowArgs& g, size_t lds, hipStream_t s) {
  if (g.tiles < 1 || g.parts < 1 || g.parts > 2 || lds > 160 * 1024 || (g.tm != 1 && g.tm != 2) ||
      (!bf16 && g.tm != 1) || (int64_t)g.tiles * 32 * g.tm < g.B)
    return hipErrorInvalidValue;
  if (!bf16) return launch_rows_t<float, 1>(g, lds, s);
  return g.tm == 1 ? launch_rows_t<bf16_t, 1>(g, lds, s) : launch_rows_t<bf16_t, 2>(g, lds, s);
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
