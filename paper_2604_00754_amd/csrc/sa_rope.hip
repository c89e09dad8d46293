// Rotary position embeddings on ORIGINAL token positions (App. B, "Attention" item; App. C, training
// paragraph; Sec. 4.2): Q and K are rotated with the position each token has in the sequence before
// any shuffling, so the permutation never enters here.  RoFormer Sec. 3.2.2: pair i of the row at
// position m turns by m * base^(-2i/d).
//
// Two kernels.  The table kernel evaluates (cos, sin) of every (position, pair) once, in fp64 (the
// angle reaches 10^5 rad at long prefill, beyond what an fp32 product resolves), and stores them as
// fp32.  The apply kernel streams rows: one thread owns the same 8 elements of one position for several
// heads, keeps the table values of their pairs in registers, and reads / writes 16 B (bf16) per head.
// HBM-bound: 2 * sizeof(T) bytes per element, the table stays in cache.
#include "sa_common.h"
#include "sa_device.h"

namespace sa {
namespace {

constexpr int ROPE_THREADS = 256;
constexpr int ROPE_HEADS_PER_BLOCK = 4;

__global__ __launch_bounds__(ROPE_THREADS) void rope_table_kernel(float2* __restrict__ table, int n, int half,
                                                                   double base, int pos0) {
  const long i = (long)blockIdx.x * ROPE_THREADS + threadIdx.x;
  if (i >= (long)n * half) return;
  const int m = (int)(i / half), pair = (int)(i % half);
  const double theta = pow(base, -(double)pair / (double)half);  // base^(-2 pair / d)
  double s, c;
  sincos((double)(pos0 + m) * theta, &s, &c);
  table[i] = make_float2((float)c, (float)s);
}

template <typename T>
struct Row8;

template <>
struct Row8<uint16_t> {  // 8 bf16 = 16 bytes
  static __device__ __forceinline__ void load(const uint16_t* p, float* x) {
    const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));  // streamed once
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      x[2 * j] = bf16lo(v[j]);
      x[2 * j + 1] = bf16hi(v[j]);
    }
  }
  static __device__ __forceinline__ void store(uint16_t* p, const float* x) {
    u32x4 v;
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = pack_bf16(x[2 * j], x[2 * j + 1]);
    __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p));
  }
};

template <>
struct Row8<float> {
  static __device__ __forceinline__ void load(const float* p, float* x) {
    const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
    x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
    x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
  }
  static __device__ __forceinline__ void store(float* p, const float* x) {
    *reinterpret_cast<float4*>(p) = make_float4(x[0], x[1], x[2], x[3]);
    *reinterpret_cast<float4*>(p + 4) = make_float4(x[4], x[5], x[6], x[7]);
  }
};

// Whether a thread owns both members of its split pairs: the halves of a row are whole 128-byte lines.
template <typename T, int d, bool INTERLEAVED>
constexpr bool rope_both_halves() {
  return !INTERLEAVED && d / 2 * sizeof(T) >= 128;
}

// X, Xout: [heads][n][d].  A thread owns 8 pairs of a position or 8 neighbouring elements, so that what neighbouring threads touch
// with one load is a contiguous piece of whole 128-byte lines:
//   adjacent pairs: elements 8c .. 8c+7, pairs 4c .. 4c+3, a row as one piece (32 heads, n = 32768, d = 128, with K of 8 heads:
//     116 us against 145 with 16 elements to a thread);
//   split halves of a line or more (fp32, or d = 128): elements 8c .. 8c+7 of both halves, pairs 8c .. 8c+7;
//   split halves of half a line (bf16, d = 64): elements 8c .. 8c+7, a row as one piece, and the other members of their pairs from the
//     thread half a row away in the wave.  As both halves per thread, lines were asked for twice: 16 x 16 heads, n = 4096, Q and K
//     115 against 90 us.
// The exchange does not pay where the halves are lines already: one tensor at d = 128 in bf16 of 32 x 1 x 17379 rows 53.4 against 50.0 us,
// 912 x 147 15.5 against 14.2, 32 x 131072 415 against 382 (256 x 4096 90.6 against 94.6), in fp32 32 x 8192 45.9 against 43.9.
template <typename T, int d, bool INTERLEAVED>
__global__ __launch_bounds__(ROPE_THREADS) void rope_apply_kernel(const T* __restrict__ X, T* __restrict__ Xout,
                                                                   const float2* __restrict__ table, int heads, int n,
                                                                   int inverse) {
  constexpr bool BOTH = rope_both_halves<T, d, INTERLEAVED>();
  constexpr int cpr = BOTH ? d / 16 : d / 8;  // threads per row: 4, 8 or 16, whole rows to a wave
  constexpr int NPAIR = INTERLEAVED ? 4 : 8;
  const long t = (long)blockIdx.x * ROPE_THREADS + threadIdx.x;
  const bool live = t < (long)n * cpr;  // (every lane takes part in the exchange)
  const int m = live ? (int)(t / cpr) : n - 1, c = (int)(t % cpr);
  const bool second = !INTERLEAVED && !BOTH && c >= cpr / 2;  // holds the second members of its pairs
  float cs[NPAIR], sn[NPAIR];
  {
    const table_float4* tp = reinterpret_cast<const table_float4*>(table + (size_t)m * (d / 2) + NPAIR * (second ? c - cpr / 2 : c));
#pragma unroll
    for (int j = 0; j < NPAIR / 2; ++j) {
      const float4 v = tp[j];
      cs[2 * j] = v.x; sn[2 * j] = v.y;
      cs[2 * j + 1] = v.z; sn[2 * j + 1] = v.w;
    }
    if ((inverse != 0) != second) {  // first members: u cos - v sin; second: v cos + u sin; the inverse turns the signs
#pragma unroll
      for (int j = 0; j < NPAIR; ++j) sn[j] = -sn[j];
    }
  }
  const int h0 = blockIdx.y * ROPE_HEADS_PER_BLOCK;
  const int h1 = min(h0 + ROPE_HEADS_PER_BLOCK, heads);
  if constexpr (BOTH) {
    if (!live) return;
    for (int h = h0; h < h1; ++h) {
      const size_t at = ((size_t)h * n + m) * d + 8 * c;
      float u[8], v[8], ou[8], ov[8];
      Row8<T>::load(X + at, u);
      Row8<T>::load(X + at + d / 2, v);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        ou[j] = u[j] * cs[j] - v[j] * sn[j];
        ov[j] = u[j] * sn[j] + v[j] * cs[j];
      }
      Row8<T>::store(Xout + at, ou);
      Row8<T>::store(Xout + at + d / 2, ov);
    }
  } else {
#pragma unroll 4
    for (int h = h0; h < h1; ++h) {
      const size_t at = ((size_t)h * n + m) * d + 8 * c;
      float x[8], o[8];
      Row8<T>::load(X + at, x);
      if (INTERLEAVED) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          o[2 * j] = x[2 * j] * cs[j] - x[2 * j + 1] * sn[j];
          o[2 * j + 1] = x[2 * j] * sn[j] + x[2 * j + 1] * cs[j];
        }
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const float other = __shfl_xor(x[j], cpr / 2);
          o[j] = x[j] * cs[j] - other * sn[j];
        }
      }
      if (live) Row8<T>::store(Xout + at, o);
    }
  }
}

template <typename T, int d, bool INTERLEAVED>
hipError_t launch_apply(const void* X, void* Xout, const float* table, int heads, int n, int inverse, hipStream_t st) {
  const long threads = (long)n * (rope_both_halves<T, d, INTERLEAVED>() ? d / 16 : d / 8);
  dim3 grid((unsigned)((threads + ROPE_THREADS - 1) / ROPE_THREADS),
            (unsigned)((heads + ROPE_HEADS_PER_BLOCK - 1) / ROPE_HEADS_PER_BLOCK));
  rope_apply_kernel<T, d, INTERLEAVED><<<grid, ROPE_THREADS, 0, st>>>(
      (const T*)X, (T*)Xout, reinterpret_cast<const float2*>(table), heads, n, inverse);
  return hipGetLastError();
}

template <typename T, int d>
hipError_t launch_apply(const void* X, void* Xout, const float* table, int heads, int n, int interleaved,
                        int inverse, hipStream_t st) {
  return interleaved ? launch_apply<T, d, true>(X, Xout, table, heads, n, inverse, st)
                     : launch_apply<T, d, false>(X, Xout, table, heads, n, inverse, st);
}

}  // namespace

hipError_t launch_rope_table(float* table, int n, int d, double base, int pos0, hipStream_t st) {
  const long total = (long)n * (d / 2);
  rope_table_kernel<<<(unsigned)((total + ROPE_THREADS - 1) / ROPE_THREADS), ROPE_THREADS, 0, st>>>(
      reinterpret_cast<float2*>(table), n, d / 2, base, pos0);
  return hipGetLastError();
}

hipError_t launch_rope_apply(const void* X, void* Xout, const float* table, int heads, int n, int d, int bf16,
                             int interleaved, int inverse, hipStream_t st) {
  if (heads > 65535 * ROPE_HEADS_PER_BLOCK) return hipErrorNotSupported;
  if (d == 64)
    return bf16 ? launch_apply<uint16_t, 64>(X, Xout, table, heads, n, interleaved, inverse, st)
                : launch_apply<float, 64>(X, Xout, table, heads, n, interleaved, inverse, st);
  if (d != 128) return hipErrorNotSupported;
  return bf16 ? launch_apply<uint16_t, 128>(X, Xout, table, heads, n, interleaved, inverse, st)
              : launch_apply<float, 128>(X, Xout, table, heads, n, interleaved, inverse, st);
}

}  // namespace sa
