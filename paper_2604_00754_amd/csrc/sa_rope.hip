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

// X, Xout: [heads][n][d].  Thread (m, c) owns elements 8c .. 8c+7 of position m, so that the threads of a row read and write it as
// one contiguous piece (a thread that owned both halves of its pairs touched half rows, 128-byte lines asked for twice: 16 x 16
// heads, n = 4096, d = 64 59 against 47 us = 5.8 TB/s; 4 heads, n = 131 072, d = 128 58 against 52 us).
//   adjacent pairs: they are pairs 4c .. 4c+3;
//   split halves: the other members of their pairs are the 8 elements of the thread half a row away in the wave.
template <typename T, bool INTERLEAVED>
__global__ __launch_bounds__(ROPE_THREADS) void rope_apply_kernel(const T* __restrict__ X, T* __restrict__ Xout,
                                                                   const float2* __restrict__ table, int heads, int n,
                                                                   int d, int inverse) {
  const int cpr = d / 8;  // threads per row: 8 or 16, whole rows to a wave
  const long t = (long)blockIdx.x * ROPE_THREADS + threadIdx.x;
  const bool live = t < (long)n * cpr;  // (every lane takes part in the exchange)
  const int m = live ? (int)(t / cpr) : n - 1, c = (int)(t % cpr);
  constexpr int NPAIR = INTERLEAVED ? 4 : 8;
  const bool second = !INTERLEAVED && c >= cpr / 2;  // holds the second members of its pairs
  float cs[NPAIR], sn[NPAIR];
  {
    const float4* tp = reinterpret_cast<const float4*>(table + (size_t)m * (d / 2) + NPAIR * (second ? c - cpr / 2 : c));
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

template <typename T>
hipError_t launch_apply(const void* X, void* Xout, const float* table, int heads, int n, int d, int interleaved,
                        int inverse, hipStream_t st) {
  const long threads = (long)n * (d / 8);
  dim3 grid((unsigned)((threads + ROPE_THREADS - 1) / ROPE_THREADS),
            (unsigned)((heads + ROPE_HEADS_PER_BLOCK - 1) / ROPE_HEADS_PER_BLOCK));
  const float2* tb = reinterpret_cast<const float2*>(table);
  if (interleaved)
    rope_apply_kernel<T, true><<<grid, ROPE_THREADS, 0, st>>>((const T*)X, (T*)Xout, tb, heads, n, d, inverse);
  else
    rope_apply_kernel<T, false><<<grid, ROPE_THREADS, 0, st>>>((const T*)X, (T*)Xout, tb, heads, n, d, inverse);
  return hipGetLastError();
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
  return bf16 ? launch_apply<uint16_t>(X, Xout, table, heads, n, d, interleaved, inverse, st)
              : launch_apply<float>(X, Xout, table, heads, n, d, interleaved, inverse, st);
}

}  // namespace sa
