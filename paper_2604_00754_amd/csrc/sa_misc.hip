// Element-wise helpers of libsa: permutation check, zero fill, permutation sampling, and the gated backward's preparation
// pass (the chain rule through the two sigmoid gates of Eq. 5, and D = rowsum(dO * O) of both branches).
#include "sa_common.h"
#include "sa_device.h"

namespace sa {
namespace {

__global__ void fill_zero_kernel(uint32_t* p, size_t words) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < words; i += stride) p[i] = 0u;
}

// seen[slice][v] counts how often value v occurs in the slice; any count other than one, or a value
// outside 0..n-1, raises the flag.
__global__ void check_perm_kernel(const int32_t* __restrict__ perm, size_t total, int n, int* seen, int* flag) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < total; i += stride) {
    const int v = perm[i];
    if (v < 0 || v >= n) {
      atomicOr(flag, 1);
    } else if (atomicAdd(&seen[(i / n) * n + v], 1) != 0) {
      atomicOr(flag, 1);
    }
  }
}

// The gather and the scatter of Alg. 1 without the attention in between (a measurement helper: the
// ceiling for rows of 2*d bytes addressed through the index tensor).  One group of LPR lanes per
// (b, hq, slot): Y[perm[p]] = Q[perm[p]] (+ K[perm[p]] + V[perm[p]] for the first query head of a KV
// group, so that every K and V row is read once per group as in the attention kernels).  Four rows
// per thread are in flight.
template <int LPR>
__global__ __launch_bounds__(256) void permuted_copy_bf16_kernel(const Pass p, const long rows) {
  constexpr int RPT = 4;
  const int sub = threadIdx.x % LPR;
  const long group = ((long)blockIdx.x * 256 + threadIdx.x) / LPR;
  const long groups = (long)gridDim.x * 256 / LPR;
  const int d = LPR * 8;
  for (long r0 = group; r0 < rows; r0 += groups * RPT) {
    long r[RPT];
    int src[RPT];
    bool ok[RPT];
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
      r[j] = r0 + j * groups;
      ok[j] = r[j] < rows;
      const long rr = ok[j] ? r[j] : 0;
      const int slot = (int)(rr % p.n);
      const long bh = rr / p.n;
      const int hq = (int)(bh % p.Hq), b = (int)(bh / p.Hq);
      src[j] = p.perm ? p.perm[(size_t)perm_slice_index(p.perm_B, p.perm_H, b, hq) * p.n + slot] : slot;
    }
    u32x4 q[RPT], k[RPT], v[RPT];
    bool lead[RPT];
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
      const long rr = ok[j] ? r[j] : 0;
      const long bh = rr / p.n;
      const int hq = (int)(bh % p.Hq), b = (int)(bh / p.Hq);
      lead[j] = hq % p.g == 0;
      const size_t qoff = ((size_t)bh * p.n + src[j]) * d + sub * 8;
      const size_t koff = (((size_t)b * p.Hkv + hq / p.g) * p.n + src[j]) * d + sub * 8;
      // every row is touched once: non-temporal loads and stores
      q[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(p.Q) + qoff));
      if (lead[j]) {
        k[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(p.K) + koff));
        v[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(p.V) + koff));
      }
    }
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
      if (!ok[j]) continue;
      u32x4 o = q[j];
      if (lead[j]) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          o[e] = pack_bf16(bf16lo(q[j][e]) + bf16lo(k[j][e]) + bf16lo(v[j][e]),
                           bf16hi(q[j][e]) + bf16hi(k[j][e]) + bf16hi(v[j][e]));
      }
      const size_t qoff = ((size_t)(r[j] / p.n) * p.n + src[j]) * d + sub * 8;
      __builtin_nontemporal_store(o, reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(p.Y) + qoff));
    }
  }
}

// ---- permutation sampler (Sec. 3.3: sigma ~ Uniform(S_n), fresh per layer): sort by random key.
// Slot p of slice s gets the 64-bit sort key  (r(p) with its low 20 bits replaced by p),  r(p) = the
// (p+1)-th output of SplitMix64 started at a per-(seed, layer, slice) stream value: 44 random bits,
// ties broken by p, all keys distinct.  perm = argsort of the keys.  The keys are uniform 64-bit numbers, so their top
// bits spread them evenly over buckets; a workgroup owns one bucket of one slice, gathers its keys in LDS together with
// the number of keys in lower buckets, ranks them among themselves and writes perm[lower + rank] = p.  The result
// depends on no order of arrival.  Two ways to gather:
//   scan    one launch, no workspace: every workgroup forms all n keys (a hash of p, 150 cycles per 64 of them) and
//           keeps its own;
//   binned  two launches, with a workspace: a first kernel forms each key once, in pieces of consecutive slots, and
//           leaves every piece ordered by bucket with the bucket boundaries beside it; the owner of a bucket then
//           reads one boundary pair and a few keys per piece, and the boundaries' sum is the number of lower keys.
__device__ __forceinline__ uint64_t splitmix_mix(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
constexpr uint64_t kGamma = 0x9E3779B97F4A7C15ull;
constexpr uint64_t kIndexMask = 0xFFFFFull;  // n <= 2^20

__device__ __forceinline__ uint64_t sort_key(uint64_t stream, int p) {
  return (splitmix_mix(stream + kGamma * (uint64_t)(p + 1)) & ~kIndexMask) | (uint64_t)p;
}

__device__ __forceinline__ uint64_t slice_stream(uint64_t seed, int layer, int slice) {
  return splitmix_mix(splitmix_mix(seed) + kGamma * (((uint64_t)(uint32_t)layer << 32) | (uint32_t)slice));
}

constexpr int SAMPLE_CAP = 1024;  // keys of a bucket held in LDS (at most 256 expected: 1024 is 48 standard deviations off)

// perm[lower + rank of the key in its bucket] = slot, for the cnt keys in LDS: four lanes share a key
__device__ __forceinline__ void rank_bucket(const uint64_t* keys, int cnt, int lower, int32_t* __restrict__ perm_slice) {
  const int sub = threadIdx.x & 3;
  for (int e0 = 0; e0 < cnt; e0 += 64) {
    const int e = e0 + (threadIdx.x >> 2);
    const uint64_t mine = keys[min(e, cnt - 1)];
    int rank = 0;
#pragma unroll 4
    for (int j = sub; j < cnt; j += 4) rank += keys[j] < mine ? 1 : 0;
    rank += __shfl_xor(rank, 1);
    rank += __shfl_xor(rank, 2);
    if (sub == 0 && e < cnt) perm_slice[lower + rank] = (int32_t)(mine & kIndexMask);
  }
}

// A bucket that does not fit in LDS (never seen): its keys are ranked against all keys of the slice, one after another.
__device__ void rank_oversized(uint64_t stream, int bucket, int shift, int n, int32_t* __restrict__ perm_slice) {
  for (int p = threadIdx.x; p < n; p += 256) {
    const uint64_t mine = sort_key(stream, p);
    if ((int)(mine >> shift) != bucket) continue;
    int rank = 0;
    for (int q = 0; q < n; ++q) rank += sort_key(stream, q) < mine ? 1 : 0;
    perm_slice[rank] = p;
  }
}

// grid (buckets, slices); bucket of key k = k >> shift, shift <= 63; cap <= SAMPLE_CAP
__global__ __launch_bounds__(256) void sample_scan_kernel(int32_t* __restrict__ perm, const int n, const uint64_t seed, const int layer,
                                                          const int shift, const int cap) {
  __shared__ uint64_t keys[SAMPLE_CAP];
  __shared__ int counters[2];  // keys in the bucket, keys below it
  const int bucket = blockIdx.x, slice = blockIdx.y;
  const uint64_t stream = slice_stream(seed, layer, slice);
  if (threadIdx.x < 2) counters[threadIdx.x] = 0;
  __syncthreads();
  int lower = 0;
#pragma unroll 4
  for (int p = threadIdx.x; p < n; p += 256) {
    const uint64_t k = sort_key(stream, p);
    const int b = (int)(k >> shift);
    lower += b < bucket ? 1 : 0;
    if (b == bucket) {
      const int at = atomicAdd(&counters[0], 1);
      if (at < cap) keys[at] = k;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) lower += __shfl_xor(lower, o);
  if ((threadIdx.x & 63) == 0) atomicAdd(&counters[1], lower);
  __syncthreads();
  const int cnt = counters[0];
  int32_t* out = perm + (size_t)slice * n;
  if (cnt > cap) rank_oversized(stream, bucket, shift, n, out);
  else rank_bucket(keys, cnt, counters[1], out);
}

struct SampleWs {
  uint64_t* keys;    // [slices][n]: pieces of `piece` slots, each ordered by bucket
  uint16_t* bounds;  // [slices][pieces][buckets + 1]: where each bucket starts in its piece
  int buckets, shift, piece, pieces;
};

constexpr int SAMPLE_MAX_BUCKETS = 4096;

// grid (pieces, slices)
__global__ __launch_bounds__(256) void sample_bin_kernel(const SampleWs w, const int n, const uint64_t seed, const int layer) {
  __shared__ int place[SAMPLE_MAX_BUCKETS];
  __shared__ int wave_sum[4];
  const int piece = blockIdx.x, slice = blockIdx.y, t = threadIdx.x;
  const uint64_t stream = slice_stream(seed, layer, slice);
  const int p0 = piece * w.piece, p1 = min(p0 + w.piece, n);
  for (int b = t; b < w.buckets; b += 256) place[b] = 0;
  __syncthreads();
  for (int p = p0 + t; p < p1; p += 256) atomicAdd(&place[(int)(sort_key(stream, p) >> w.shift)], 1);
  __syncthreads();
  // exclusive prefix sum: a thread sums its run of buckets, the runs are scanned over the workgroup
  const int run = (w.buckets + 255) / 256, b0 = t * run, b1 = min(b0 + run, w.buckets);
  int sum = 0;
  for (int b = b0; b < b1; ++b) sum += place[b];
  int incl = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int v = __shfl_up(incl, o);
    if ((t & 63) >= o) incl += v;
  }
  if ((t & 63) == 63) wave_sum[t >> 6] = incl;
  __syncthreads();
  int at = incl - sum;
  for (int v = 0; v < (t >> 6); ++v) at += wave_sum[v];
  for (int b = b0; b < b1; ++b) {
    const int c = place[b];
    place[b] = at;
    at += c;
  }
  __syncthreads();
  uint16_t* bounds = w.bounds + ((size_t)slice * w.pieces + piece) * (w.buckets + 1);
  for (int b = t; b <= w.buckets; b += 256) bounds[b] = (uint16_t)(b < w.buckets ? place[b] : p1 - p0);
  __syncthreads();
  uint64_t* keys = w.keys + (size_t)slice * n + p0;
  for (int p = p0 + t; p < p1; p += 256) {
    const uint64_t k = sort_key(stream, p);
    keys[atomicAdd(&place[(int)(k >> w.shift)], 1)] = k;
  }
}

// grid (buckets, slices)
__global__ __launch_bounds__(256) void sample_merge_kernel(const SampleWs w, int32_t* __restrict__ perm, const int n, const uint64_t seed,
                                                           const int layer, const int cap) {
  __shared__ uint64_t keys[SAMPLE_CAP];
  __shared__ int counters[2];
  const int bucket = blockIdx.x, slice = blockIdx.y;
  if (threadIdx.x < 2) counters[threadIdx.x] = 0;
  __syncthreads();
  int lower = 0;
  for (int c = threadIdx.x; c < w.pieces; c += 256) {
    const uint16_t* bounds = w.bounds + ((size_t)slice * w.pieces + c) * (w.buckets + 1) + bucket;
    const int i0 = bounds[0], i1 = bounds[1];
    const uint64_t* src = w.keys + (size_t)slice * n + (size_t)c * w.piece;
    lower += i0;
    int at = i1 > i0 ? atomicAdd(&counters[0], i1 - i0) : 0;
    for (int i = i0; i < i1; ++i, ++at)
      if (at < cap) keys[at] = src[i];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) lower += __shfl_xor(lower, o);
  if ((threadIdx.x & 63) == 0) atomicAdd(&counters[1], lower);
  __syncthreads();
  const int cnt = counters[0];
  int32_t* out = perm + (size_t)slice * n;
  if (cnt > cap) rank_oversized(slice_stream(seed, layer, slice), bucket, w.shift, n, out);
  else rank_bucket(keys, cnt, counters[1], out);
}

template <int LPR>  // lanes per row, each lane owns 16 bytes of the row
__device__ __forceinline__ float group_sum(float v) {
#pragma unroll
  for (int o = LPR / 2; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// One group of LPR lanes per row; E = elements per 16-byte vector (8 bf16 / 4 f32).
template <bool BF16, int LPR>
__global__ __launch_bounds__(256) void bwd_prepare_kernel(Prep p) {
  constexpr int E = BF16 ? 8 : 4;
  const int sub = threadIdx.x % LPR;
  const long row = ((long)blockIdx.x * 256 + threadIdx.x) / LPR;
  const bool valid = row < p.rows;
  const size_t r = valid ? (size_t)row : 0;
  const size_t off = r * p.d + (size_t)sub * E;

  float dy[E], ya[E], yb[E];
  if (BF16) {
    const u32x4 a = *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(p.dY) + off);
    const u32x4 b = *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(p.Y_a) + off);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      dy[2 * k] = bf16lo(a[k]); dy[2 * k + 1] = bf16hi(a[k]);
      ya[2 * k] = bf16lo(b[k]); ya[2 * k + 1] = bf16hi(b[k]);
    }
    const u32x4 c = *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(p.Y_b) + off);
#pragma unroll
    for (int k = 0; k < 4; ++k) { yb[2 * k] = bf16lo(c[k]); yb[2 * k + 1] = bf16hi(c[k]); }
  } else {
    const f32x4 a = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(p.dY) + off);
    const f32x4 b = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(p.Y_a) + off);
#pragma unroll
    for (int k = 0; k < 4; ++k) { dy[k] = a[k]; ya[k] = b[k]; }
    const f32x4 c = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(p.Y_b) + off);
#pragma unroll
    for (int k = 0; k < 4; ++k) yb[k] = c[k];
  }

  // dO_x = sig(gamma_x) * dY;  D_x = sum_d dO_x * Y_x;  dgamma_x = sig'(gamma_x) * dY * Y_x
  // (bf16 rows with one gate each go to bwd_fold_kernel)
  const bool per_dim = BF16 || p.gate_per_dim;
  float ga[E], gb[E];
  if (per_dim) {
#pragma unroll
    for (int k = 0; k < E; ++k) {
      ga[k] = sigmoidf_exact(load_gate(p.gate_a, off + k, p.gate_f32));
      gb[k] = sigmoidf_exact(load_gate(p.gate_b, off + k, p.gate_f32));
    }
  } else {  // one gate per row: one sigmoid, not one per element
    const float a1 = sigmoidf_exact(load_gate(p.gate_a, r, p.gate_f32));
    const float b1 = sigmoidf_exact(load_gate(p.gate_b, r, p.gate_f32));
#pragma unroll
    for (int k = 0; k < E; ++k) {
      ga[k] = a1;
      gb[k] = b1;
    }
  }
  float da[E], db[E], sa = 0.f, sb = 0.f, ra = 0.f, rb = 0.f;
#pragma unroll
  for (int k = 0; k < E; ++k) {
    da[k] = ga[k] * dy[k];
    db[k] = gb[k] * dy[k];
    sa = fmaf(da[k], ya[k], sa);
    sb = fmaf(db[k], yb[k], sb);
    ra = fmaf(dy[k], ya[k], ra);
    rb = fmaf(dy[k], yb[k], rb);
  }
  sa = group_sum<LPR>(sa);
  sb = group_sum<LPR>(sb);
  if (valid && sub == 0) {
    p.D_a[r] = sa;
    p.D_b[r] = sb;
  }
  if (per_dim) {
    if (valid) {
#pragma unroll
      for (int k = 0; k < E; ++k) {
        store_gate(p.dgate_a, off + k, p.gate_f32, ga[k] * (1.f - ga[k]) * dy[k] * ya[k]);
        store_gate(p.dgate_b, off + k, p.gate_f32, gb[k] * (1.f - gb[k]) * dy[k] * yb[k]);
      }
    }
  } else {
    ra = group_sum<LPR>(ra);
    rb = group_sum<LPR>(rb);
    if (valid && sub == 0) {
      store_gate(p.dgate_a, r, p.gate_f32, ga[0] * (1.f - ga[0]) * ra);
      store_gate(p.dgate_b, r, p.gate_f32, gb[0] * (1.f - gb[0]) * rb);
    }
  }
  if (valid) {
    if (BF16) {
      u32x4 oa, ob;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        oa[k] = pack_bf16(da[2 * k], da[2 * k + 1]);
        ob[k] = pack_bf16(db[2 * k], db[2 * k + 1]);
      }
      *reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(p.dO_a) + off) = oa;
      *reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(p.dO_b) + off) = ob;
    } else {
      f32x4 oa, ob;
#pragma unroll
      for (int k = 0; k < 4; ++k) { oa[k] = da[k]; ob[k] = db[k]; }
      *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(p.dO_a) + off) = oa;
      *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(p.dO_b) + off) = ob;
    }
  }
}

// The same for bf16 and one gate per row with the gate folded into the per-row scalars: E_x = rowsum(dY o Y_x),
// LSE_x - ln g_x, dgamma_x; no copy of dY.  Reads three rows and writes six scalars a row: bound by memory.  A lane group takes
// U rows (12 loads of 16 bytes in flight a lane at U = 4) and its lanes share the logarithms and the stores, one (row, branch)
// each, so that a wave stores 32 neighbouring scalars of both branches with one instruction; with one row per group and one
// lane in eight storing, B4 H16 n8192 d64 took 66 us (3.3 TB/s), now 37 us (5.8 TB/s).
template <int LPR>
__global__ __launch_bounds__(256) void bwd_fold_kernel(const Prep p) {
  constexpr int U = LPR / 2;      // rows per group: two branches x U rows = its lanes
  constexpr int GPW = 64 / LPR;   // groups per wave
  const int lane = threadIdx.x & 63, sub = lane % LPR, grp = lane / LPR;
  const long wave_row0 = ((long)blockIdx.x * 4 + (threadIdx.x >> 6)) * (U * GPW);
  u32x4 dy[U], ya[U], yb[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {  // rows past the last one: the last one again, never stored
    const long row = wave_row0 + u * GPW + grp;
    const size_t off = (size_t)(row < p.rows ? row : p.rows - 1) * p.d + (size_t)sub * 8;
    dy[u] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(p.dY) + off);
    ya[u] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(p.Y_a) + off);
    yb[u] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(p.Y_b) + off);
  }
  // this lane's share of the rest: branch a or b of row `mine`
  const bool is_b = sub >= U;
  const int own = sub % U;
  const long mine = wave_row0 + own * GPW + grp;
  const bool valid = mine < p.rows;
  const size_t r = valid ? (size_t)mine : 0;
  const float x = load_gate(is_b ? p.gate_b : p.gate_a, r, p.gate_f32);
  const float lse = (is_b ? p.lse_b : p.lse_a)[r];
  float e = 0.f;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    float ra = 0.f, rb = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      ra = fmaf(bf16hi(dy[u][k]), bf16hi(ya[u][k]), fmaf(bf16lo(dy[u][k]), bf16lo(ya[u][k]), ra));
      rb = fmaf(bf16hi(dy[u][k]), bf16hi(yb[u][k]), fmaf(bf16lo(dy[u][k]), bf16lo(yb[u][k]), rb));
    }
    ra = group_sum<LPR>(ra);
    rb = group_sum<LPR>(rb);
    if (own == u) e = is_b ? rb : ra;
  }
  if (!valid) return;
  const float g = sigmoidf_exact(x);
  // -ln sigmoid(x) = ln(1 + e^-x), evaluated without cancellation on either side
  const float nl = x > 0.f ? log1pf(__expf(-x)) : -x + log1pf(__expf(x));
  (is_b ? p.D_b : p.D_a)[r] = e;
  (is_b ? p.L_b : p.L_a)[r] = lse + nl;
  store_gate(is_b ? p.dgate_b : p.dgate_a, r, p.gate_f32, g * (1.f - g) * e);
}

template <int LPR>
hipError_t launch_fold_t(const Prep& p, hipStream_t st) {
  const long per_block = 4 * 32;  // rows: LPR / 2 rows of 64 / LPR groups in each of 4 waves
  hipLaunchKernelGGL(bwd_fold_kernel<LPR>, dim3((unsigned)((p.rows + per_block - 1) / per_block)), dim3(256), 0, st, p);
  return hipGetLastError();
}

template <bool BF16, int LPR>
hipError_t launch_prepare_t(const Prep& p, hipStream_t st) {
  const long threads = (long)p.rows * LPR;
  const unsigned blocks = (unsigned)((threads + 255) / 256);
  hipLaunchKernelGGL((bwd_prepare_kernel<BF16, LPR>), dim3(blocks), dim3(256), 0, st, p);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_fill_zero(void* ptr, size_t bytes, hipStream_t st) {
  if (bytes % 4 != 0) return hipErrorInvalidValue;
  const size_t words = bytes / 4;
  if (words == 0) return hipSuccess;
  const unsigned blocks = (unsigned)((words + 1023) / 1024 < 4096 ? (words + 1023) / 1024 : 4096);
  hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks), dim3(256), 0, st, reinterpret_cast<uint32_t*>(ptr), words);
  return hipGetLastError();
}

hipError_t launch_check_perm(const int32_t* perm, int slices, int n, int* seen, int* flag, hipStream_t st) {
  const size_t total = (size_t)slices * n;
  hipError_t e = launch_fill_zero(seen, total * sizeof(int), st);
  if (e != hipSuccess) return e;
  e = launch_fill_zero(flag, sizeof(int), st);
  if (e != hipSuccess) return e;
  const unsigned blocks = (unsigned)((total + 255) / 256 < 4096 ? (total + 255) / 256 : 4096);
  hipLaunchKernelGGL(check_perm_kernel, dim3(blocks), dim3(256), 0, st, perm, total, n, seen, flag);
  return hipGetLastError();
}

// log2 of the number of buckets: `per_bucket` keys each on average, at least two buckets (a shift by 64 is undefined)
static int sample_bits(int n, int per_bucket) {
  int bits = 1;
  while (((long)per_bucket << bits) < n) ++bits;
  return bits;
}

// Binned form: 64 to 128 keys a bucket on average (past 2^19 slots, with SAMPLE_MAX_BUCKETS, up to 256), pieces of at
// least as many slots as there are buckets, so that the boundaries stay smaller than the keys.
static SampleWs sample_layout(int n) {
  SampleWs w = {};
  int bits = sample_bits(n, 128);
  while ((1 << bits) > SAMPLE_MAX_BUCKETS) --bits;
  w.buckets = 1 << bits;
  w.shift = 64 - bits;
  w.piece = w.buckets < 512 ? 512 : w.buckets;
  w.pieces = (n + w.piece - 1) / w.piece;
  return w;
}

size_t sample_perm_workspace_bytes(int slices, int n) {
  const SampleWs w = sample_layout(n);
  return (size_t)slices * ((size_t)n * 8 + (size_t)w.pieces * (w.buckets + 1) * 2) + 512;
}

hipError_t launch_sample_perm(int32_t* perm, int slices, int n, uint64_t seed, int layer, void* ws, hipStream_t st, int cap) {
  if (cap < 1 || cap > SAMPLE_CAP) cap = SAMPLE_CAP;
  if (!perm || slices < 1 || slices > 65535 || n < 1) return hipErrorInvalidValue;
  if (n > (1 << 20)) return hipErrorNotSupported;  // the slot index takes the low 20 bits of the sort key
  const int bits = sample_bits(n, n <= 32768 ? 64 : 256);
  // The scan forms n keys in every workgroup, 6 million of them in about the time of the second launch of the binned form
  // (event times, both forms: 1 slice of 16 384 12.6 / 15.4 us, of 24 000 17.7 / 15.6 us, of 131 072 78 / 16.8 us;
  // 12 slices of 8192 19.2 / 16.8 us).  Sorting by counting every key against every other took 38 us at n = 16 384, and
  // five launches over global counters 44 us at 32 768 (now 15.8) and 60 us at 131 072.
  if (ws && (double)slices * n * (1 << bits) > 6e6) {
    SampleWs w = sample_layout(n);
    char* base = reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(ws) + 255) & ~(uintptr_t)255);
    w.keys = reinterpret_cast<uint64_t*>(base);
    w.bounds = reinterpret_cast<uint16_t*>(base + (size_t)slices * n * 8);
    hipLaunchKernelGGL(sample_bin_kernel, dim3((unsigned)w.pieces, (unsigned)slices), dim3(256), 0, st, w, n, seed, layer);
    hipLaunchKernelGGL(sample_merge_kernel, dim3((unsigned)w.buckets, (unsigned)slices), dim3(256), 0, st, w, perm, n, seed, layer, cap);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(sample_scan_kernel, dim3(1u << bits, (unsigned)slices), dim3(256), 0, st, perm, n, seed, layer, 64 - bits, cap);
  return hipGetLastError();
}

hipError_t launch_permuted_copy_bf16(const Pass& p, hipStream_t st) {
  if (p.n < 1 || p.B < 1 || p.Hq < 1 || p.Hkv < 1 || p.g * p.Hkv != p.Hq || !p.Q || !p.K || !p.V || !p.Y)
    return hipErrorInvalidValue;
  if (!(p.d == 64 || p.d == 128)) return hipErrorNotSupported;
  const long rows = (long)p.B * p.Hq * p.n;
  const int lpr = p.d / 8;
  const long want = (rows * lpr + 256 * 4 - 1) / (256 * 4);  // four rows per lane group
  const unsigned blocks = (unsigned)(want < 1 ? 1 : (want > 0x7fffffffL ? 0x7fffffffL : want));
  if (p.d == 64) hipLaunchKernelGGL(permuted_copy_bf16_kernel<8>, dim3(blocks), dim3(256), 0, st, p, rows);
  else hipLaunchKernelGGL(permuted_copy_bf16_kernel<16>, dim3(blocks), dim3(256), 0, st, p, rows);
  return hipGetLastError();
}

hipError_t launch_bwd_prepare(const Prep& p, hipStream_t st) {
  if (p.rows < 1 || !(p.d == 64 || p.d == 128)) return hipErrorInvalidValue;
  if (p.bf16 && !p.gate_per_dim) return p.d == 64 ? launch_fold_t<8>(p, st) : launch_fold_t<16>(p, st);
  if (p.bf16) return p.d == 64 ? launch_prepare_t<true, 8>(p, st) : launch_prepare_t<true, 16>(p, st);
  return p.d == 64 ? launch_prepare_t<false, 16>(p, st) : launch_prepare_t<false, 32>(p, st);
}

}  // namespace sa
