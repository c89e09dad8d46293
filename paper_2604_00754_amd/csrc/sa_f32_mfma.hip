// fp32 path of libsa on the fp32 matrix instructions (dtype == SA_F32, tolerance 1e-5 against the fp64 definition).
//
// v_mfma_f32_16x16x4_f32 multiplies and adds in full fp32 and does twice the flop per cycle of the vector FMA, so
// the products of Eq. 1 and of its gradient run there; the exponentials are v_exp_f32 on scores
// scaled by log2(e) / sqrt(d) in fp32.
// One workgroup (1, 2 or 4 wavefronts) owns a tile of 16 slots of one head in permuted order; the streamed blocks of 16
// slots of the window band (Eq. 3) are dealt to its wavefronts in turn, and what they accumulate is added through
// LDS at the end.  Streamed rows are requested one block ahead and there is no barrier in the loop, so the wavefronts of
// a SIMD run freely against each other.  What bounds a call is the chain of a wavefront: rows -> LDS -> scores -> weights -> sums
// for every block, index -> rows before the first one.  A 16 x 16 block costs 32 cycles of the matrix pipe for every 4
// elements of the head size and each product; at two wavefronts a SIMD (B2 H8 n2039 d64 w128) that pipe is busy 33 % (forward)
// to 44 % (dK, dV) of the time and a wavefront waits 47 to 60 % of its life.
//
// Operand layouts (lane = 16 g + c).  The instruction takes A[c][g], B[g][c] and leaves C[4g + i][c] in
// accumulator i.  Which element of a row is contraction index g of which instruction is free as long as both
// operands agree, so rows are loaded 16 bytes per lane:
//   "rows":    lane (g, c) holds elements 16 j + 4 g + e of row c (contraction over the head size, instruction 4j + e)
//   "columns": lane (g, c) holds elements 64 h + 4 c + e of row 4 g + i (contraction over the 16 rows, instruction i;
//              output row c of block 4 h + e is element 64 h + 4 c + e), so the 16 lanes of a group read whole rows
// The accumulators of the first product (keys or queries 4g + i) are the B operand of the second one as they are.
#include "sa_common.h"
#include "sa_mfma.h"

namespace sa {
namespace {

constexpr int FT = 16;    // slots per tile and per streamed block

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// Rows come in as "columns" (whole rows, 16 lanes of 16 bytes each: with one row per lane every lane would be a cache
// access of its own) and reach the "rows" layout through an area of LDS that belongs to the wavefront.  16 bytes of
// padding per row keep both patterns free of bank conflicts.
template <int D>
struct Stage {
  static constexpr int STR = D + 4;          // floats per staged row
  static constexpr int FLOATS = FT * STR;    // one operand of one wavefront
};

// f[i * (D / 64) + h]: row i of the lane's group, half h of the row
template <int D>
__device__ __forceinline__ void load_columns(const float* __restrict__ head, int row_c, int g, int c, f32x4* f) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float* r = head + (size_t)(unsigned)__shfl(row_c, 4 * g + i) * D + 4 * c;
#pragma unroll
    for (int h = 0; h < D / 64; ++h) f[i * (D / 64) + h] = *reinterpret_cast<const f32x4*>(r + 64 * h);
  }
}

template <int D>
__device__ __forceinline__ void put_columns(float* stage, int g, int c, const f32x4* f) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int h = 0; h < D / 64; ++h) *reinterpret_cast<f32x4*>(stage + (4 * g + i) * Stage<D>::STR + 64 * h + 4 * c) = f[i * (D / 64) + h];
}

template <int D>
__device__ __forceinline__ void get_columns(const float* stage, int g, int c, f32x4* f) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int h = 0; h < D / 64; ++h) f[i * (D / 64) + h] = *reinterpret_cast<const f32x4*>(stage + (4 * g + i) * Stage<D>::STR + 64 * h + 4 * c);
}

template <int D>
__device__ __forceinline__ void get_rows(const float* stage, int g, int c, f32x4* f) {
#pragma unroll
  for (int j = 0; j < D / 16; ++j) f[j] = *reinterpret_cast<const f32x4*>(stage + c * Stage<D>::STR + 16 * j + 4 * g);
}

// Rows to the staging area and into the "rows" layout.
template <int D>
__device__ __forceinline__ void stage_rows(float* stage, int g, int c, const f32x4* cols, f32x4* f) {
  wave_lds_sync();
  put_columns<D>(stage, g, c, cols);
  wave_lds_sync();
  get_rows<D>(stage, g, c, f);
}

// C[streamed 4g + i][stationary c] = <streamed row, stationary row>, on two accumulators: a chain on one would wait for
// every instruction's result
template <int D>
__device__ __forceinline__ f32x4 product_rows(const f32x4* a, const f32x4* b) {
  f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
#pragma unroll
  for (int j = 0; j < D / 16; ++j) {
    s0 = mfma_f32(a[j][0], b[j][0], s0);
    s1 = mfma_f32(a[j][1], b[j][1], s1);
    s0 = mfma_f32(a[j][2], b[j][2], s0);
    s1 = mfma_f32(a[j][3], b[j][3], s1);
  }
  return s0 + s1;
}

// acc[4h + e] += sum over the block's rows of columns[row][64 h + 4 (4g + i) + e] * w[row][c]
template <int D>
__device__ __forceinline__ void product_columns(f32x4* acc, const f32x4* cols, const f32x4 w) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int b = 0; b < D / 16; ++b) acc[b] = mfma_f32(cols[i * (D / 64) + b / 4][b % 4], w[i], acc[b]);
}

// The same sum over the staged rows of a block with the rows of weight zero left out.  A matrix instruction multiplies them as
// well, and zero times an infinity or NaN in a row that query (or key) c does not see would be a NaN in its sum: a band whose
// sums are not finite is walked again with this form, so that only what is seen can make them so.
template <int D>
__device__ __forceinline__ void add_weighted_rows(f32x4* acc, const float* stage, const f32x4 w, int g, int c) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll 1
    for (int from = 0; from < 4; ++from) {
      const float wr = __shfl(w[i], 16 * from + c);
      const float* row = stage + (4 * from + i) * Stage<D>::STR + 16 * g;
#pragma unroll
      for (int h = 0; h < D / 64; ++h)
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(row + 64 * h + 4 * x);
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[4 * h + e][x] = wr != 0.f ? fmaf(wr, v[e], acc[4 * h + e][x]) : acc[4 * h + e][x];
        }
    }
}

// A copy of the lane number that the optimiser cannot trace: what follows from it is formed where it is used and not kept in
// registers across the tile loop.
__device__ __forceinline__ int fresh(int lane) {
  asm volatile("" : "+v"(lane));
  return lane;
}

// Is one of the sums of a lane that counts infinite or NaN?  The same answer in every lane.
template <int D>
__device__ __forceinline__ bool any_not_finite(const f32x4* acc, bool counts) {
  float t = 0.f;
#pragma unroll
  for (int b = 0; b < D / 16; ++b)
#pragma unroll
    for (int x = 0; x < 4; ++x) t = fmaf(acc[b][x], 0.f, t);
  return __any(counts & (t != 0.f));  // (NaN != 0)
}

// The slot tile of a workgroup and the band it streams.
struct Tile {
  int b, h, s0, s_last, lo, hi, nblocks;
};

// Work item of this workgroup: tiles of one head next to each other, one contiguous piece of the list per XCD (the
// row count of a call is below 2^31, so the list is indexed with 32-bit integers).  false: surplus workgroup.
__device__ __forceinline__ bool pick_tile(Tile& t, const Pass& p, unsigned num_tiles, unsigned total, unsigned heads) {
  const unsigned chunk = (total + NXCD - 1) / NXCD, local = blockIdx.x / NXCD, work = (blockIdx.x % NXCD) * chunk + local;
  if (local >= chunk || work >= total) return false;
  const unsigned bh = work / num_tiles;
  t.s0 = (int)(work - bh * num_tiles) * FT;
  t.b = (int)(bh / heads);
  t.h = (int)(bh - t.b * heads);
  t.s_last = min(t.s0 + FT - 1, p.n - 1);
  return true;
}

__device__ __forceinline__ void set_band(Tile& t, const Pass& p, int lo_reach, int hi_reach) {
  t.lo = t.s0 - lo_reach;
  t.hi = t.s_last + hi_reach;
  if (!p.win.circular) {
    t.lo = max(t.lo, 0);
    t.hi = min(t.hi, p.n - 1);
  }
  t.nblocks = (t.hi - t.lo + FT) / FT;
}

// PERM = false: identity permutation.
template <bool PERM>
__device__ __forceinline__ const int32_t* perm_of(const Pass& p, int b, int hq) {
  return PERM ? p.perm + (size_t)perm_slice_index(p.perm_B, p.perm_H, b, hq) * p.n : nullptr;
}

// Original index of row c of streamed block blk (past the band: its last slot, masked where it is used).
template <bool PERM>
__device__ __forceinline__ int streamed_row(const Tile& t, const int32_t* __restrict__ perm, int blk, int c, int n) {
  const int slot = wrap_slot(min(t.lo + FT * min(blk, t.nblocks - 1) + c, t.hi), n);
  return PERM ? perm[slot] : slot;
}

// Sum over the four lane groups (lanes with the same c).
__device__ __forceinline__ float group_sum4(float v) {
  v += __shfl_xor(v, 16);
  return v + __shfl_xor(v, 32);
}
__device__ __forceinline__ float group_max4(float v) {
  v = fmaxf(v, __shfl_xor(v, 16));
  return fmaxf(v, __shfl_xor(v, 32));
}

// Adds the wavefronts' accumulators (D / 4 values per lane) through their staging areas, `stride` floats apart:
// wavefront `wave` gets element quads i = wave + FW q of every block, i.e. for half h the elements 64 h + 16 g + 4 i
// .. +3 of row c in out[q][h].  scale[w]: factor of wavefront w.
template <int D, int FW>
__device__ __forceinline__ void merge_waves(float* area, int stride, const f32x4* acc, const float* scale, int wave, int lane, f32x4 (*out)[D / 64]) {
  static_assert(D / 4 * 64 <= Stage<D>::FLOATS, "the accumulators of a wavefront fit its staging area");
#pragma unroll
  for (int b = 0; b < D / 16; ++b)
#pragma unroll
    for (int i = 0; i < 4; ++i) area[wave * stride + (4 * b + i) * 64 + lane] = acc[b][i];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4 / FW; ++q)
#pragma unroll
    for (int h = 0; h < D / 64; ++h)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < FW; ++w) v = fmaf(scale[w], area[w * stride + (4 * (4 * h + e) + wave + FW * q) * 64 + lane], v);
        out[q][h][e] = v;
      }
}

// ------------------------------------------------------------------------------------- forward
template <int D, bool PERM, int FW>
__global__ __launch_bounds__(64 * FW, D == 64 ? 4 : 2) void fwd_f32_kernel(const Pass p, const unsigned num_tiles, const unsigned total_work) {
  __shared__ __attribute__((aligned(16))) float area[FW * Stage<D>::FLOATS];
  __shared__ float lds_m[FW][FT], lds_l[FW][FT];
  Tile t;
  if (!pick_tile(t, p, num_tiles, total_work, p.Hq)) return;
  const int n = p.n;
  set_band(t, p, p.win.L, p.win.R);
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int32_t* __restrict__ perm = perm_of<PERM>(p, t.b, t.h);
  const float* __restrict__ Kh = reinterpret_cast<const float*>(p.K) + ((size_t)t.b * p.Hkv + (t.h / p.g)) * n * (size_t)D;
  const float* __restrict__ Vh = reinterpret_cast<const float*>(p.V) + ((size_t)t.b * p.Hkv + (t.h / p.g)) * n * (size_t)D;
  const size_t head_row0 = ((size_t)t.b * p.Hq + t.h) * n;

  const int s = t.s0 + c;
  const int orig_q = PERM ? perm[min(s, n - 1)] : min(s, n - 1);
  const int last_q = p.causal ? orig_q : 0x7fffffff;  // no key after it is seen
  const int Ll = p.win.circular ? p.win.L : min(p.win.L, s);  // key slot k is in the window iff 0 <= k - s + Ll <= LRl
  const unsigned LRl = (unsigned)(Ll + (p.win.circular ? p.win.R : min(p.win.R, max(n - 1 - s, 0))));
  // row indices two blocks ahead, K and V rows one block ahead.  Blocks past the end load the last one again: a branch
  // around a load makes the wait before the next product one for all loads
  float* stage = area + wave * Stage<D>::FLOATS;
  int pos = streamed_row<PERM>(t, perm, wave, c, n), pos1 = streamed_row<PERM>(t, perm, wave + FW, c, n);
  f32x4 qf[D / 16], kn[D / 16], vn[D / 16], o[D / 16];
  load_columns<D>(reinterpret_cast<const float*>(p.Q) + head_row0 * D, orig_q, g, c, qf);
  load_columns<D>(Kh, pos, g, c, kn);
  load_columns<D>(Vh, pos, g, c, vn);
  stage_rows<D>(stage, g, c, qf, qf);
#pragma unroll
  for (int b = 0; b < D / 16; ++b) o[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float cs = p.scale * kLog2e;  // exp(scale * x) = exp2(cs * x)
  float m = -INFINITY, l = 0.f;
  // weights of a block (keys 4g + i, query c) from its scores; the sums so far follow the running maximum
  auto weigh = [&](int blk, const f32x4 st, const int* kpos) -> f32x4 {
    const int t0 = t.lo + FT * blk + 4 * g - s + Ll;
    f32x4 z, pe;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool seen = ((unsigned)(t0 + i) <= LRl) & (kpos[i] <= last_q);
      z[i] = seen ? st[i] : -INFINITY;
    }
    // m: running maximum of the unscaled scores (the key that holds it gets weight one exactly)
    const float zmax = group_max4(fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3])));
    if (__any(zmax > m)) {
      const float m_new = fmaxf(m, zmax), alpha = m_new == m ? 1.f : __builtin_amdgcn_exp2f((m - m_new) * cs);
      m = m_new;
      l *= alpha;
#pragma unroll
      for (int b = 0; b < D / 16; ++b) o[b] *= alpha;
    }
    const float ms = m == -INFINITY ? 0.f : m;
#pragma unroll
    for (int i = 0; i < 4; ++i) pe[i] = __builtin_amdgcn_exp2f((z[i] - ms) * cs);
    l += (pe[0] + pe[1]) + (pe[2] + pe[3]);  // this lane group's keys; the groups are added at the end
    return pe;
  };
  for (int blk = wave; blk < t.nblocks; blk += FW) {
    wave_lds_sync();
    put_columns<D>(stage, g, c, kn);
    wave_lds_sync();
    int kpos[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) kpos[i] = __shfl(pos, 4 * g + i);
    pos = pos1;
    load_columns<D>(Kh, pos, g, c, kn);
    pos1 = streamed_row<PERM>(t, perm, blk + 2 * FW, c, n);
    f32x4 kf[D / 16];
    get_rows<D>(stage, g, c, kf);
    __builtin_amdgcn_sched_barrier(0);
    const f32x4 st = product_rows<D>(kf, qf);  // S^T: keys 4g + i, query c
    const f32x4 pe = weigh(blk, st, kpos);
    product_columns<D>(o, vn, pe);
    __builtin_amdgcn_sched_barrier(0);
    load_columns<D>(Vh, pos, g, c, vn);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (__builtin_expect(any_not_finite<D>(o, s < n), 0)) {
    const int le = fresh(lane), g = le >> 4, c = le & 15;
    m = -INFINITY;
    l = 0.f;
#pragma unroll
    for (int b = 0; b < D / 16; ++b) o[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int blk = wave; blk < t.nblocks; blk += FW) {
      pos = streamed_row<PERM>(t, perm, blk, c, n);
      load_columns<D>(Kh, pos, g, c, kn);
      load_columns<D>(Vh, pos, g, c, vn);
      stage_rows<D>(stage, g, c, kn, kn);
      int kpos[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) kpos[i] = __shfl(pos, 4 * g + i);
      const f32x4 pe = weigh(blk, product_rows<D>(kn, qf), kpos);
      stage_rows<D>(stage, g, c, vn, kn);
      add_weighted_rows<D>(o, stage, pe, g, c);
    }
  }
  l = group_sum4(l);
  if (g == 0) {
    lds_m[wave][c] = m;
    lds_l[wave][c] = l;
  }
  __syncthreads();
  float M = lds_m[0][c], L = 0.f, scale[FW];
#pragma unroll
  for (int w = 1; w < FW; ++w) M = fmaxf(M, lds_m[w][c]);
#pragma unroll
  for (int w = 0; w < FW; ++w) {
    scale[w] = __builtin_amdgcn_exp2f((lds_m[w][c] - (M == -INFINITY ? 0.f : M)) * cs);
    L = fmaf(scale[w], lds_l[w][c], L);
  }
  const float inv_l = 1.f / L;
  f32x4 y[4 / FW][D / 64];
  merge_waves<D, FW>(area, Stage<D>::FLOATS, o, scale, wave, lane, y);
  if (s >= n) return;
  const size_t row = head_row0 + orig_q;
  if (p.LSE && wave == 0 && g == 0) p.LSE[row] = M * p.scale + logf(L);
#pragma unroll
  for (int qh = 0; qh < 4 / FW * (D / 64); ++qh) {
    const int q = qh / (D / 64), h = qh % (D / 64), col = 64 * h + 16 * g + 4 * (wave + FW * q);
    const size_t at = row * D + col;
    y[q][h] *= inv_l;
    if (p.Y) *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(p.Y) + at) = y[q][h];
    if (p.gate_mode) {
      // Eq. 5: independent sigmoid gates on the two branches
      const f32x4 other = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(p.Y_other) + at);
      f32x4 r;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const size_t gi = p.gate_per_dim ? at + e : row;
        r[e] = sigmoidf_exact(load_gate(p.gate_this, gi, p.gate_f32)) * y[q][h][e] +
               sigmoidf_exact(load_gate(p.gate_other, gi, p.gate_f32)) * other[e];
      }
      *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(p.Yout) + at) = r;
    }
  }
}

// ------------------------------------------------------------------------------------------ dQ
// dQ_i = scale * sum_j dS_ij K_j with dS_ij = P_ij (<dO_i, V_j> - D_i), P_ij = exp(z_ij - LSE_i).
template <int D, bool PERM, int FW>
__global__ __launch_bounds__(64 * FW, D == 64 ? 3 : 2) void bwd_dq_f32_kernel(const Pass p, const unsigned num_tiles, const unsigned total_work) {
  __shared__ __attribute__((aligned(16))) float area[FW * 2 * Stage<D>::FLOATS];
  Tile t;
  if (!pick_tile(t, p, num_tiles, total_work, p.Hq)) return;
  const int n = p.n;
  set_band(t, p, p.win.L, p.win.R);
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int32_t* __restrict__ perm = perm_of<PERM>(p, t.b, t.h);
  const float* __restrict__ Kh = reinterpret_cast<const float*>(p.K) + ((size_t)t.b * p.Hkv + (t.h / p.g)) * n * (size_t)D;
  const float* __restrict__ Vh = reinterpret_cast<const float*>(p.V) + ((size_t)t.b * p.Hkv + (t.h / p.g)) * n * (size_t)D;
  const size_t head_row0 = ((size_t)t.b * p.Hq + t.h) * n;

  const int s = t.s0 + c;
  const int orig_q = PERM ? perm[min(s, n - 1)] : min(s, n - 1);
  const int last_q = p.causal ? orig_q : 0x7fffffff;  // no key after it is seen
  const int Ll = p.win.circular ? p.win.L : min(p.win.L, s);  // key slot k is in the window iff 0 <= k - s + Ll <= LRl
  const unsigned LRl = (unsigned)(Ll + (p.win.circular ? p.win.R : min(p.win.R, max(n - 1 - s, 0))));
  float* stage_k = area + wave * 2 * Stage<D>::FLOATS;
  float* stage_v = stage_k + Stage<D>::FLOATS;
  int pos = streamed_row<PERM>(t, perm, wave, c, n), pos1 = streamed_row<PERM>(t, perm, wave + FW, c, n);
  f32x4 qf[D / 16], gf[D / 16], kn[D / 16], vn[D / 16], dq[D / 16];
  load_columns<D>(reinterpret_cast<const float*>(p.Q) + head_row0 * D, orig_q, g, c, qf);
  load_columns<D>(reinterpret_cast<const float*>(p.dO) + head_row0 * D, orig_q, g, c, gf);
  const float cs = p.scale * kLog2e, lse2 = p.lse_in[head_row0 + orig_q] * kLog2e;
  float Dq;
  if (p.O_rows) {  // rowsum(dO o O) from the rows this wavefront holds anyway: row 4g + i in the 16 lanes of group g
    f32x4 of[D / 16];
    load_columns<D>(reinterpret_cast<const float*>(p.O_rows) + head_row0 * D, orig_q, g, c, of);
    float part[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      part[i] = 0.f;
#pragma unroll
      for (int h = 0; h < D / 64; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e) part[i] = fmaf(gf[i * (D / 64) + h][e], of[i * (D / 64) + h][e], part[i]);
#pragma unroll
      for (int x = 1; x < 16; x <<= 1) part[i] += __shfl_xor(part[i], x);
    }
    const float mine = (c & 2) ? ((c & 1) ? part[3] : part[2]) : ((c & 1) ? part[1] : part[0]);  // row 4g + c % 4
    Dq = __shfl(mine, 16 * (c >> 2) + (c & 3));
    if (wave == 0 && g == 0 && s < n) p.Dsum_out[head_row0 + orig_q] = Dq;
  } else {
    Dq = p.Dsum[head_row0 + orig_q];
  }
  load_columns<D>(Kh, pos, g, c, kn);
  load_columns<D>(Vh, pos, g, c, vn);
  stage_rows<D>(stage_k, g, c, qf, qf);
  stage_rows<D>(stage_v, g, c, gf, gf);
#pragma unroll
  for (int b = 0; b < D / 16; ++b) dq[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto weigh = [&](int blk, const f32x4 st, const f32x4 dp, const int* kpos) -> f32x4 {  // dS of keys 4g + i, query c
    const int t0 = t.lo + FT * blk + 4 * g - s + Ll;
    f32x4 ds;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool seen = ((unsigned)(t0 + i) <= LRl) & (kpos[i] <= last_q);
      const float pr = __builtin_amdgcn_exp2f(fmaf(st[i], cs, -lse2));
      ds[i] = seen ? pr * (dp[i] - Dq) : 0.f;
    }
    return ds;
  };
  for (int blk = wave; blk < t.nblocks; blk += FW) {
    wave_lds_sync();
    put_columns<D>(stage_k, g, c, kn);
    put_columns<D>(stage_v, g, c, vn);
    wave_lds_sync();
    int kpos[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) kpos[i] = __shfl(pos, 4 * g + i);
    pos = pos1;
    load_columns<D>(Kh, pos, g, c, kn);
    load_columns<D>(Vh, pos, g, c, vn);
    pos1 = streamed_row<PERM>(t, perm, blk + 2 * FW, c, n);
    f32x4 x[D / 16];
    get_rows<D>(stage_k, g, c, x);
    __builtin_amdgcn_sched_barrier(0);
    const f32x4 st = product_rows<D>(x, qf);
    get_rows<D>(stage_v, g, c, x);
    const f32x4 dp = product_rows<D>(x, gf);
    get_columns<D>(stage_k, g, c, x);
    product_columns<D>(dq, x, weigh(blk, st, dp, kpos));
  }
  if (__builtin_expect(any_not_finite<D>(dq, s < n), 0)) {
    const int le = fresh(lane), g = le >> 4, c = le & 15;
#pragma unroll
    for (int b = 0; b < D / 16; ++b) dq[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int blk = wave; blk < t.nblocks; blk += FW) {
      pos = streamed_row<PERM>(t, perm, blk, c, n);
      f32x4 x[D / 16];
      load_columns<D>(Kh, pos, g, c, x);
      stage_rows<D>(stage_k, g, c, x, x);
      const f32x4 st = product_rows<D>(x, qf);
      load_columns<D>(Vh, pos, g, c, x);
      stage_rows<D>(stage_v, g, c, x, x);
      const f32x4 dp = product_rows<D>(x, gf);
      int kpos[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) kpos[i] = __shfl(pos, 4 * g + i);
      add_weighted_rows<D>(dq, stage_k, weigh(blk, st, dp, kpos), g, c);
    }
  }
  float ones[FW];
#pragma unroll
  for (int w = 0; w < FW; ++w) ones[w] = 1.f;
  f32x4 y[4 / FW][D / 64];
  merge_waves<D, FW>(area, 2 * Stage<D>::FLOATS, dq, ones, wave, lane, y);
  if (s >= n) return;
#pragma unroll
  for (int qh = 0; qh < 4 / FW * (D / 64); ++qh) {
    const int q = qh / (D / 64), h = qh % (D / 64), col = 64 * h + 16 * g + 4 * (wave + FW * q);
    float* at = reinterpret_cast<float*>(p.dQ) + (head_row0 + orig_q) * D + col;
    y[q][h] *= p.scale;
    if (p.accumulate) y[q][h] += *reinterpret_cast<const f32x4*>(at);
    *reinterpret_cast<f32x4*>(at) = y[q][h];
  }
}

// -------------------------------------------------------------------------------------- dK, dV
// A tile of 16 key slots; dV_j = sum_i P_ij dO_i, dK_j = scale * sum_i dS_ij Q_i over the queries whose window
// holds the key and over the query heads hg_begin .. hg_end - 1 of the group (they share a slot order, or there is
// one of them), whose (head, query block) pairs are dealt to the wavefronts in turn.
// OWN: every head has an order of its own.  The tile holds 16 keys in their original order, its band is all slots, and the slot
// of a key in a head's order is looked for in that order: for a few slots only, see launch_bwd_f32.
template <int D, bool PERM, int FW, bool OWN = false>
__global__ __launch_bounds__(64 * FW, 2) void bwd_dkv_f32_kernel(const Pass p, const unsigned num_tiles, const unsigned total_work) {
  __shared__ __attribute__((aligned(16))) float area[FW * 2 * Stage<D>::FLOATS];
  Tile t;
  if (!pick_tile(t, p, num_tiles, total_work, p.Hkv)) return;
  const int n = p.n;
  if constexpr (OWN) {
    t.lo = 0;
    t.nblocks = (n + FT - 1) / FT;
  } else {
    set_band(t, p, p.win.R, p.win.L);  // queries at slots s with -L <= t - s <= R, i.e. s in [t - R, t + L]
  }
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int hg0 = p.hq_only >= 0 ? p.hq_only : 0, heads = p.hq_only >= 0 ? 1 : p.g;
  const int32_t* __restrict__ perm = perm_of<PERM>(p, t.b, t.h * p.g + hg0);
  const size_t kv_row0 = ((size_t)t.b * p.Hkv + t.h) * n;

  const int k = t.s0 + c;  // this lane's key slot
  const int orig_k = PERM && !OWN ? perm[min(k, n - 1)] : min(k, n - 1);
  const int first_q = p.causal ? orig_k : -1;  // no query before it sees this key
  // query slot s sees the key iff 0 <= s - k + Rl <= LRl
  const int Rl = p.win.circular ? p.win.R : min(p.win.R, k);
  const unsigned LRl = (unsigned)(Rl + (p.win.circular ? p.win.L : min(p.win.L, max(n - 1 - k, 0))));
  float* stage_q = area + wave * 2 * Stage<D>::FLOATS;
  float* stage_g = stage_q + Stage<D>::FLOATS;
  f32x4 kf[D / 16], vf[D / 16], dk[D / 16], dv[D / 16];
  load_columns<D>(reinterpret_cast<const float*>(p.K) + kv_row0 * D, orig_k, g, c, kf);
  load_columns<D>(reinterpret_cast<const float*>(p.V) + kv_row0 * D, orig_k, g, c, vf);
#pragma unroll
  for (int b = 0; b < D / 16; ++b) dk[b] = dv[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float cs = p.scale * kLog2e;
  const int units = heads * t.nblocks;
  auto unit_row0 = [&](int u) -> size_t { return ((size_t)t.b * p.Hq + t.h * p.g + hg0 + min(u, units - 1) / t.nblocks) * n; };
  auto unit_order = [&](int u) { return perm_of<PERM>(p, t.b, t.h * p.g + min(u, units - 1) / t.nblocks); };
  auto unit_row = [&](int u) -> int {
    if constexpr (OWN) return unit_order(u)[min(FT * (min(u, units - 1) % t.nblocks) + c, n - 1)];
    else return streamed_row<PERM>(t, perm, min(u, units - 1) % t.nblocks, c, n);
  };
  const float* __restrict__ Q = reinterpret_cast<const float*>(p.Q);
  const float* __restrict__ dO = reinterpret_cast<const float*>(p.dO);
  int pos = unit_row(wave), pos1 = unit_row(wave + FW);
  f32x4 qn[D / 16], gn[D / 16];
  auto probabilities = [&](int u, const f32x4 st, const int* qpos, const float* lse2) -> f32x4 {  // of queries 4g + i for key c
    const int s0 = t.lo + FT * (u % t.nblocks) + 4 * g - k + Rl;
    int own_at = -(1 << 20);  // (a key without a slot is seen by no query)
    if constexpr (OWN) {
      const int32_t* __restrict__ order = unit_order(u);
      for (int s = 0; s < n; ++s) own_at = order[s] == orig_k ? s : own_at;
    }
    f32x4 pr;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      bool seen = ((unsigned)(s0 + i) <= LRl) & (first_q <= qpos[i]);
      if constexpr (OWN) {
        const int s = FT * (u % t.nblocks) + 4 * g + i;
        int r = s - own_at + p.win.R;
        if (p.win.circular) r = r < 0 ? r + n : r >= n ? r - n : r;
        seen = (s < n) & ((unsigned)r <= (unsigned)(p.win.L + p.win.R)) & (first_q <= qpos[i]);
      }
      const float pe = __builtin_amdgcn_exp2f(fmaf(st[i], cs, -lse2[i]));
      pr[i] = seen ? pe : 0.f;
    }
    return pr;
  };
  load_columns<D>(Q + unit_row0(wave) * D, pos, g, c, qn);
  load_columns<D>(dO + unit_row0(wave) * D, pos, g, c, gn);
  stage_rows<D>(stage_q, g, c, kf, kf);
  stage_rows<D>(stage_g, g, c, vf, vf);
  for (int u = wave; u < units; u += FW) {
    const size_t head_row0 = unit_row0(u), next_row0 = unit_row0(u + FW);
    wave_lds_sync();
    put_columns<D>(stage_q, g, c, qn);
    put_columns<D>(stage_g, g, c, gn);
    wave_lds_sync();
    int qpos[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) qpos[i] = __shfl(pos, 4 * g + i);
    float lse2[4], dd[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      lse2[i] = p.lse_in[head_row0 + qpos[i]] * kLog2e;
      dd[i] = p.Dsum[head_row0 + qpos[i]];
    }
    pos = pos1;
    load_columns<D>(Q + next_row0 * D, pos, g, c, qn);
    load_columns<D>(dO + next_row0 * D, pos, g, c, gn);
    pos1 = unit_row(u + 2 * FW);
    f32x4 x[D / 16];
    get_rows<D>(stage_q, g, c, x);
    __builtin_amdgcn_sched_barrier(0);
    const f32x4 st = product_rows<D>(x, kf);  // S: queries 4g + i, key c
    const f32x4 pr = probabilities(u, st, qpos, lse2);
    get_columns<D>(stage_g, g, c, x);
    product_columns<D>(dv, x, pr);
    get_rows<D>(stage_g, g, c, x);
    const f32x4 dp = product_rows<D>(x, vf);
    get_columns<D>(stage_q, g, c, x);
    f32x4 ds;
#pragma unroll
    for (int i = 0; i < 4; ++i) ds[i] = pr[i] == 0.f ? 0.f : pr[i] * (dp[i] - dd[i]);
    product_columns<D>(dk, x, ds);
  }
  if (__builtin_expect(any_not_finite<D>(dk, k < n) | any_not_finite<D>(dv, k < n), 0)) {
    const int le = fresh(lane), g = le >> 4, c = le & 15;
#pragma unroll
    for (int b = 0; b < D / 16; ++b) dk[b] = dv[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int u = wave; u < units; u += FW) {
      const size_t head_row0 = unit_row0(u);
      pos = unit_row(u);
      int qpos[4];
      float lse2[4], dd[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        qpos[i] = __shfl(pos, 4 * g + i);
        lse2[i] = p.lse_in[head_row0 + qpos[i]] * kLog2e;
        dd[i] = p.Dsum[head_row0 + qpos[i]];
      }
      f32x4 x[D / 16];
      load_columns<D>(Q + head_row0 * D, pos, g, c, x);
      stage_rows<D>(stage_q, g, c, x, x);
      const f32x4 pr = probabilities(u, product_rows<D>(x, kf), qpos, lse2);
      load_columns<D>(dO + head_row0 * D, pos, g, c, x);
      stage_rows<D>(stage_g, g, c, x, x);
      const f32x4 dp = product_rows<D>(x, vf);
      f32x4 ds;
#pragma unroll
      for (int i = 0; i < 4; ++i) ds[i] = pr[i] == 0.f ? 0.f : pr[i] * (dp[i] - dd[i]);
      add_weighted_rows<D>(dv, stage_g, pr, g, c);
      add_weighted_rows<D>(dk, stage_q, ds, g, c);
    }
  }
  // (lane numbers from a fresh copy: with them 167 or 168 registers at d = 64, three wavefronts per SIMD)
  const int le = fresh(lane), ge = le >> 4, ke = t.s0 + (le & 15);
  float ones[FW];
#pragma unroll
  for (int w = 0; w < FW; ++w) ones[w] = 1.f;
  f32x4 yk[4 / FW][D / 64], yv[4 / FW][D / 64];
  merge_waves<D, FW>(area, 2 * Stage<D>::FLOATS, dk, ones, wave, le, yk);
  __syncthreads();
  merge_waves<D, FW>(area, 2 * Stage<D>::FLOATS, dv, ones, wave, le, yv);
  if (ke >= n) return;
#pragma unroll
  for (int qh = 0; qh < 4 / FW * (D / 64); ++qh) {
    const int q = qh / (D / 64), h = qh % (D / 64), col = 64 * h + 16 * ge + 4 * (wave + FW * q);
    const size_t at = (kv_row0 + (PERM ? orig_k : ke)) * D + col;
    float* dK = reinterpret_cast<float*>(p.dK) + at;
    float* dV = reinterpret_cast<float*>(p.dV) + at;
    yk[q][h] *= p.scale;
    if (p.accumulate) {
      yk[q][h] += *reinterpret_cast<const f32x4*>(dK);
      yv[q][h] += *reinterpret_cast<const f32x4*>(dV);
    }
    *reinterpret_cast<f32x4*>(dK) = yk[q][h];
    *reinterpret_cast<f32x4*>(dV) = yv[q][h];
  }
}

bool f32_shape_ok(const Pass& p) {
  return (p.d == 64 || p.d == 128) && p.n >= 1 && p.B >= 1 && p.Hq >= 1 && p.g >= 1 && p.g * p.Hkv == p.Hq &&
         p.win.L >= 0 && p.win.R >= 0 && p.win.L < p.n && p.win.R < p.n &&
         (!p.win.circular || p.win.L + p.win.R + 1 <= p.n);
}

}  // namespace

// Wavefronts that share a tile's band: the most that are all resident at once.  A call with few tiles needs the split to
// occupy the chip and to shorten the chain of one tile (B1 H2 n1024 d64 w64, 128 tiles: forward 9.2 / 7.2 / 6.4 us with 1 / 2 / 4);
// past one round of workgroups every wavefront that shares a tile repeats its index and row round trips for nothing.  8 heads,
// w = 128, us with 1 / 2 / 4, on both sides of the lines:
//   tiles                  512                640                768                1000               1280               1536               2000
//   forward d = 64         13.0/10.8/8.6      13.8/11.8/10.6     14.0/12.0/10.6     14.7/13.0/13.7     18.6/15.8/17.4     19.4/18.6/19.8     21.5/20.9/22.8
//   dQ d = 64              13.7/12.4/11.8     15.4/13.9/13.5     15.8/14.1/14.1     16.4/15.5/18.0     22.3/19.4/22.9     22.9/20.4/23.9     26.2/29.6/30.0
//   dK, dV d = 64          18.8/16.5/13.4     20.0/17.6/17.0     20.8/18.5/17.5     22.1/20.3/24.6     29.6/25.5/28.3     29.8/27.9/29.4     33.9/38.9/37.6
//   forward d = 128        18.4/16.2/13.4     19.1/17.8/19.8     20.0/18.7/23.4     21.7/21.3/24.7     30.1/31.5/32.9     31.4/35.6/35.0     36.9/38.2/44.4
//   dQ d = 128             22.0/20.6/16.4     23.7/22.4/24.6     24.6/23.2/28.8     27.2/26.8/30.4     40.7/38.1/40.7     42.4/46.2/43.8     47.9/50.6/55.7
//   dK, dV d = 128         32.2/29.2/23.9     34.0/31.4/35.1     35.5/32.7/41.2     39.2/38.6/44.1     53.6/59.7/60.6     56.9/67.5/63.9     69.4/73.6/83.0
// `resident`: wavefronts that the registers let the 1024 SIMDs hold.  Four to a tile do not pay for a fourth on a SIMD.
static int wavefronts_per_tile(long tiles, int resident) {
  if (tiles * 4 <= (resident < 3072 ? resident : 3072)) return 4;
  return tiles * 2 <= resident ? 2 : 1;
}
// (the forward at d = 64: four a SIMD, less a few: B2 H8 n2039 w128, 2048 tiles, forward + backward 84.5 us with one, 88.9 with two)
constexpr int kResidentFwd64 = 4000, kResidentBwd64 = 3072, kResident128 = 2048;

#define SA_LAUNCH_F32_W(KERNEL_, W_)                                                                              \
  do {                                                                                                            \
    const dim3 block(64 * W_);                                                                                    \
    if (p.d == 64 && p.perm) hipLaunchKernelGGL((KERNEL_<64, true, W_>), grid, block, 0, st, p, t, w);            \
    else if (p.d == 64) hipLaunchKernelGGL((KERNEL_<64, false, W_>), grid, block, 0, st, p, t, w);                \
    else if (p.perm) hipLaunchKernelGGL((KERNEL_<128, true, W_>), grid, block, 0, st, p, t, w);                   \
    else hipLaunchKernelGGL((KERNEL_<128, false, W_>), grid, block, 0, st, p, t, w);                              \
  } while (0)
#define SA_LAUNCH_F32(KERNEL_, HEADS_, RES64_)                                                                              \
  do {                                                                                                            \
    const int tiles = (p.n + FT - 1) / FT;                                                                        \
    const long total = (long)tiles * (HEADS_)*p.B;                                                                \
    if (total > 0x7ffffff0L) return hipErrorInvalidValue;                                                         \
    const dim3 grid((unsigned)xcd_grid_blocks(total));                                                            \
    const unsigned t = (unsigned)tiles, w = (unsigned)total;                                                      \
    switch (wavefronts_per_tile(total, p.d == 64 ? RES64_ : kResident128)) {                                            \
      case 4: SA_LAUNCH_F32_W(KERNEL_, 4); break;                                                                 \
      case 2: SA_LAUNCH_F32_W(KERNEL_, 2); break;                                                                 \
      default: SA_LAUNCH_F32_W(KERNEL_, 1); break;                                                                \
    }                                                                                                             \
  } while (0)

hipError_t launch_fwd_f32(const Pass& p, hipStream_t st) {
  if (!f32_shape_ok(p)) return hipErrorInvalidValue;
  SA_LAUNCH_F32(fwd_f32_kernel, p.Hq, kResidentFwd64);
  return hipGetLastError();
}

static hipError_t launch_dkv_f32(const Pass& p, hipStream_t st) {
  SA_LAUNCH_F32(bwd_dkv_f32_kernel, p.Hkv, kResidentBwd64);
  return hipGetLastError();
}

// Grouped heads with permutations of their own: up to 64 slots one launch walks all slots of all heads of a group, beyond that a pass
// per head walks bands.  The passes are launches of 5 us one behind the other; whole sequences instead of bands cost more from 65
// slots on, and once the tiles are more than the chip takes in about a round.  Whole backward, w = 64, passes / one launch, us:
//   slots                              16          32          64          65          128
//   10 x 32 / 4 heads of 64            53.0/17.4   56.3/25.6   72.4/54.1   74.3/63.7   95.2/151
//   1 x 8 / 2 heads of 64              29.2/14.3   29.3/16.0   36.6/28.8   36.1/33.0   36.9/66.7
//   2 x 32 / 8 heads of 128            40.5/16.9   41.7/22.2   54.7/39.5   58.0/48.0   59.7/87.7
//   64 x 32 / 8 heads of 64, tiles     42.7/19.9   72.8/49.6   161/140 (2048)
//   500 x 8 / 4 heads of 64, tiles     56.2/44.1 (2000)        258/292 (8000); 33 slots (6000) 128/147
constexpr int kOwnOrderSlots = 64;
constexpr long kOwnOrderTiles = 2048;

hipError_t launch_bwd_f32(const Pass& p, hipStream_t st) {
  if (!f32_shape_ok(p)) return hipErrorInvalidValue;
  if (p.O_rows ? !p.Dsum_out : !p.Dsum) return hipErrorInvalidValue;
  SA_LAUNCH_F32(bwd_dq_f32_kernel, p.Hq, kResidentBwd64);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  Pass kv = p;
  if (p.O_rows) kv.Dsum = p.Dsum_out;  // the dQ kernel has left the row sums there
  if (!(p.perm && p.perm_H != 1 && p.g > 1)) return launch_dkv_f32(kv, st);
  // every query head of a group has its own slot order
  const int tiles = (p.n + FT - 1) / FT;
  const long total = (long)tiles * p.Hkv * p.B;
  if (p.n <= kOwnOrderSlots && total <= kOwnOrderTiles) {
    const dim3 grid((unsigned)xcd_grid_blocks(total)), block(64 * 4);
    if (p.d == 64) hipLaunchKernelGGL((bwd_dkv_f32_kernel<64, true, 4, true>), grid, block, 0, st, kv, (unsigned)tiles, (unsigned)total);
    else hipLaunchKernelGGL((bwd_dkv_f32_kernel<128, true, 4, true>), grid, block, 0, st, kv, (unsigned)tiles, (unsigned)total);
    return hipGetLastError();
  }
  // one pass per head, summed in place
  for (int hg = 0; hg < p.g; ++hg) {
    kv.hq_only = hg;
    kv.accumulate = hg == 0 ? p.accumulate : 1;
    e = launch_dkv_f32(kv, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace sa
