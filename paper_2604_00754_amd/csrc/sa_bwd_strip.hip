// bf16 backward of Stochastic Attention in one pass (d = 64, one query head per KV head, windows up to 257 slots).
//
// The gradient is that of sa_bwd_mfma.hip, which needs two kernels because one owns queries and the other keys: S, dP and
// the exponentials are formed in both, and Q, K, V and dO are read by both.  Here a workgroup walks a strip of slots of one
// head and forms every block of scores once.  It owns the queries and the keys of its strip; the pairs across the strip's
// ends are formed by both neighbours (one for dQ, the other for dK and dV), so nothing is summed between workgroups.
//
//   interval i      the 32 query slots of block i against the NB blocks of 32 key slots that their windows reach
//   active wave     one key block for NB intervals: K and V as operands, dK and dV as accumulators in registers.
//                   S = Q K^T, dP = dO V^T, P, dS (left in LDS for dQ), dV^T += dO^T P, dK^T += Q^T dS
//   the other three between two key blocks, one interval each: (1) dQ of block i - 1 (dQ^T = K^T dS^T over the NB blocks, K and dS
//                   from LDS), (2) dK and dV of the finished key block leave, K and V of the next are requested, (3) dQ of
//                   block i - 2 leaves; D, LSE, positions and rotation of the query block that comes next
// With NB + 3 waves every interval has NB active waves and one in each of the three other roles; a wave's key blocks are
// NB + 3 apart.  One barrier per interval; dS and the rows of dQ on their way out have two buffers.
//
// Bound: the issue of vector instructions (per SIMD and interval about 3000 cycles of 4500 at NB = 9: 150 instructions and 16
// exponentials for a block of 32 x 32, 2.25 blocks a SIMD, 1000 instructions for the three other roles), then the LDS latencies of the
// slowest role.  Measured against the two kernels (us): 64 heads, 8192 slots, d = 64, w = 256, one call alone 242 -> 158, calls in a row
// 238 -> 146, the one-sided branch 223 -> 150; 256 heads, 4096 slots with rotations 590 -> 342 (430 while dK's table rows went through LDS to the
// accumulators); other sizes at strips_are_faster().  NB + 3 waves of 168 registers at NB = 9 fill a CU; its LDS (155 136 bytes, with rotations
// 163 328 of the 163 840) holds query tiles three intervals ahead and one K tile a wave.  The strip is as long as one round of 256
// workgroups allows (2048 slots there): every strip walks its windows' reach on top of its own slots.
#include "sa_common.h"
#include "sa_mfma.h"

#include <algorithm>
#include <cmath>

namespace sa {
namespace {

constexpr int D = 64;
constexpr int RB = 32;                 // slots of a block
constexpr int TILE = RB * D * 2;       // bytes of a block's rows, unpadded, 16-byte chunks swizzled (swz<64>)
constexpr int DS_TILE = RB * RB * 2;   // bytes of one block of dS
constexpr int ROWS_F32 = RB * D * 4;   // bytes of 32 fp32 rows on their way out
constexpr int kCUs = 256;
constexpr int kMostSlots = 4096;       // slots of a strip
constexpr int kMostReach = 256;        // L + R
constexpr int kMostPos = kMostSlots + 2 * kMostReach + 4 * RB;  // slots of the blocks that a strip walks

enum { CAUSAL_NONE = 0, CAUSAL_I16 = 2 };
// The rows on their way: written, added to what the outputs hold (second branch of the gated sum), or turned (Q arrives
// unrotated, dQ leaves unrotated).
enum { ROWS_PLAIN = 0, ROWS_ADD = 1, ROWS_TURN = 2 };
typedef short s16x2 __attribute__((ext_vector_type(2)));

template <int NB, int ROWS>
struct Cfg {
  static constexpr int W = NB + 3;        // waves
  static constexpr int NT = 64 * W;
  static constexpr int NQ = 4;            // query tiles: requested three intervals early
  static constexpr int OFF_Q = 0;                              // Q | dO tiles
  static constexpr int OFF_K = OFF_Q + NQ * 2 * TILE;
  static constexpr int OFF_V = OFF_K + W * TILE;               // one K tile a wave; V tiles until their wave has them in registers
  static constexpr int OFF_DS = OFF_V + 2 * TILE;              // dS [2][NB][32 keys][32 queries]
  static constexpr int OFF_DQ = OFF_DS + 2 * NB * DS_TILE;     // dQ rows, fp32, [2]
  static constexpr int VALS = RB * 16 + RB * 2;                // operand rows of -LSE / scale and -D | 16-bit positions in accumulator order
  static constexpr int OFF_VAL = OFF_DQ + 2 * ROWS_F32;
  static constexpr int OFF_POS = OFF_VAL + NQ * VALS;          // positions of the strip's slots and of those its windows reach
  static constexpr int OFF_TURN = OFF_POS + kMostPos * 2;      // fp32 rows of dK that are turned on their way out
  static constexpr int LDS_BYTES = OFF_TURN + (ROWS == ROWS_TURN ? ROWS_F32 : 0);
  static_assert(LDS_BYTES <= 160 * 1024, "LDS of a CU");
};

struct Strips {
  int per_head, slots;   // strips of a head, slots of a strip (a multiple of 32)
};

// Position of tile row r in accumulator order: accumulator 4*mq + x of lane group g2 is row 8*mq + 4*g2 + x.
__device__ __forceinline__ int acc_order_pos(int r) { return (((r >> 2) & 1) << 4) | (((r >> 3) & 3) << 2) | (r & 3); }

// Accumulators (lane = row c32, four consecutive columns per quad) into 32 fp32 rows of LDS, 16-byte chunks XORed with the row.
__device__ __forceinline__ void put_rows(char* area, const f32x16& acc, int col_chunk0, int lane) {
  const int g2 = lane >> 5, c32 = lane & 31;
#pragma unroll
  for (int mq = 0; mq < 4; ++mq) {
    const f32x4 v = {acc[4 * mq], acc[4 * mq + 1], acc[4 * mq + 2], acc[4 * mq + 3]};
    *reinterpret_cast<f32x4*>(area + c32 * (D * 4) + (((col_chunk0 + 2 * mq + g2) ^ (c32 & 15)) * 16)) = v;
  }
}
// columns 8*c .. 8*c + 7 of row `row`
__device__ __forceinline__ void get_row8(const char* area, int row, int c, float* x) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(area + row * (D * 4) + (((2 * c + h) ^ (row & 15)) * 16));
#pragma unroll
    for (int e = 0; e < 4; ++e) x[4 * h + e] = v[e];
  }
}

// Reads by 32-bit LDS address.  Tiles start on multiples of their size, so the chunks of a lane's row differ in address bits
// that can be flipped after the tile's base is added: one address register per tile instead of one per chunk.
typedef __attribute__((address_space(3))) const bf16x8* lds_bf16x8;
typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
__device__ __forceinline__ bf16x8 lds_row(uint32_t at) { return *(lds_bf16x8)(uintptr_t)(at); }
// A operand X^T of 16 rows (lds_read_transposed_swz): `at` = the lane's 8 bytes of the first 8 rows in a tile of d = 64
__device__ __forceinline__ bf16x8 lds_transposed(uint32_t at) {
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(uintptr_t)(at));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(uintptr_t)((at ^ 32) + 8 * D * 2));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// What a row adds to all its products enters as one more product: three bf16 values that sum to it to the last bit of fp32,
// against ones.  (In accumulator order a lane needs 16 rows' values, which would be four 16-byte reads each.)  Eight contraction indices, the
// lane group's four: S and dP have an operand each, so that an infinite D stays out of S and of dV.
__device__ __forceinline__ void put_split(char* at, float x) {
  const float h = bf16lo(pack_bf16(x, 0.f)), m = bf16lo(pack_bf16(x - h, 0.f));
  *reinterpret_cast<u32x2*>(at) = u32x2{pack_bf16(h, m), pack_bf16(x - h - m, 0.f)};
}
__device__ __forceinline__ f32x16 mfma_row_values(s16x4 rows, s16x4 ones) {
  const f32x16 zero = {};
  return __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(rows, ones, zero, 0, 0, 0);
}
constexpr float kFar = 1e30f;  // an LSE of +infinity (a gate of zero): as far as a finite operand can be

// 16 bytes at a byte offset (scalar base, 32-bit lane offset)
__device__ __forceinline__ u32x4 row_at_offset(const void* base, uint32_t off) {
  return *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(base) + off);
}
__device__ __forceinline__ u32x4 table_at_offset(const void* base, uint32_t off) {
  return *reinterpret_cast<const table_u32x4*>(reinterpret_cast<const char*>(base) + off);
}
__device__ __forceinline__ void store_at_offset(void* base, uint32_t off, u32x4 v) {
  __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(reinterpret_cast<char*>(base) + off));
}

// x of the lane that the DPP control names
template <int CTRL>
__device__ __forceinline__ float from_lane(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}

// What lanes hold of 32 fp32 rows in LDS, turned back by the angles of their rows (the transpose of RoPE), times mul, as 16-byte
// chunks of bf16 rows.  Lane (r8, c8) turns pairs 4 c8 .. 4 c8 + 3 of rows 8 v + r8; t = their (cos, sin), 32 bytes a row.  Split halves:
// a lane has four columns of either half, and neighbours trade so that the even one leaves with eight of the lower half and the
// odd one with eight of the upper.  Returns the lane's chunk.
__device__ __forceinline__ int turn_rows(const char* area, const u32x4* t, float mul, int interleaved, int lane, u32x4* w) {
  const int r8 = lane >> 3, c8 = lane & 7;
  f32x4 a[4], b[4];
  auto fetch = [&](int v) {
    const int row = 8 * v + r8;
    a[v] = *reinterpret_cast<const f32x4*>(area + row * (D * 4) + (((interleaved ? 2 * c8 : c8) ^ (row & 15)) * 16));
    b[v] = *reinterpret_cast<const f32x4*>(area + row * (D * 4) + (((interleaved ? 2 * c8 + 1 : 8 + c8) ^ (row & 15)) * 16));
  };
  fetch(0);
  fetch(1);
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    if (v == 1) { fetch(2); fetch(3); }
    __builtin_amdgcn_sched_barrier(0);
    const f32x4 t0 = __builtin_bit_cast(f32x4, t[2 * v]), t1 = __builtin_bit_cast(f32x4, t[2 * v + 1]);
    f32x4 x, y;
    if (interleaved) {
      x = f32x4{a[v][0] * t0[0] + a[v][1] * t0[1], a[v][1] * t0[0] - a[v][0] * t0[1], a[v][2] * t0[2] + a[v][3] * t0[3], a[v][3] * t0[2] - a[v][2] * t0[3]};
      y = f32x4{b[v][0] * t1[0] + b[v][1] * t1[1], b[v][1] * t1[0] - b[v][0] * t1[1], b[v][2] * t1[2] + b[v][3] * t1[3], b[v][3] * t1[2] - b[v][2] * t1[3]};
    } else {
      x = f32x4{a[v][0] * t0[0] + b[v][0] * t0[1], a[v][1] * t0[2] + b[v][1] * t0[3], a[v][2] * t1[0] + b[v][2] * t1[1], a[v][3] * t1[2] + b[v][3] * t1[3]};
      y = f32x4{b[v][0] * t0[0] - a[v][0] * t0[1], b[v][1] * t0[2] - a[v][1] * t0[3], b[v][2] * t1[0] - a[v][2] * t1[1], b[v][3] * t1[2] - a[v][3] * t1[3]};
    }
    const u32x2 lo = {pack_bf16(x[0] * mul, x[1] * mul), pack_bf16(x[2] * mul, x[3] * mul)};
    const u32x2 hi = {pack_bf16(y[0] * mul, y[1] * mul), pack_bf16(y[2] * mul, y[3] * mul)};
    if (interleaved) {
      w[v] = u32x4{lo[0], lo[1], hi[0], hi[1]};
    } else {
      const bool odd = c8 & 1;
      u32x2 got;
#pragma unroll
      for (int e = 0; e < 2; ++e)  // quad_perm [1,0,3,2]
        got[e] = (uint32_t)__builtin_amdgcn_mov_dpp((int)(odd ? lo[e] : hi[e]), 0xB1, 0xf, 0xf, true);
      w[v] = odd ? u32x4{got[0], got[1], hi[0], hi[1]} : u32x4{lo[0], lo[1], got[0], got[1]};
    }
  }
  return interleaved ? c8 : (c8 & 1) * 4 + (c8 >> 1);
}

// The lane's number, formed anew at each use: a copy that the optimiser cannot trace, so that what a role derives from it is
// formed in that role instead of being kept in registers through all the others.
__device__ __forceinline__ int fresh(int lane) {
  asm volatile("" : "+v"(lane));
  return lane;
}

template <int NB, int CAUSAL, int ROWS>
__global__ __launch_bounds__((Cfg<NB, ROWS>::NT)) void bwd_strip_bf16_kernel(const Pass p, const Strips strips, const long total_work) {
  using C = Cfg<NB, ROWS>;
  __shared__ __attribute__((aligned(1024))) char smem[C::LDS_BYTES];
  const long work = xcd_work_index(total_work);
  if (work < 0) return;
  const int strip = (int)(work % strips.per_head);
  const int head = (int)(work / strips.per_head);
  const int hq = head % p.Hq, b = head / p.Hq;

  const int tid = threadIdx.x, lane0 = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = p.n, L = p.win.L, R = p.win.R;
  const bool circular = p.win.circular != 0;
  const int32_t* __restrict__ perm = p.perm ? p.perm + (size_t)perm_slice_index(p.perm_B, p.perm_H, b, hq) * n : nullptr;
  const size_t row0 = (size_t)head * n;
  const bf16_t* __restrict__ Qh = reinterpret_cast<const bf16_t*>(p.Q) + row0 * D;
  const bf16_t* __restrict__ Gh = reinterpret_cast<const bf16_t*>(p.dO) + row0 * D;
  const bf16_t* __restrict__ Kh = reinterpret_cast<const bf16_t*>(p.K) + row0 * D;
  const bf16_t* __restrict__ Vh = reinterpret_cast<const bf16_t*>(p.V) + row0 * D;
  const bf16_t* __restrict__ Oh = p.O_rows ? reinterpret_cast<const bf16_t*>(p.O_rows) + row0 * D : nullptr;

  // the strip's slots, the query and key slots it needs, and the block grids: query block i starts at Q0 + 32 i, and the
  // windows of its queries start with key block i
  const int k0 = strip * strips.slots, k1 = min(k0 + strips.slots, n);
  const int q_lo = circular ? k0 - R : max(k0 - R, 0), q_hi = circular ? k1 - 1 + L : min(k1 - 1 + L, n - 1);
  const int t_lo = circular ? k0 - L : max(k0 - L, 0), t_hi = circular ? k1 - 1 + R : min(k1 - 1 + R, n - 1);
  const int Q0 = k0 - (k0 - q_lo + RB - 1) / RB * RB;
  const int T0 = Q0 - L;
  const int nqb = (q_hi - Q0) / RB + 1;
  const int nact = (L + R + RB - 1) / RB + 1;  // key blocks that the windows of 32 neighbouring queries reach
  const int last = max(nqb + 1, (k1 - 1 - T0) / RB + 2);  // the interval in which the last rows (of dQ; of dK and dV) leave

  auto query_block_owned = [&](int i) { return Q0 + RB * i < k1 && Q0 + RB * i + RB > k0; };
  auto key_block_owned = [&](int j) { return T0 + RB * j < k1 && T0 + RB * j + RB > k0; };

  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
  // positions of the slots of all blocks, from T0 on; slots that no pair needs get a neighbour's
  uint16_t* const pos_lds = reinterpret_cast<uint16_t*>(smem + C::OFF_POS);
  const int nkb = nqb + nact - 1, p_lo = min(q_lo, t_lo), p_hi = max(q_hi, t_hi);
  for (int s = tid; s < nkb * RB; s += C::NT)
    pos_lds[s] = (uint16_t)slot_to_orig(perm, wrap_slot(min(max(T0 + s, p_lo), p_hi), n));
  const uint16_t* const qpos_lds = pos_lds + (Q0 - T0);
  // byte offset of a row of d = 64 inside its head (n <= 65535 rows)
  auto query_row = [&](int i, int r) { return (uint32_t)qpos_lds[RB * i + r] * (uint32_t)(D * 2); };
  auto key_row = [&](int j, int r) { return (uint32_t)pos_lds[RB * j + r] * (uint32_t)(D * 2); };
  // a wave moves 8 rows with one instruction, lane's chunk lane % 8 of rows 8 v + lane / 8: the logical chunk it holds
  auto lane_chunk = [](int lane, int v) {
    const int r8 = lane >> 3;
    return (lane & 7) ^ ((((r8 >> 1) & 1) << 2) | (r8 >> 2)) ^ ((v & 1) << 1);
  };
  const float cs = p.scale * kLog2e;

  // the active wave, by the intervals it has left, that requests a query block (3 at least: key block 0 for query block 0; six
  // instead of three: 542 -> 533 us for the gated training step)
  constexpr int kAsks = NB - 3 > 3 ? NB - 3 : 3;
  int i = -(NB + 2);  // interval; the first wave requests key block 0
  // the end of an interval: what this wave wrote to LDS is there before the barrier; loads and stores stay under way
  auto next_interval = [&]() -> bool {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    return ++i > last;
  };

  // dQ of query block i - 1: dQ^T = K^T dS^T over its key blocks
  auto form_dq = [&]() {
    const int iq = i - 1;
    if (iq < 0 || iq >= nqb || !query_block_owned(iq)) return;
    const int lane = fresh(lane0);
    const char* ds = smem + C::OFF_DS + (iq & 1) * (NB * DS_TILE);
    const int first = iq % C::W;
    // dS tiles: row = key, 64 bytes, 16-byte chunks XORed with bits 2..3 of the row (a lane writes 8 bytes of its own key's row)
    int ds_tr[2];
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      const int G = lane >> 4, j16 = lane & 15;
      const int row = 4 * (G >> 1) + (j16 >> 2) + 8 * hf, col = 16 * (G & 1) + 4 * (j16 & 3);
      ds_tr[hf] = row * RB + (((col >> 3) ^ ((row >> 2) & 3)) << 3) + (col & 7);
    }
    bf16x8 ka[2][4], da[2][2];  // the operands of the next key block are under way while the products of one issue
    f32x16 acc[2];
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[0][e] = acc[1][e] = 0.f;
    auto operands = [&](int ph, bf16x8* k4, bf16x8* d2) {
      const int slot = first + ph < C::W ? first + ph : first + ph - C::W;
      const char* Kt = smem + C::OFF_K + slot * TILE + lane * 16;
      const bf16_t* dst = reinterpret_cast<const bf16_t*>(ds + ph * DS_TILE);
#pragma unroll
      for (int c = 0; c < 2; ++c) d2[c] = lds_read_transposed_swz(dst + 16 * c * RB, ds_tr);
#pragma unroll
      for (int m = 0; m < 4; ++m) k4[m] = *reinterpret_cast<const bf16x8*>(Kt + m * 1024);
    };
    operands(0, ka[0], da[0]);
#pragma unroll
    for (int ph = 0; ph < NB; ++ph) {
      if (ph >= nact) break;
      if (ph + 1 < NB) operands(ph + 1, ka[(ph + 1) & 1], da[(ph + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int m = 0; m < 4; ++m) acc[m & 1] = mfma_bf16(ka[ph & 1][2 * (m & 1) + (m >> 1)], da[ph & 1][m >> 1], acc[m & 1]);
      __builtin_amdgcn_sched_barrier(0);
    }
    put_rows(smem + C::OFF_DQ + (iq & 1) * ROWS_F32, acc[0], 0, lane);
    put_rows(smem + C::OFF_DQ + (iq & 1) * ROWS_F32, acc[1], 8, lane);
  };

  bf16_t* const dQh = reinterpret_cast<bf16_t*>(p.dQ) + row0 * D;
  bf16_t* const dKh = reinterpret_cast<bf16_t*>(p.dK) + row0 * D;
  bf16_t* const dVh = reinterpret_cast<bf16_t*>(p.dV) + row0 * D;
  const float* const rope = p.rope_table;  // (cos, sin) of D / 2 pairs a row

  __syncthreads();
  for (int w = 0; w < wave; ++w)
    if (next_interval()) return;

  f32x16 dk[2], dv[2];
  for (int j = wave;; j += C::W) {
    const uint32_t ktile = C::OFF_K + (uint32_t)wave * TILE;
    // ---- between two key blocks, first interval (i = j - NB - 2)
    __builtin_amdgcn_s_setprio(2);
    const int iq = i + 3;                       // the query block of which this wave brings in what goes with its rows
    const bool want_q = iq >= 0 && iq < nqb;
    const int jp = j - C::W;                    // the key block that this wave has finished
    const bool out_kv = jp >= 0 && key_block_owned(jp);
    form_dq();
    __builtin_amdgcn_sched_barrier(0);
    u32x4 aux[8] = {};  // what the rows of dK and dV hold already, or the rows of the rotation table they need
    if (out_kv && (ROWS == ROWS_ADD || (ROWS == ROWS_TURN && p.rope_dk))) {
      const int lane = fresh(lane0), r8 = lane >> 3;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const uint32_t row = key_row(jp, 8 * v + r8), c = (uint32_t)lane_chunk(lane, v) * 16;
        if (ROWS == ROWS_ADD) {
          aux[v] = row_at_offset(dKh, row + c);
          aux[4 + v] = row_at_offset(dVh, row + c);
        } else {
#pragma unroll
          for (int h = 0; h < 2; ++h) aux[2 * v + h] = table_at_offset(rope, 2 * row + (lane & 7) * 32 + h * 16);
        }
      }
    }
    int pos_q = 0;  // position of this lane's query slot (both halves of the wave alike)
    u32x4 orow[4] = {};
    float lse = 0.f, dsum = 0.f;
    auto request_scalars = [&]() {
      const int lane = fresh(lane0), r8 = lane >> 3;
      pos_q = qpos_lds[want_q ? RB * iq + (lane & 31) : 0];
      if (want_q) {
        lse = p.lse_in[row0 + pos_q];
        if (!Oh) dsum = p.Dsum[row0 + pos_q];
        if (Oh) {
#pragma unroll
          for (int v = 0; v < 4; ++v) orow[v] = row_at_offset(Oh, query_row(iq, 8 * v + r8) + (uint32_t)lane_chunk(lane, v) * 16);
        }
      }
    };
    // (in the interval that is the shorter one: gated step 549 us with both branches' in the second, 533 here; a plain branch whose row
    // sums are formed here, w = 128, 64 heads of 8192 slots, 135 us here, 123 in the second)
    const bool scalars_later = ROWS == ROWS_PLAIN && Oh;
    if (!scalars_later) request_scalars();
    if (next_interval()) return;

    // ---- second interval: dK and dV of the finished block leave
    const bool out_q = i - 1 >= 0 && i - 1 < nqb && query_block_owned(i - 1);  // in the next interval
    // dK and dV take the way through LDS (this wave's K tile, which dQ no longer needs, and its V tile): out of the accumulators
    // a lane has 8-byte pieces of its own row; what comes in and goes out of memory are whole rows.
    const uint32_t vtile = C::OFF_V + (uint32_t)(i & 1) * TILE;
    if (out_kv) {
      const int lane = fresh(lane0), g2 = lane >> 5, c32 = lane & 31, r8 = lane >> 3;
      const uint32_t own = (uint32_t)(c32 * D * 2 + swz<D>(c32) * 16);  // 16-byte chunk c of the lane's row: ^ 16 c
      if (ROWS == ROWS_ADD) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          *reinterpret_cast<u32x4*>(smem + ktile + v * 1024 + lane * 16) = aux[v];
          *reinterpret_cast<u32x4*>(smem + vtile + v * 1024 + lane * 16) = aux[4 + v];
        }
        wave_lds_sync();
      }
      const bool turn = ROWS == ROWS_TURN && p.rope_dk;
      auto put = [&](const f32x16* acc, float mul, uint32_t tile) {
        u32x2 old[8];
        if (ROWS == ROWS_ADD) {
#pragma unroll
          for (int c = 0; c < 8; ++c) old[c] = *reinterpret_cast<const u32x2*>(smem + tile + (own ^ (16 * c)) + 8 * g2);
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          float x[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] = acc[c >> 2][4 * (c & 3) + e] * mul;
          if (ROWS == ROWS_ADD) {
            x[0] += bf16lo(old[c][0]); x[1] += bf16hi(old[c][0]);
            x[2] += bf16lo(old[c][1]); x[3] += bf16hi(old[c][1]);
          }
          *reinterpret_cast<u32x2*>(smem + tile + (own ^ (16 * c)) + 8 * g2) = u32x2{pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3])};
        }
      };
      if (turn) {
        put_rows(smem + C::OFF_TURN, dk[0], 0, lane);
        put_rows(smem + C::OFF_TURN, dk[1], 8, lane);
      } else {
        put(dk, p.scale, ktile);
      }
      put(dv, 1.f, vtile);
      wave_lds_sync();
      uint32_t at[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) at[v] = key_row(jp, 8 * v + r8);
      // one tensor at a time where the rotation's registers leave no room for both
      auto tiles_out = [&](bool with_k, bool with_v) {
        u32x4 wk[4], wv[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          if (with_k) wk[v] = *reinterpret_cast<const u32x4*>(smem + ktile + v * 1024 + lane * 16);
          if (with_v) wv[v] = *reinterpret_cast<const u32x4*>(smem + vtile + v * 1024 + lane * 16);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int s = T0 + RB * jp + 8 * v + r8;
          if (s >= k0 && s < k1) {
            const uint32_t to = at[v] + (uint32_t)lane_chunk(lane, v) * 16;
            if (with_k) store_at_offset(dKh, to, wk[v]);
            if (with_v) store_at_offset(dVh, to, wv[v]);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      };
      tiles_out(ROWS != ROWS_TURN, true);
      if (turn) {
        u32x4 w[4];
        const int c = turn_rows(smem + C::OFF_TURN, aux, p.scale, p.rope_interleaved, lane, w);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int s = T0 + RB * jp + 8 * v + r8;
          if (s >= k0 && s < k1) store_at_offset(dKh, at[v] + c * 16, w[v]);
        }
      } else if (ROWS == ROWS_TURN) {
        tiles_out(true, false);
      }
    }
    __builtin_amdgcn_sched_barrier(0);  // the accumulators' registers are free from here on
    u32x4 auxq[8] = {};
    if (out_q && ROWS != ROWS_PLAIN) {
      const int lane = fresh(lane0), r8 = lane >> 3, c8 = lane & 7;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const uint32_t row = query_row(i - 1, 8 * v + r8);
        if (ROWS == ROWS_ADD) auxq[v] = row_at_offset(dQh, row + c8 * 16);
        else {
#pragma unroll
          for (int h = 0; h < 2; ++h) auxq[2 * v + h] = table_at_offset(rope, 2 * row + c8 * 32 + h * 16);
        }
      }
    }
    u32x4 tq[8] = {};
    {
      const int lane = fresh(lane0), r8 = lane >> 3, c8 = lane & 7;
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the rows have been read: their tiles take the next key block
      // past the last key block nothing is requested (this wave's tiles then hold old rows that no product reads): every request has been waited
      // for when a wave ends, and one-block strips bring in the blocks they need and no more
      if (j < nkb) {
        uint32_t goff[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) goff[v] = key_row(j, 8 * v + r8) + (uint32_t)lane_chunk(lane, v) * 16;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          load_to_lds_16(Kh, goff[v], lds0 + ktile + v * 1024);
          load_to_lds_16(Vh, goff[v], lds0 + vtile + v * 1024);
        }
      }
      if (scalars_later) request_scalars();
      if (ROWS == ROWS_TURN && want_q) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const uint32_t row = query_row(iq, 8 * v + r8);
#pragma unroll
          for (int h = 0; h < 2; ++h) tq[2 * v + h] = table_at_offset(rope, 2 * row + c8 * 32 + h * 16);
        }
      }
    }
    if (next_interval()) return;

    // ---- third interval: dQ of block i - 2 leaves
    if (out_q) {
      const int lane = fresh(lane0), r8 = lane >> 3, c8 = lane & 7;
      const int slot0 = Q0 + RB * (i - 2);
      char* const area = smem + C::OFF_DQ + (i & 1) * ROWS_F32;
      uint32_t at[4];
      u32x4 w[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) at[v] = query_row(i - 2, 8 * v + r8);
      int c = c8;
      if (ROWS == ROWS_TURN) {
        c = turn_rows(area, auxq, p.scale, p.rope_interleaved, lane, w);
      } else {
        float x[4][8];
#pragma unroll
        for (int v = 0; v < 4; ++v) get_row8(area, 8 * v + r8, c8, x[v]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float v0 = x[v][2 * e] * p.scale, v1 = x[v][2 * e + 1] * p.scale;
            if (ROWS == ROWS_ADD) {
              v0 += bf16lo(auxq[v][e]);
              v1 += bf16hi(auxq[v][e]);
            }
            w[v][e] = pack_bf16(v0, v1);
          }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int s = slot0 + 8 * v + r8;
        if (s >= k0 && s < k1) store_at_offset(dQh, at[v] + c * 16, w[v]);
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the query tiles requested two intervals ago (not seen by the compiler)
    if (want_q) {
      const int lane = fresh(lane0), r8 = lane >> 3, c8 = lane & 7;
      char* const vals = smem + C::OFF_VAL + (iq & 3) * C::VALS;
      char* const qt = smem + C::OFF_Q + (iq & 3) * 2 * TILE;
      if (ROWS == ROWS_TURN) {  // Q arrives unrotated: RoPE on the query's original position; a lane turns pairs 4 c8 .. 4 c8 + 3
        // split halves: 8 bytes of chunk c8 / 2 and of the chunk four further; adjacent pairs: chunk c8
        const int step = p.rope_interleaved ? 8 : 64;
        u32x2 a[4], bb[4];
        char* al[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = 8 * v + r8, c = p.rope_interleaved ? c8 : c8 >> 1;
          al[v] = qt + row * (D * 2) + ((c ^ swz<D>(row)) * 16) + (p.rope_interleaved ? 0 : (c8 & 1) * 8);
          a[v] = *reinterpret_cast<const u32x2*>(al[v]);
          bb[v] = *reinterpret_cast<const u32x2*>(smem + ((al[v] - smem) ^ step));
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const f32x4 t0 = __builtin_bit_cast(f32x4, tq[2 * v]), t1 = __builtin_bit_cast(f32x4, tq[2 * v + 1]);
          const float a0 = bf16lo(a[v][0]), a1 = bf16hi(a[v][0]), a2 = bf16lo(a[v][1]), a3 = bf16hi(a[v][1]);
          const float b0 = bf16lo(bb[v][0]), b1 = bf16hi(bb[v][0]), b2 = bf16lo(bb[v][1]), b3 = bf16hi(bb[v][1]);
          u32x2 oa, ob;
          if (p.rope_interleaved) {
            oa = u32x2{pack_bf16(a0 * t0[0] - a1 * t0[1], a0 * t0[1] + a1 * t0[0]), pack_bf16(a2 * t0[2] - a3 * t0[3], a2 * t0[3] + a3 * t0[2])};
            ob = u32x2{pack_bf16(b0 * t1[0] - b1 * t1[1], b0 * t1[1] + b1 * t1[0]), pack_bf16(b2 * t1[2] - b3 * t1[3], b2 * t1[3] + b3 * t1[2])};
          } else {
            oa = u32x2{pack_bf16(a0 * t0[0] - b0 * t0[1], a1 * t0[2] - b1 * t0[3]), pack_bf16(a2 * t1[0] - b2 * t1[1], a3 * t1[2] - b3 * t1[3])};
            ob = u32x2{pack_bf16(a0 * t0[1] + b0 * t0[0], a1 * t0[3] + b1 * t0[2]), pack_bf16(a2 * t1[1] + b2 * t1[0], a3 * t1[3] + b3 * t1[2])};
          }
          *reinterpret_cast<u32x2*>(al[v]) = oa;
          *reinterpret_cast<u32x2*>(smem + ((al[v] - smem) ^ step)) = ob;
        }
      }
      if (Oh) {  // D = rowsum(dO o O): eight lanes share a row
        u32x4 gw[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) gw[v] = *reinterpret_cast<const u32x4*>(qt + TILE + v * 1024 + lane * 16);
        float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            part[v] = fmaf(bf16hi(gw[v][e]), bf16hi(orow[v][e]), fmaf(bf16lo(gw[v][e]), bf16lo(orow[v][e]), part[v]));
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) part[v] += from_lane<0xB1>(part[v]);  // quad_perm [1,0,3,2]
#pragma unroll
        for (int v = 0; v < 4; ++v) part[v] += from_lane<0x4E>(part[v]);  // quad_perm [2,3,0,1]
#pragma unroll
        for (int v = 0; v < 4; ++v) part[v] += from_lane<0x141>(part[v]);  // row_half_mirror: the other quad of the eight
        if (c8 == 0) {
#pragma unroll
          for (int v = 0; v < 4; ++v) put_split(vals + (8 * v + r8) * 16 + 8, -part[v]);
        }
      }
      if (lane < 32) {
        const float l = lse * (1.f / p.scale);
        put_split(vals + lane * 16, -(l > kFar ? kFar : l));
        if (!Oh) put_split(vals + lane * 16 + 8, -dsum);
        if (CAUSAL == CAUSAL_I16) reinterpret_cast<short*>(vals + RB * 16)[acc_order_pos(lane)] = (short)(pos_q - 32767);
      }
    }
    // ---- what the active intervals keep in registers
    const int lane_a = fresh(lane0), g2 = lane_a >> 5, c32 = lane_a & 31;
    const uint32_t row_at = lds0 + (uint32_t)(c32 * D + 8 * (g2 ^ swz<D>(c32))) * 2;  // chunk g2 of row c32; chunk 2 kk + g2: ^ 32 kk
    uint32_t tr_at;  // columns 0..31 of the lane's row of a transposing read; columns 32..63: ^ 64
    {
      const int G = lane_a >> 4, j16 = lane_a & 15, row = 4 * (G >> 1) + (j16 >> 2), col = 16 * (G & 1) + 4 * (j16 & 3);
      tr_at = lds0 + (uint32_t)(row * D + 8 * ((col >> 3) ^ swz<D>(row)) + (col & 7)) * 2;
    }
    const int orig_k = pos_lds[RB * min(j, nkb - 1) + c32];
    bf16x8 kf[D / 16], vf[D / 16];
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) {
      kf[kk] = lds_row((row_at + ktile) ^ (32 * kk));
      vf[kk] = lds_row((row_at + vtile) ^ (32 * kk));
    }
    // ones against the three values of -LSE / scale, of -D
    const uint32_t one2 = g2 == 0 ? 0x3F803F80u : 0u;
    const s16x4 ones = __builtin_bit_cast(s16x4, (u32x2{one2, one2 & 0xffffu}));
    __builtin_amdgcn_s_setprio(0);
    if (next_interval()) return;

    // ---- NB intervals with key block j
    {  // dQ needs the K tile as the transposed operand (columns 32 db.., key rows 16 c..): laid out so once instead of NB times
      bf16x8 kt[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) kt[m] = lds_transposed((tr_at + ktile + 16 * (m & 1) * D * 2) ^ (64 * (m >> 1)));
      wave_lds_sync();
#pragma unroll
      for (int m = 0; m < 4; ++m) *reinterpret_cast<bf16x8*>(smem + ktile + m * 1024 + lane_a * 16) = kt[m];
    }
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
      for (int e = 0; e < 16; ++e) dk[db][e] = dv[db][e] = 0.f;
    const int tb = T0 + RB * j, t = tb + c32;
    const bool own_k = key_block_owned(j);
    // query slot s sees this lane's key iff s - smin <= srange (unsigned)
    int smin = circular ? t - R : max(t - R, 0);
    const unsigned srange = (unsigned)max((circular ? t + L : min(t + L, n - 1)) - smin, 0);
    if (!circular && (t < 0 || t >= n)) smin = 1 << 30;
    smin -= 4 * g2;  // accumulators of the wave's upper half start four rows further
    const s16x2 okm1 = {(short)(orig_k - 32768), (short)(orig_k - 32768)};
    for (int ph = NB - 1; ph >= 0; --ph) {
      const int qb = Q0 + RB * i;
      if (ph == kAsks && i + 3 >= 0 && i + 3 < nqb) {  // the query block three intervals ahead is requested
        const int lane = fresh(lane0);
        uint32_t goff[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) goff[v] = query_row(i + 3, 8 * v + (lane >> 3)) + (uint32_t)lane_chunk(lane, v) * 16;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          load_to_lds_16(Qh, goff[v], lds0 + C::OFF_Q + ((i + 3) & 3) * 2 * TILE + v * 1024);
          load_to_lds_16(Gh, goff[v], lds0 + C::OFF_Q + ((i + 3) & 3) * 2 * TILE + TILE + v * 1024);
        }
      }
      if (i >= 0 && i < nqb && ph < nact && (own_k || query_block_owned(i))) {
        const uint32_t qrow = row_at + C::OFF_Q + (i & 3) * 2 * TILE, qtr = tr_at + C::OFF_Q + (i & 3) * 2 * TILE;
        const char* vals = smem + C::OFF_VAL + (i & 3) * C::VALS;
        const int lane_u = fresh(lane0), r_u = lane_u & 31, h_u = lane_u >> 5;
        const uint32_t ds_put = (uint32_t)(r_u * RB + 4 * h_u + (((r_u >> 2) & 3) << 3)) * 2;
        const int dmin = tb - (qb + RB - 1), dmax = tb + RB - 1 - qb;  // range of t - s over the block
        const bool inside = dmin >= -L && dmax <= R && (circular || (tb >= 0 && tb + RB <= n && qb + RB <= n));
        f32x16 s, dp;
        {
          const u32x4 rows = *reinterpret_cast<const u32x4*>(vals + r_u * 16);
          s = mfma_row_values(__builtin_bit_cast(s16x4, (u32x2{rows[0], rows[1]})), ones);   // S / scale starts from -LSE / scale, dP from -D
          dp = mfma_row_values(__builtin_bit_cast(s16x4, (u32x2{rows[2], rows[3]})), ones);
        }
        {
          bf16x8 qa[2], ga[2];
          qa[0] = lds_row(qrow);
          ga[0] = lds_row(qrow + TILE);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int kk = 0; kk < D / 16; ++kk) {
            if (kk + 1 < D / 16) {
              qa[(kk + 1) & 1] = lds_row(qrow ^ (32 * (kk + 1)));
              ga[(kk + 1) & 1] = lds_row((qrow ^ (32 * (kk + 1))) + TILE);
              __builtin_amdgcn_sched_barrier(0);
            }
            s = mfma_bf16(qa[kk & 1], kf[kk], s);     // S = Q K^T
            dp = mfma_bf16(ga[kk & 1], vf[kk], dp);   // dP = dO V^T
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        if (!inside) {
          const int base = qb - smin;
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if ((unsigned)(base + 8 * (e / 4) + (e % 4)) > srange) s[e] = -INFINITY;
        }
        char* const dst = smem + C::OFF_DS + (i & 1) * (NB * DS_TILE) + ph * DS_TILE;
        // 16 query rows: P and dS, two accumulators at a time
        auto weights = [&](const int half, u32x4& wp, u32x4& wd) {
          u32x4 iw = {0, 0, 0, 0};
          if (CAUSAL == CAUSAL_I16) iw = *reinterpret_cast<const u32x4*>(vals + RB * 16 + (16 * h_u + 8 * half) * 2);
#pragma unroll
          for (int mq = 2 * half; mq < 2 * half + 2; ++mq) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const int e0 = 4 * mq + 2 * h, e1 = e0 + 1, w = 2 * (mq & 1) + h;
              const float pe0 = __builtin_amdgcn_exp2f(s[e0] * cs);
              const float pe1 = __builtin_amdgcn_exp2f(s[e1] * cs);
              uint32_t vis = 0xffffffffu;
              if (CAUSAL == CAUSAL_I16)  // visible iff the query's position >= the key's: (orig_k - 1) - pq < 0
                vis = __builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(okm1, __builtin_bit_cast(s16x2, (uint32_t)iw[w])) >> (short)15);
              wp[w] = pack_bf16(pe0, pe1) & vis;
              wd[w] = pack_bf16(pe0 * dp[e0], pe1 * dp[e1]) & vis;
            }
            const u32x2 pair = {wd[2 * (mq & 1)], wd[2 * (mq & 1) + 1]};
            *reinterpret_cast<u32x2*>(dst + (ds_put ^ (mq << 4))) = pair;
          }
        };
        auto operands = [&](const int half, bf16x8* a) {  // dO^T, Q^T of those rows: columns 0..31, 32..63
#pragma unroll
          for (int db = 0; db < 2; ++db) {
            a[2 * db] = lds_transposed(((qtr + 16 * half * D * 2) ^ (64 * db)) + TILE);
            a[2 * db + 1] = lds_transposed((qtr + 16 * half * D * 2) ^ (64 * db));
          }
        };
        auto products = [&](const bf16x8* a, const u32x4& wp, const u32x4& wd) {
          const bf16x8 pf = __builtin_bit_cast(bf16x8, wp), df = __builtin_bit_cast(bf16x8, wd);
#pragma unroll
          for (int db = 0; db < 2; ++db) {
            dv[db] = mfma_bf16(a[2 * db], pf, dv[db]);
            dk[db] = mfma_bf16(a[2 * db + 1], df, dk[db]);
          }
        };
        // the operands of the first half are on their way during the second half's exponentials
        u32x4 wp0, wd0, wp1, wd1;
        bf16x8 a0[4], a1[4];
        weights(0, wp0, wd0);
        operands(0, a0);
        __builtin_amdgcn_sched_barrier(0);
        weights(1, wp1, wd1);
        __builtin_amdgcn_sched_barrier(0);
        products(a0, wp0, wd0);
        operands(1, a1);
        __builtin_amdgcn_sched_barrier(0);
        products(a1, wp1, wd1);
      }
      if (ph == kAsks - 1) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // requested in the interval before
      if (next_interval()) return;
    }
  }
}

// Strips of a call: as many per head as fill k rounds of the card's CUs (one workgroup per CU), with the k for which the rounds'
// intervals are fewest.
Strips plan(const Pass& p, int nb) {
  const long heads = (long)p.B * p.Hq;
  const int most = (p.n + RB - 1) / RB;
  Strips best = {};
  long least = -1;
  for (int k = 1; k <= 8; ++k) {
    int m = (int)(kCUs * (long)k / heads);
    m = m < 1 ? 1 : (m > most ? most : m);
    if ((long)m * kMostSlots < p.n) m = (p.n + kMostSlots - 1) / kMostSlots;
    const int slots = ((p.n + m - 1) / m + RB - 1) / RB * RB;
    m = (p.n + slots - 1) / slots;
    const long rounds = (heads * m + kCUs - 1) / kCUs;
    const long cost = rounds * ((slots + p.win.L + p.win.R) / RB + nb + 4);
    if (least < 0 || cost < least) {
      least = cost;
      best = {m, slots};
    }
  }
  return best;
}

int key_blocks(const Pass& p) { return p.win.L + p.win.R <= 128 ? 5 : 9; }
// plain causal SWA: the window already leaves out every later key
bool masks_positions(const Pass& p) { return p.causal && !(!p.perm && !p.win.circular && p.win.R == 0); }

// Intervals with pairs of the strip that has most of them (the kernel's block grids).
int intervals(const Pass& p, const Strips& s) {
  const int L = p.win.L, R = p.win.R;
  int most = 0;
  for (const int strip : {0, s.per_head / 2, s.per_head - 1}) {
    const int k0 = strip * s.slots, k1 = std::min(k0 + s.slots, p.n);
    const int q_lo = p.win.circular ? k0 - R : std::max(k0 - R, 0), q_hi = p.win.circular ? k1 - 1 + L : std::min(k1 - 1 + L, p.n - 1);
    const int Q0 = k0 - (k0 - q_lo + RB - 1) / RB * RB;
    most = std::max({most, (q_hi - Q0) / RB + 1, (k1 - 1 - Q0 + L) / RB + 1});
  }
  return most;
}

// Microseconds of a call with either form, as far as the choice needs them.  Strips come in rounds of 256 workgroups, each with the intervals of
// its longest strip, and are slowed down by HBM where there are many rows.  The two kernels' workgroups of 128 slots go up in steps: a second one to a
// CU costs little, a third is a second round of the dK/dV kernel.  The constants are those for which fewest of 4200 calls measured with both forms take
// the slower one (1 to 1200 heads, 40 to 65535 slots, w = 1 to 257, circular and one-sided, with rotations and without; a third of them at the
// heads and lengths of training steps, a quarter at edges of rounds): both estimates are within 7 % of their times (standard deviation), 18 calls take
// a form that is more than a tenth slower than the other, against 94 with strips for all, and the calls as a whole 0.2 % longer than with the faster form each.
// Two kernels / strips (us), no rotations, circular, by heads x slots, w = 33 | 129 | 257:
//   1 x 300     14.5 / 9.1  | 18.1 / 11.6 | 23.4 / 18.3      64 x 512    15.9 / 13.0 | 19.5 / 16.8 | 24.5 / 25.2
//   12 x 16384  65.9 / 39.9 | 79.1 / 46.8 | 94.1 / 63.8      64 x 8192   161 / 115   | 196 / 122   | 238 / 146
//   256 x 256   21.8 / 18.6 | 26.9 / 23.0 | 34.0 / 32.5      257 x 256   29.1 / 34.5 | 36.9 / 42.9 | 46.4 / 61.0
//   320 x 512   58.8 / 54.1 | 68.8 / 64.7 | 83.0 / 89.2      480 x 300   54.2 / 38.6 | 65.9 / 50.3 | 85.1 / 69.2
//   1024 x 256  83.5 / 69.6 | 98.5 / 87.3 | 119 / 124        2048 x 256  159 / 159   | 192 / 182   | 236 / 256
// One-sided without a permutation, w = 257: 256 x 256 24.8 / 28.6, 257 x 256 33.6 / 53.7, 192 x 512 48.5 / 40.8; rotations, w = 257: 64 x 512
// 28.7 / 30.9, 480 x 300 87 / 76.
bool strips_are_faster(const Pass& p) {
  const Strips s = plan(p, key_blocks(p));
  const long heads = (long)p.B * p.Hq;
  const int reach = p.win.L + p.win.R, turned = p.rope_table ? 1 : 0;
  // what neighbouring slots see beyond themselves, on average over a sequence with ends
  double seen = reach;
  if (!p.win.circular)
    for (const double side : {(double)p.win.L, (double)p.win.R}) seen -= side * (side + 128) / (2. * p.n);
  if (seen < 0) seen = 0;

  const double rounds = (double)((heads * s.per_head + kCUs - 1) / kCUs);
  const double walk = rounds * (6.8 + intervals(p, s) * (1.0 + 0.062 * seen / RB + 0.48 * turned)) + 1.5 * turned;
  const double rows = (0.13 + 0.08 * turned) * 1e-3 * (double)heads * p.n;
  const double strips = std::sqrt(walk * walk + rows * rows);

  const long tiles = (p.n + 127) / 128;
  const double per_cu = (double)heads * tiles / kCUs, filled = p.n / (128. * tiles);
  const double one = 21 + (masks_positions(p) ? 7.2 : 6.0) * seen / 128 - (reach ? 0 : 2.4);
  const double steps = per_cu <= 1 ? 1 : (per_cu <= 2 ? 1.05 + 0.09 * per_cu : 0.71 + 0.41 * per_cu);
  const double two = one * steps * (0.73 + 0.27 * filled) - 5.2 + turned * (1.8 + 2.6 * filled * per_cu);
  return strips <= two;
}

template <int NB, int CAUSAL>
hipError_t launch_t(const Pass& p, hipStream_t st) {
  const Strips s = plan(p, NB);
  const long total = (long)p.B * p.Hq * s.per_head;
  const long blocks = xcd_grid_blocks(total);
  if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks), block((Cfg<NB, ROWS_PLAIN>::NT));
  if (p.rope_table) hipLaunchKernelGGL((bwd_strip_bf16_kernel<NB, CAUSAL, ROWS_TURN>), grid, block, 0, st, p, s, total);
  else if (p.accumulate) hipLaunchKernelGGL((bwd_strip_bf16_kernel<NB, CAUSAL, ROWS_ADD>), grid, block, 0, st, p, s, total);
  else hipLaunchKernelGGL((bwd_strip_bf16_kernel<NB, CAUSAL, ROWS_PLAIN>), grid, block, 0, st, p, s, total);
  return hipGetLastError();
}
template <int NB>
hipError_t launch_t(const Pass& p, bool causal, hipStream_t st) {
  return causal ? launch_t<NB, CAUSAL_I16>(p, st) : launch_t<NB, CAUSAL_NONE>(p, st);
}

}  // namespace

// Where it can: the registers of a wave hold d = 64, its W waves a window of 257 slots, LDS 16-bit positions; the two-kernel form
// reads K, V and dO once more after dQ is written, so outputs laid over inputs (dK over K, dV over V) stay with it.
// Where it is the faster one: by strips_are_faster(), and not in calls of more than one round of workgroups over fewer than 256 slots, where a
// workgroup's first and last intervals are most of it (480 heads, 128 slots, w = 64: 25 us in two kernels, 28 us here).
bool bwd_strip_serves(const Pass& p) {
  if (p.d != D || p.g != 1 || p.win.L + p.win.R > kMostReach || p.n > 65535 || !(p.scale > 1e-20f)) return false;
  if ((long)p.B * p.Hq > kCUs && p.n < 256) return false;
  const uintptr_t bytes = (uintptr_t)p.B * p.Hq * p.n * D * 2;
  const void* ins[] = {p.Q, p.K, p.V, p.dO, p.O_rows};
  const void* outs[] = {p.dQ, p.dK, p.dV};
  for (const void* o : outs)
    for (const void* in : ins) {
      const uintptr_t x = reinterpret_cast<uintptr_t>(o), y = reinterpret_cast<uintptr_t>(in);
      if (in && x < y + bytes && y < x + bytes) return false;
    }
  return strips_are_faster(p);
}

hipError_t launch_bwd_strip_bf16(const Pass& p, hipStream_t st) {
  if (!bwd_strip_serves(p)) return hipErrorNotSupported;
  if (p.n < 1 || p.B < 1 || p.Hq < 1 || p.Hq != p.Hkv || (long)p.n * D * 2 >= (1L << 31)) return hipErrorInvalidValue;
  if (p.win.L < 0 || p.win.R < 0 || p.win.L >= p.n || p.win.R >= p.n) return hipErrorInvalidValue;
  if (p.win.circular && p.win.L + p.win.R + 1 > p.n) return hipErrorInvalidValue;
  if (!p.dO || !p.lse_in || !p.dQ || !p.dK || !p.dV || !(p.O_rows || p.Dsum)) return hipErrorInvalidValue;
  if ((p.rope_dk && !p.rope_table) || (p.rope_table && p.accumulate)) return hipErrorInvalidValue;
  return key_blocks(p) == 5 ? launch_t<5>(p, masks_positions(p), st) : launch_t<9>(p, masks_positions(p), st);
}

}  // namespace sa
