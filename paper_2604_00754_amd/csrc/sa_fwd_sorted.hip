// bf16 forward of Stochastic Attention for grouped query heads that share a permutation, d = 128, causal on original
// positions: the kernel of sa_fwd_mfma.hip without the work its causal test throws away.
//
// In permuted order half of the pairs inside a window are later keys, spread evenly over it.  Here a group of 128 slots is
// cut by ORIGINAL position into four quarters of 32 queries, one workgroup each (4 wavefronts = the same 32 queries of four
// query heads of a KV group), and the keys of the group's band (128 + w - 1 slots) that come after all 32 queries of the
// quarter are left out: quarter r walks (r + 1) / 4 of the band, 5/8 on average, i.e. 400 keys at w = 512 and 720 at
// w = 1024, where 32 neighbouring slots need 544 and 1056.
// What a workgroup walks is a list in LDS of the keys' original positions, made in its prologue: first the keys that no test
// applies to (before all 32 queries, inside the windows of the whole group), then those for the causal test alone, then
// those for both tests, so that tests are compiled per section of the list.  Because the queries are sorted the causal test
// compares a key's rank among the 32 of them (16 bits at any n) with the query's place.
// Everything else is as there: S^T = K Q^T, softmax with the reference at zero first and in the online form if a row sum leaves
// the range of fp32, O^T += V^T P^T, K/V rows by direct global-to-LDS loads one 32-key tile ahead, rows scattered to
// their original positions.
#include <type_traits>

#include "sa_common.h"
#include "sa_mfma.h"

namespace sa {
namespace {

constexpr int D = 128;
constexpr int NT = 256;
constexpr int BN = 32;          // keys per tile
constexpr int GROUP = 128;      // slots of a group
// A tile operand lies in LDS as it is loaded: 4 rows (1024 bytes) per wave-wide instruction, 16 bytes of padding after each,
// the 16-byte chunks of a row permuted by an XOR with 4 * (row % 4).  Rows r and r + 4 are then shifted by one chunk and rows of
// one instruction by four, which makes both read patterns conflict-free (16 rows x the same chunk; 4 rows x 4
// neighbouring chunks), and the XOR touches only the bits of the chunk number above the two lowest: four lane addresses
// per operand, the rest are immediate offsets.
constexpr int QUAD_BYTES = 4 * D * 2 + 16;
constexpr int TILE_BYTES = BN / 4 * QUAD_BYTES;
constexpr int BUF_BYTES = 2 * TILE_BYTES;              // K | V
constexpr int STR = D + 8;                             // bf16 per staged Q / O row
constexpr int QSTAGE_BYTES = 4 * 16 * STR * 2;         // 16 query rows of each wave at a time
constexpr int TABLE_STR = D + 4;                       // floats per staged row of the RoPE table
static_assert(32 * TABLE_STR * 4 <= QSTAGE_BYTES, "the table rows of 32 queries fit where the query rows were");
constexpr int OSTAGE_BYTES = 4 * 32 * STR * 2;

constexpr int AREA_BYTES = BUF_BYTES + (BUF_BYTES > QSTAGE_BYTES ? BUF_BYTES : QSTAGE_BYTES);  // two buffers; query rows pass through the second
constexpr int LIST_OFF = AREA_BYTES > OSTAGE_BYTES ? AREA_BYTES : OSTAGE_BYTES;  // positions (4 bytes) | ranks (2) | slots in the band (2)
constexpr int CAP = 2048;                              // band of a group that a list can hold
constexpr int OWN_OFF = LIST_OFF + CAP * 8;            // positions | slots of the 32 queries | section counts [4][4]
constexpr int LDS_BYTES = OWN_OFF + 32 * 4 + 32 * 4 + 16 * 4;
static_assert(3 * LDS_BYTES <= 160 * 1024 && LIST_OFF % 16 == 0, "three workgroups per CU, 16-byte accesses");

typedef short s16x2 __attribute__((ext_vector_type(2)));

template <bool ROPE>
__global__ __launch_bounds__(NT, 3) void fwd_sorted_bf16_kernel(const Pass p, const unsigned num_quarters, const unsigned total_work,
                                                                const int per) {
  __shared__ __attribute__((aligned(16))) char smem[LDS_BYTES];
  // Work list: the quarters of a slot group, then the next group (neighbours share K/V rows), then the next `per` head sets
  // (four query heads of a KV group each), which one workgroup takes one after another: the list is the same for all of them.
  // Workgroups are dealt to the four shader engines of an XCD in turn, so the quarters of a group start with another one in
  // every group: in one fixed order one engine gets all the long lists (32 768 slots, w = 512: 391 -> 344 us when this was
  // measured; now 291 us with 2.4 of three waves a SIMD resident on average)
  const unsigned chunk_work = (total_work + NXCD - 1) / NXCD, local = blockIdx.x / NXCD;
  const unsigned work = (blockIdx.x % NXCD) * chunk_work + local;
  if (local >= chunk_work || work >= total_work) return;
  const int sets = p.g >> 2, all_sets = sets * p.Hkv, set_chunks = (all_sets + per - 1) / per;
  const unsigned rest = work / num_quarters, q4 = work - rest * num_quarters;
  const int b = (int)(rest / (unsigned)set_chunks), set0 = ((int)rest - b * set_chunks) * per;
  const int set_end = min(set0 + per, all_sets);
  const int p0 = (int)(q4 >> 2) * GROUP, quarter = (int)((q4 + (q4 >> 2)) & 3);
  const int n = p.n, L = p.win.L, R = p.win.R;
  const int nq = min(GROUP, n - p0);  // queries of the group
  if (32 * quarter >= nq) return;
  const int own = min(32, nq - 32 * quarter);  // of them in this quarter

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g2 = lane >> 5, c32 = lane & 31;
  const int32_t* __restrict__ perm = p.perm + (size_t)perm_slice_index(p.perm_B, p.perm_H, b, 0) * n;
  // head set `set` = query heads hk * g + 4 * (set % sets) + wave of KV head hk = set / sets
  auto q_row0 = [&](int set) -> size_t {
    return ((size_t)b * p.Hq + (set / sets) * p.g + (set % sets) * 4 + wave) * n;
  };

  int* const list_pos = reinterpret_cast<int*>(smem + LIST_OFF);
  short* const list_rank = reinterpret_cast<short*>(smem + LIST_OFF + CAP * 4);
  short* const list_slot = list_rank + CAP;
  int* const own_pos = reinterpret_cast<int*>(smem + OWN_OFF);
  int* const own_slot = own_pos + 32;
  int* const counts = own_slot + 32;

  // ---- band of the group, unwrapped; u = slot - u0 is what a query at slot p0 + s sees iff 0 <= u - s <= L + R
  const int u0 = p0 - L;
  int t_lo = u0, t_hi = p0 + nq - 1 + R;
  if (!p.win.circular) {
    t_lo = max(t_lo, 0);
    t_hi = min(t_hi, n - 1);
  }
  const int band = t_hi - t_lo + 1;

  // ---- queries of the quarter and list of its keys, J slots of the band per thread (straight-line code: the searches of a
  // thread's keys overlap)
  int ntiles = 0, tile_causal = 0, tile_window = 0;  // tiles; first tile with the causal test; first with both
  auto build = [&](auto jc) {
    constexpr int J = decltype(jc)::value;
    const int qp = (tid & 127) < nq ? perm[p0 + (tid & 127)] : 0x7fffffff;
    int kp[J];
#pragma unroll
    for (int j = 0; j < J; ++j) kp[j] = perm[wrap_slot(min(t_lo + j * NT + tid, t_hi), n)];

    // rank of every query of the group: two threads per query with half of the comparisons each.  Positions (below 2^23, the
    // host bounds n * D * 2) are compared together with the slot, so that every place is taken once even where a
    // caller's index tensor names a position twice (undefined rows, but rows of the tensors)
    const int qk = (tid & 127) < nq ? (int)((unsigned)qp * GROUP + (tid & 127)) : 0x7fffffff;
    int* const all_q = reinterpret_cast<int*>(smem);
    int* const half_rank = all_q + GROUP;
    if (tid < GROUP) all_q[tid] = qk;
    if (tid < 32) own_pos[tid] = 0x7fffffff;
    __syncthreads();
    int rank = 0;
    const int4* other = reinterpret_cast<const int4*>(all_q + (tid >> 7) * 64);
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int4 o = other[j];
      rank += (o.x < qk ? 1 : 0) + (o.y < qk ? 1 : 0) + (o.z < qk ? 1 : 0) + (o.w < qk ? 1 : 0);
    }
    half_rank[tid] = rank;
    __syncthreads();
    if (tid < nq) {
      const int mine = half_rank[tid] + half_rank[tid + GROUP] - 32 * quarter;
      if (mine >= 0 && mine < 32) {
        own_pos[mine] = qp;
        own_slot[mine] = tid;
      }
    }
    __syncthreads();

    // A key's section is its class; its place follows from the counts of the sections, of the waves and of the lanes before
    // it, so the order does not depend on timing.
    int r[J], at[J], section[J];
#pragma unroll
    for (int j = 0; j < J; ++j) r[j] = 0;  // queries of the quarter before the key
#pragma unroll
    for (int step = 16; step > 0; step >>= 1)
#pragma unroll
      for (int j = 0; j < J; ++j) r[j] += own_pos[r[j] + step - 1] < kp[j] ? step : 0;
    int mine[3] = {0, 0, 0};
#pragma unroll
    for (int j = 0; j < J; ++j) {
      r[j] += own_pos[r[j]] < kp[j] ? 1 : 0;
      const int e = j * NT + tid, u = e + t_lo - u0;
      const bool inside = (u >= nq - 1) & (u <= L + R);  // inside the windows of all queries of the group
      section[j] = inside ? (r[j] == 0 ? 0 : 1) : 2;
      if ((e >= band) | (r[j] >= own)) section[j] = 3;
      int before = 0;
#pragma unroll
      for (int x = 0; x < 3; ++x) {
        const uint64_t m = __ballot(section[j] == x);
        const int here = mine[x] + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
        before = section[j] == x ? here : before;
        mine[x] += __popcll(m);
      }
      at[j] = before;
    }
    if (lane == 0) {
#pragma unroll
      for (int x = 0; x < 3; ++x) counts[4 * x + wave] = mine[x];
    }
    __syncthreads();
    int total = 0, first[3];
#pragma unroll
    for (int x = 0; x < 3; ++x) {
      const int4 k = *reinterpret_cast<const int4*>(counts + 4 * x);
      first[x] = total + (wave > 0 ? k.x : 0) + (wave > 1 ? k.y : 0) + (wave > 2 ? k.z : 0);
      total = __builtin_amdgcn_readfirstlane(total + k.x + k.y + k.z + k.w);
      if (x == 0) tile_causal = total / BN;
      if (x == 1) tile_window = total / BN;
    }
    ntiles = (total + BN - 1) / BN;
    auto place = [&](int i, int pos, int rk, int u) {
      list_pos[i] = pos;
      // ranks and slots in accumulator order: the 16 keys of a tile that a lane group g2 holds are contiguous
      const int acc = (i & ~31) | ((i & 4) << 2) | ((i >> 1) & 12) | (i & 3);
      list_rank[acc] = (short)rk;
      list_slot[acc] = (short)u;
    };
#pragma unroll
    for (int j = 0; j < J; ++j)
      if (section[j] < 3)
        place(at[j] + (section[j] == 0 ? first[0] : (section[j] == 1 ? first[1] : first[2])), kp[j], r[j], j * NT + tid + t_lo - u0);
    if (tid < ntiles * BN - total) place(total + tid, own_pos[0], 0x7fff, 0);  // rest of the last tile: seen by nobody
  };
  if (band <= 3 * NT) build(std::integral_constant<int, 3>{});
  else if (band <= 5 * NT) build(std::integral_constant<int, 5>{});
  else build(std::integral_constant<int, CAP / NT>{});

  // ---- loads of the query rows (issued per head set, once the list is complete)
  constexpr int NP = 8;  // passes of 4 rows
  const int prow = lane >> 4, chunk16 = lane & 15;
  u32x4 qv[NP];
  // (lane numbers outside the tile loop are taken from copies the optimiser cannot trace: what follows from them is then
  // formed where it is used and not kept in registers across the tile loop)
  auto fresh_lane = [&]() -> int {
    int l = lane;
    asm volatile("" : "+v"(l));
    return l;
  };
  auto load_q = [&](int set) {
    const int ln = fresh_lane(), prow = ln >> 4, chunk16 = ln & 15;
    const char* Qh = reinterpret_cast<const char*>(p.Q) + q_row0(set) * (D * 2);
#pragma unroll
    for (int pass = 0; pass < NP; ++pass) {
      const uint32_t off = (uint32_t)own_pos[min(4 * pass + prow, own - 1)] * (uint32_t)(D * 2) + (uint32_t)chunk16 * 16u;
      qv[pass] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(Qh + off));
    }
  };


  __syncthreads();  // list complete

  // ---- tile loader: instruction j of a wave fills rows 16 j + 4 wave .. + 3
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
  const uint32_t ld_chunk_off = (uint32_t)((chunk16 ^ (prow << 2)) * 16);
  const bf16_t *Kh = nullptr, *Vh = nullptr;
  auto load_tile = [&](const int tile, const int buf) {
    const int r0 = list_pos[tile * BN + 4 * wave + prow], r1 = list_pos[tile * BN + 16 + 4 * wave + prow];
    const uint32_t dst = lds0 + buf * BUF_BYTES + wave * QUAD_BYTES;
    const uint32_t off0 = (uint32_t)r0 * (uint32_t)(D * 2) + ld_chunk_off, off1 = (uint32_t)r1 * (uint32_t)(D * 2) + ld_chunk_off;
    load_to_lds_16(Kh, off0, dst);
    load_to_lds_16(Vh, off0, dst + TILE_BYTES);
    load_to_lds_16(Kh, off1, dst + 4 * QUAD_BYTES);
    load_to_lds_16(Vh, off1, dst + 4 * QUAD_BYTES + TILE_BYTES);
  };

  // ---- lane addresses of the operand reads inside a tile (bytes).  K operand kk: row c32, chunk 2 kk + g2; V^T operand (half
  // hf, columns 32 db ..): row 4 (G / 2) + j / 4 + 8 hf of 16, chunk 4 db + 2 (G % 2) + (j % 4) / 2 for lane 16 G + j
  int koff[4], voff[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    koff[m] = (c32 >> 2) * QUAD_BYTES + (c32 & 3) * 256 + (((m ^ (c32 & 3)) << 2) | g2) * 16;
    const int G = lane >> 4, j = lane & 15, x = j >> 2;
    voff[m] = (G >> 1) * QUAD_BYTES + x * 256 + (((m ^ x) << 2) | (2 * (G & 1)) | ((j & 3) >> 1)) * 16 + (j & 1) * 8;
  }
  const float cs = p.scale * kLog2e;  // exp(scale*x) = exp2(cs*x)
  const float lazy = 8.0f / cs;       // online form: move the reference maximum only for jumps above 2^8

  for (int set = set0; set < set_end; ++set) {
  const size_t kv_row0 = ((size_t)b * p.Hkv + set / sets) * n, head_row0 = q_row0(set);
  Kh = reinterpret_cast<const bf16_t*>(p.K) + kv_row0 * D;
  Vh = reinterpret_cast<const bf16_t*>(p.V) + kv_row0 * D;
  load_q(set);
  // RoPE on the queries' ORIGINAL positions (App. B, App. C; Sec. 4.2): the four heads turn by the same angles.  Each wave
  // brings in a quarter of the table rows, whole rows at a time; they take the place of the staged query rows once those
  // are in registers (read from memory in the operand layout, every lane of every wave is a cache access of its own)
  u32x4 angles[4];
  if constexpr (ROPE) {
    const int ln = fresh_lane();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = own_pos[min(8 * wave + 2 * i + (ln >> 5), own - 1)];
      angles[i] = *reinterpret_cast<const table_u32x4*>(p.rope_table + (size_t)row * D + 4 * (ln & 31));
    }
  }
  load_tile(0, 0);

  // ---- this wave's query rows to B operands, 16 at a time through its part of the second buffer
  bf16x8 qf[D / 16];
  {
    const int ln = fresh_lane(), prow = ln >> 4, chunk16 = ln & 15, c32 = ln & 31, g2 = ln >> 5;
    bf16_t* Qs = reinterpret_cast<bf16_t*>(smem + BUF_BYTES) + wave * 16 * STR;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
      for (int pass = 0; pass < NP / 2; ++pass) *reinterpret_cast<u32x4*>(Qs + (4 * pass + prow) * STR + chunk16 * 8) = qv[4 * half + pass];
      wave_lds_sync();
      if ((c32 >> 4) == half) {
#pragma unroll
        for (int kk = 0; kk < D / 16; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(Qs + (c32 & 15) * STR + 16 * kk + 8 * g2);
      }
      wave_lds_sync();
    }
  }
  if constexpr (ROPE) {
    const int ln = fresh_lane();
    float* const table = reinterpret_cast<float*>(smem + BUF_BYTES);
    __syncthreads();  // every wave has its query rows
#pragma unroll
    for (int i = 0; i < 4; ++i) *reinterpret_cast<u32x4*>(table + (8 * wave + 2 * i + (ln >> 5)) * TABLE_STR + 4 * (ln & 31)) = angles[i];
    __syncthreads();
    rope_row_fragments<D, true>(qf, reinterpret_cast<const float2*>(table + (ln & 31) * TABLE_STR), ln >> 5, p.rope_interleaved);
  }

  float m_ref = 0.f, l_run = 0.f;
  f32x16 oacc[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) oacc[db][i] = 0.f;

  // one tile; the buffer, the form of the softmax and the tests (0 none, 1 causal, 2 causal and window) are compile-time
  // constants
  auto do_tile = [&](const int tile, auto bufc, auto fastc, auto testsc) {
    constexpr int buf = decltype(bufc)::value, TESTS = decltype(testsc)::value;
    constexpr bool FAST = decltype(fastc)::value;
    wait_all_loads();  // this wave's share of the tile has landed; after the barrier the whole tile is visible and everyone
    __syncthreads();   // is done with the other buffer
    if (tile + 1 < ntiles) load_tile(tile + 1, buf ^ 1);
    const char* Ks = smem + buf * BUF_BYTES;
    const char* Vs = Ks + TILE_BYTES;

    // ---- S^T = K Q^T, operands requested four at a time
    f32x16 sacc;
#pragma unroll
    for (int i = 0; i < 16; ++i) sacc[i] = 0.f;
#pragma unroll
    for (int k0 = 0; k0 < D / 16; k0 += 4) {
      bf16x8 ka[4];
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) ka[kk] = *reinterpret_cast<const bf16x8*>(Ks + koff[(k0 + kk) >> 1] + ((k0 + kk) & 1) * 32);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) sacc = mfma_bf16(ka[kk], qf[k0 + kk], sacc);
      if (k0 + 4 < D / 16) __builtin_amdgcn_sched_barrier(0);
    }

    // ---- softmax (Eq. 1) on the lane's query column; accumulator i is key 8*(i/4) + 4*g2 + i%4 of the tile
    if (!FAST) {
      const int slot = own_slot[min(c32, own - 1)];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int e = BN * tile + 16 * g2 + i, off = list_slot[e] - slot;
        if (list_rank[e] > c32 || off < 0 || off > L + R) sacc[i] = -INFINITY;
      }
      float mx = sacc[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) mx = fmaxf(mx, sacc[i]);
      mx = max_with_other_half(mx);
      if (__any(mx > m_ref + lazy)) {  // (-inf + lazy = -inf: the first visible key always triggers)
        const float m_new = fmaxf(m_ref, mx);
        const float alpha = (mx > m_ref + lazy) ? __builtin_amdgcn_exp2f((m_ref - m_new) * cs) : 1.f;
        if (mx > m_ref + lazy) m_ref = m_new;
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
          for (int i = 0; i < 16; ++i) oacc[db][i] *= alpha;
      }
    }
    const float mc = FAST ? 0.f : (m_ref == -INFINITY ? 0.f : m_ref) * cs;
    // A key is seen iff its rank is at most the query's place c32 and its slot lies 0 .. L + R after the query's: three
    // differences that are negative then.  Pair e of the lane = accumulators 2e, 2e+1 = one dword of the list.
    const bf16x2 ones = {(bf16_t)1.f, (bf16_t)1.f};
    u32x4 ra = {0u, 0u, 0u, 0u}, rb = ra, sa = ra, sb = ra;
    s16x2 rank1 = {0, 0}, before = rank1, after = rank1;
    if (FAST && TESTS > 0) {
      int le = lane;  // lane constants of the tests are formed here, from a copy the optimiser cannot hoist, not kept
      asm volatile("" : "+v"(le));
      const int place = le & 31;
      const uint32_t* rk = reinterpret_cast<const uint32_t*>(list_rank + BN * tile) + 8 * (le >> 5);
      ra = *reinterpret_cast<const u32x4*>(rk);
      rb = *reinterpret_cast<const u32x4*>(rk + 4);
      rank1 = s16x2{(short)(place + 1), (short)(place + 1)};
      if (TESTS == 2) {
        const uint32_t* sl = reinterpret_cast<const uint32_t*>(list_slot + BN * tile) + 8 * (le >> 5);
        sa = *reinterpret_cast<const u32x4*>(sl);
        sb = *reinterpret_cast<const u32x4*>(sl + 4);
        const int slot = own_slot[min(place, own - 1)];
        before = s16x2{(short)(slot - 1), (short)(slot - 1)};
        after = s16x2{(short)(slot + L + R + 1), (short)(slot + L + R + 1)};
      }
    }
    u32x4 w[2];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float p0 = __builtin_amdgcn_exp2f(fmaf(sacc[2 * e], cs, -mc));
      const float p1 = __builtin_amdgcn_exp2f(fmaf(sacc[2 * e + 1], cs, -mc));
      uint32_t pp = pack_bf16(p0, p1);
      if (FAST && TESTS > 0) {
        s16x2 seen = __builtin_bit_cast(s16x2, e < 4 ? ra[e & 3] : rb[e & 3]) - rank1;
        if (TESTS == 2) {
          const s16x2 u2 = __builtin_bit_cast(s16x2, e < 4 ? sa[e & 3] : sb[e & 3]);
          seen = seen & (u2 - after) & (before - u2);
        }
        pp &= __builtin_bit_cast(uint32_t, seen >> (short)15);
      }
      l_run = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pp), ones, l_run, false);
      w[e >> 2][e & 3] = pp;
    }

    // ---- O^T += V^T P^T.  Step c contracts tile rows 16 c + {0..3, 8..11} + 4 g2 (+4 for the second half of the lane's
    // values); the transposing read collects them from the row-major V tile.
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int db = 0; db < D / 32; ++db) {
        const char* v = Vs + 4 * c * QUAD_BYTES + voff[db];
        const s16x4 lo = lds_read_tr16(reinterpret_cast<const bf16_t*>(v));
        const s16x4 hi = lds_read_tr16(reinterpret_cast<const bf16_t*>(v + 2 * QUAD_BYTES));
        oacc[db] = mfma_bf16(__builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7)),
                             __builtin_bit_cast(bf16x8, w[c]), oacc[db]);
      }
  };
  // tiles `tile` .. last - 1, the buffer of each a compile-time constant
  auto run_tiles = [&](int tile, const int last, auto fastc, auto testsc) {
    if ((tile & 1) && tile < last) do_tile(tile++, std::integral_constant<int, 1>{}, fastc, testsc);
    for (; tile < last; tile += 2) {
      do_tile(tile, std::integral_constant<int, 0>{}, fastc, testsc);
      if (tile + 1 < last) do_tile(tile + 1, std::integral_constant<int, 1>{}, fastc, testsc);
    }
  };
  run_tiles(0, tile_causal, std::true_type{}, std::integral_constant<int, 0>{});
  run_tiles(tile_causal, tile_window, std::true_type{}, std::integral_constant<int, 1>{});
  run_tiles(tile_window, ntiles, std::true_type{}, std::integral_constant<int, 2>{});
  float l_tot = sum_with_other_half(l_run);
  const bool out_of_range = (fresh_lane() & 31) < own && !(l_tot > 0x1p-80f && l_tot < 0x1p80f);
  if (__syncthreads_or(out_of_range ? 1 : 0)) {
    m_ref = -INFINITY;
    l_run = 0.f;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) oacc[db][i] = 0.f;
    load_tile(0, 0);
    run_tiles(0, ntiles, std::false_type{}, std::integral_constant<int, 0>{});
    l_tot = sum_with_other_half(l_run);
    __syncthreads();  // every wave is through its last tile (on the other path the vote above says so)
  }



  // ---- epilogue: normalise, transpose through LDS, scatter rows to their original positions
  const float inv_l = 1.f / l_tot;
  const int le = fresh_lane();
  if (p.LSE && le < own) p.LSE[head_row0 + own_pos[le]] = m_ref * p.scale + __logf(l_tot);
  bf16_t* Os = reinterpret_cast<bf16_t*>(smem) + wave * 32 * STR;
  {
    bf16_t* mine = Os + (le & 31) * STR + 4 * (le >> 5);
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int mq = 0; mq < 4; ++mq) {
        u32x2 w;
        w[0] = pack_bf16(oacc[db][4 * mq + 0] * inv_l, oacc[db][4 * mq + 1] * inv_l);
        w[1] = pack_bf16(oacc[db][4 * mq + 2] * inv_l, oacc[db][4 * mq + 3] * inv_l);
        *reinterpret_cast<u32x2*>(mine + 32 * db + 8 * mq) = w;
      }
  }
  wave_lds_sync();  // the staging rows are this wave's own
#pragma unroll
  for (int pass = 0; pass < NP; ++pass) {
    const int row = 4 * pass + (le >> 4), col = (le & 15) * 8;
    if (row < own)
      __builtin_nontemporal_store(*reinterpret_cast<const u32x4*>(Os + row * STR + col),
                                  reinterpret_cast<u32x4*>(reinterpret_cast<bf16_t*>(p.Y) + (head_row0 + own_pos[row]) * D + col));
  }
  __syncthreads();  // the staging area is free for the next tiles
  }
}

}  // namespace

static long quarters_of(const Pass& p) { return (long)((p.n + GROUP - 1) / GROUP) * (GROUP / 32); }

// Where the shorter walk pays for the list (a workgroup spends about six tiles' time on its prologue, hidden the better the
// more workgroups a CU goes through).  Items: quarters that hold queries x sets of four heads; window: its slots, at most n.  Time here over time of the
// kernel of sa_fwd_mfma.hip at the line and at the next smaller window measured, 32 query heads on 8 KV heads (4 to 48
// heads in groups of 4 to 12 are within 0.02 of it), without rotation:
//   items                256    512    1024   1536   2048   4096   8192   16 384
//   window at the line   767    639    575    448    383    287    256    192
//   here / there         0.98   0.98   0.99   0.96   0.95   0.97   0.94   0.99
//   smaller window       703    575    511    383    351    255    223    159
//   here / there         1.01   1.00   1.02   1.02   0.98   0.99   0.98   1.02
// With rotation the other kernel reads the table row of every lane by itself and the lines lie lower: 447 slots 1.00 at 256 items and
// 0.94 at 768 (383 slots: 1.01, 0.96), 255 slots 0.94 at 2048, 191 slots 0.90 at 8192.
struct Line {
  long items;
  int window;
};
constexpr Line kLines[] = {{256, 767}, {512, 639}, {1024, 575}, {1536, 448}, {2048, 383}, {4096, 287}, {8192, 256}, {16384, 192}};
constexpr Line kLinesRotated[] = {{256, 448}, {2048, 256}, {8192, 192}};

bool fwd_sorted_serves(const Pass& p) {
  const int reach = p.win.L + p.win.R + 1, w = reach < p.n ? reach : p.n;
  if (!(p.d == D && p.perm && p.perm_H == 1 && p.causal && p.g % 4 == 0 && !p.gate_mode && reach - 1 + GROUP <= CAP)) return false;
  const long items = (long)(p.n / GROUP * (GROUP / 32) + (p.n % GROUP + 31) / 32) * (p.Hq >> 2) * p.B;
  int least = 0x7fffffff;
  auto lower = [&](const Line& l) { least = items >= l.items ? l.window : least; };
  if (p.rope_table) for (const Line& l : kLinesRotated) lower(l);
  else for (const Line& l : kLines) lower(l);
  return w >= least;
}

hipError_t launch_fwd_sorted_bf16(const Pass& p, hipStream_t st) {
  if (!fwd_sorted_serves(p)) return hipErrorInvalidValue;
  const long quarters = quarters_of(p);
  const int all_sets = (p.g >> 2) * p.Hkv;
  // two head sets a workgroup where more than five rounds of workgroups are left then (the list is made half as often:
  // 65 536 slots, w = 512: 548 -> 535 us; fewer rounds end too unevenly, four sets gain nothing more)
  const int per = quarters * ((all_sets + 1) / 2) * p.B >= 4096 ? 2 : 1;
  const long total = quarters * ((all_sets + per - 1) / per) * p.B;
  if (total > 0x7ffffff0L) return hipErrorInvalidValue;
  const dim3 grid((unsigned)xcd_grid_blocks(total)), block(NT);
  const unsigned q = (unsigned)quarters, t = (unsigned)total;
  if (p.rope_table) hipLaunchKernelGGL(fwd_sorted_bf16_kernel<true>, grid, block, 0, st, p, q, t, per);
  else hipLaunchKernelGGL(fwd_sorted_bf16_kernel<false>, grid, block, 0, st, p, q, t, per);
  return hipGetLastError();
}

}  // namespace sa
