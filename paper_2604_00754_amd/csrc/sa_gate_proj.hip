// Gate projections of the dual-path layer on gfx950 matrix cores: Eq. 6 followed by Eq. 5
// (Alg. 2, "Gated Combination").
//
// Per token t = (b, i) the heads are concatenated to y_x[t] in R^{dm}, dm = Hq*d, and
//   logit_x[t,:] = W_x y_x[t],  g_x = sigmoid(logit_x),  Y[t,:] = g_sa * y_sa[t] + g_swa * y_swa[t].
// This is two dm x dm GEMMs over all tokens with an element-wise epilogue that needs the GEMM's own
// input at the output position.  One workgroup (4 waves, 2 x 2) owns 128 tokens x 128 output
// features and runs the two branches one after the other through the same LDS buffers, keeping the
// running sum in registers; a wave owns 64 x 64 as 2 x 2 blocks of v_mfma_f32_32x32x16_bf16, so
// every operand read from LDS feeds two matrix instructions.  Both operands have the contraction
// index contiguous in memory (the token's features inside a head, the weight's input features), so
// the tiles are staged row-major (+16 B row padding) and read with plain 16-byte loads.  The product
// is formed transposed (A operand = weight rows, B operand = token rows): a lane then owns one
// token and each accumulator quad four consecutive output features, i.e. 8 contiguous bytes of
// Y_x and Y.  The forward walks the contraction in rotated order, ending with the 128 input features
// that are the workgroup's own output features: the y_x values the epilogue multiplies the gates with
// are then the token tiles still lying in the two LDS buffers, and are not loaded a second time.
//
// Backward (given dY; g_x saved by the forward):
//   dz_x = dY * y_x * g_x * (1 - g_x)                     element-wise pass, rounded to bf16
//   dy_x = dY * g_x + W_x^T dz_x                          the forward kernel again: tokens = dz_x,
//                                                         weights = W_x^T (transposed once), epilogue = + dY * g_x
//   dW_x = sum_t dz_x[t] y_x[t]^T                         contraction over tokens: both operands are
//                                                         read by the transposing LDS read, a workgroup
//                                                         owns 128 x 128 of dW for a piece of the tokens and
//                                                         adds it with fp32 atomics
#include "sa_common.h"
#include "sa_mfma.h"

namespace sa {
namespace {

constexpr int TM = 128;  // tokens per workgroup
constexpr int TN = 128;  // output features per workgroup
constexpr int TK = 64;   // contraction step
constexpr int GNT = 256;
constexpr int GSTR = TK + 8;                 // bf16 per LDS row
constexpr int TILE_BYTES = TM * GSTR * 2;    // one operand tile (TM == TN)
constexpr int GBUF_BYTES = 2 * TILE_BYTES;   // token tile | weight tile

struct GateProj {
  const void* Y_x[2];  // branch outputs [B,Hq,n,d]; Y_x[1] == nullptr: single path
  const void* W_x[2];  // [dm, dm] row-major, row = output feature
  void* G_x[2];        // optional: gate values sigmoid(logit) [B,Hq,n,d]
  void* Y;             // [B,Hq,n,d]
  // backward-input mode: the branches are independent parts of the work list, Y_out[x] = acc + E1 * E2[x] (E1 = dY,
  // E2[x] = g_x), all [B,Hq,n,d]
  void* Y_out[2];
  const void* E1;
  const void* E2[2];
  int B, Hq, n, d;
};

enum { GP_FORWARD = 0, GP_BWD_INPUT = 1 };

template <int D, int MODE>
__global__ __launch_bounds__(GNT, 2) void gate_proj_fwd_bf16_kernel(const GateProj p, const int num_tt, const int num_ft,
                                                                    const long total_work) {
  __shared__ __attribute__((aligned(16))) char smem[2 * GBUF_BYTES];
  const long work = xcd_work_index(total_work);
  if (work < 0) return;
  // feature tiles vary fastest: consecutive workgroups read the same token tile
  const int ft = (int)(work % num_ft);
  long rest = work / num_ft;
  const int tt = (int)(rest % num_tt);
  rest /= num_tt;
  const int b = (int)(rest % p.B);
  const int only = MODE == GP_BWD_INPUT ? (int)(rest / p.B) : 0;  // backward-input mode: this workgroup's branch

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave & 1, wn = wave >> 1;  // token half, feature half of the workgroup tile
  const int g2 = lane >> 5, c32 = lane & 31;
  const int n = p.n, H = p.Hq, dm = H * D;
  const int i0 = tt * TM, o0 = ft * TN;
  const int nk = dm / TK;

  // loader: 128 rows x 8 chunks of 16 bytes per operand tile, 4 chunks per thread and operand
  const int lrow = tid >> 3, lchunk = tid & 7;  // rows lrow + 32*j
  u32x4 areg[4], wreg[4];
  // Forward: the two contraction steps that cover the workgroup's own 128 output features are taken last, so that
  // the token tiles left in the two buffers are the Y_x values Eq. 5 needs at the output positions (the epilogue
  // reads them from LDS instead of from memory).  The other steps keep their order: the workgroups that share a
  // token tile (the feature tiles of one token tile run side by side) then walk it nearly in step and find each
  // other's rows in L2 (fully rotated orders kept the whole tile of every group alive there: 4 x the fetches).
  const int own = MODE == GP_FORWARD ? o0 / TK : nk;  // (dm is a multiple of TN = 2 TK: nk >= 2)
  auto load_tiles = [&](const bf16_t* Yx, const bf16_t* Wx, int step) {
    const int kk = MODE != GP_FORWARD ? step : (step < nk - 2 ? (step < own ? step : step + 2) : own + step - (nk - 2));
    const int k0 = kk * TK, h = k0 / D, e0 = k0 % D;
    const bf16_t* abase = Yx + ((size_t)b * H + h) * n * (size_t)D + e0 + lchunk * 8;
    const bf16_t* wbase = Wx + (size_t)k0 + lchunk * 8;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = lrow + 32 * j;
      areg[j] = *reinterpret_cast<const u32x4*>(abase + (size_t)min(i0 + row, n - 1) * D);
      wreg[j] = *reinterpret_cast<const u32x4*>(wbase + (size_t)(o0 + row) * dm);
    }
  };
  auto store_tiles = [&](int buf) {
    bf16_t* As = reinterpret_cast<bf16_t*>(smem + buf * GBUF_BYTES);
    bf16_t* Ws = reinterpret_cast<bf16_t*>(smem + buf * GBUF_BYTES + TILE_BYTES);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = lrow + 32 * j;
      *reinterpret_cast<u32x4*>(As + row * GSTR + lchunk * 8) = areg[j];
      *reinterpret_cast<u32x4*>(Ws + row * GSTR + lchunk * 8) = wreg[j];
    }
  };

  // running sum of Eq. 5: (fi, ti) = 32-feature block, 32-token block of the wave; accumulator
  // 4q + x of lane (g2, c32) is token 64wm + 32ti + c32, feature 64wn + 32fi + 8q + 4g2 + x
  f32x16 out[2][2];
#pragma unroll
  for (int fi = 0; fi < 2; ++fi)
#pragma unroll
    for (int ti = 0; ti < 2; ++ti)
#pragma unroll
      for (int i = 0; i < 16; ++i) out[fi][ti][i] = 0.f;

  // Output rows leave through a wave-private LDS area: the accumulator layout gives a lane 8-byte pieces of
  // 32 different rows, the staged copy lets 8 lanes write one full 128-byte piece of a row (non-temporal:
  // the outputs are written once).  Staging follows a workgroup barrier: the area lies on the two weight
  // tiles (waves 0, 1 on the first buffer's, waves 2, 3 on the second's), so the token tiles stay readable.
  constexpr int OSTR = 64 + 8;  // bf16 per staged row (64 features of one token + 16 B pad)
  static_assert(2 * 64 * OSTR * 2 == TILE_BYTES, "two waves' staging rows fill one weight tile");
  bf16_t* ostage = reinterpret_cast<bf16_t*>(smem + (wave >> 1) * GBUF_BYTES + TILE_BYTES) + (wave & 1) * 64 * OSTR;
  auto stage_put = [&](int fi, int ti, int q, u32x2 w) {
    *reinterpret_cast<u32x2*>(ostage + (32 * ti + c32) * OSTR + 32 * fi + 8 * q + 4 * g2) = w;
  };
  auto stage_flush = [&](bf16_t* dst) {
    wave_lds_sync();
    const int o = o0 + 64 * wn;  // first of the wave's 64 features: inside one head
    const size_t col = (size_t)(o % D) + (lane & 7) * 8;
#pragma unroll
    for (int pass = 0; pass < 8; ++pass) {
      const int tl = pass * 8 + (lane >> 3);
      const int token = i0 + 64 * wm + tl;
      if (token < n) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(ostage + tl * OSTR + (lane & 7) * 8);
        __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(dst + (((size_t)b * H + o / D) * n + token) * D + col));
      }
    }
    wave_lds_sync();
  };

  // The other way round: the wave's 64 tokens x 64 features of a tensor come in as whole 128-byte pieces of rows
  // and are handed out in the accumulator layout (rows past n: the last row's values, never stored).
  auto stage_fetch_rows = [&](const bf16_t* src, u32x4* v) {
    const int o = o0 + 64 * wn;
    const size_t col = (size_t)(o % D) + (lane & 7) * 8;
#pragma unroll
    for (int pass = 0; pass < 8; ++pass) {
      const int token = min(i0 + 64 * wm + pass * 8 + (lane >> 3), n - 1);
      v[pass] = *reinterpret_cast<const u32x4*>(src + (((size_t)b * H + o / D) * n + token) * D + col);
    }
  };
  auto stage_fetch_put = [&](const u32x4* v) {
#pragma unroll
    for (int pass = 0; pass < 8; ++pass)
      *reinterpret_cast<u32x4*>(ostage + (pass * 8 + (lane >> 3)) * OSTR + (lane & 7) * 8) = v[pass];
    wave_lds_sync();
  };
  auto stage_get = [&](int fi, int ti, int q) -> u32x2 {
    return *reinterpret_cast<const u32x2*>(ostage + (32 * ti + c32) * OSTR + 32 * fi + 8 * q + 4 * g2);
  };

  const int first = MODE == GP_BWD_INPUT ? only : 0;
  const int last = MODE == GP_BWD_INPUT ? only : (p.Y_x[1] ? 1 : 0);
  for (int x = first; x <= last; ++x) {
    const bf16_t* Yx = reinterpret_cast<const bf16_t*>(p.Y_x[x]);
    const bf16_t* Wx = reinterpret_cast<const bf16_t*>(p.W_x[x]);
    f32x16 acc[2][2];
#pragma unroll
    for (int fi = 0; fi < 2; ++fi)
#pragma unroll
      for (int ti = 0; ti < 2; ++ti)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[fi][ti][i] = 0.f;

    __syncthreads();  // the previous branch is done with both buffers
    load_tiles(Yx, Wx, 0);
    store_tiles(0);
    if (nk > 1) load_tiles(Yx, Wx, 1);
    for (int kk = 0; kk < nk; ++kk) {
      const int buf = kk & 1;
      __syncthreads();  // buffer `buf` is complete; everyone is done with the other one
      if (kk + 1 < nk) {
        store_tiles(buf ^ 1);
        if (kk + 2 < nk) load_tiles(Yx, Wx, kk + 2);
      }
      const bf16_t* As = reinterpret_cast<const bf16_t*>(smem + buf * GBUF_BYTES) + (64 * wm + c32) * GSTR + 8 * g2;
      const bf16_t* Ws = reinterpret_cast<const bf16_t*>(smem + buf * GBUF_BYTES + TILE_BYTES) + (64 * wn + c32) * GSTR + 8 * g2;
#pragma unroll
      for (int ks = 0; ks < TK / 16; ++ks) {
        bf16x8 fa[2], fb[2];
#pragma unroll
        for (int fi = 0; fi < 2; ++fi) fa[fi] = *reinterpret_cast<const bf16x8*>(Ws + 32 * fi * GSTR + 16 * ks);
#pragma unroll
        for (int ti = 0; ti < 2; ++ti) fb[ti] = *reinterpret_cast<const bf16x8*>(As + 32 * ti * GSTR + 16 * ks);
#pragma unroll
        for (int fi = 0; fi < 2; ++fi)
#pragma unroll
          for (int ti = 0; ti < 2; ++ti) acc[fi][ti] = mfma_bf16(fa[fi], fb[ti], acc[fi][ti]);
      }
    }

    // Eq. 6 / Eq. 5 for this branch: out += sigmoid(logit) * Y_x at the same (token, feature)
    // (backward-input mode: out = product + dY * g_x)
    bf16_t* Gx = reinterpret_cast<bf16_t*>(p.G_x[x]);
    const bf16_t* E1 = reinterpret_cast<const bf16_t*>(p.E1);
    const bf16_t* E2 = reinterpret_cast<const bf16_t*>(p.E2[x]);
    // step nk-2 left features o0 .. o0+63 of the token tile in its buffer, step nk-1 the next 64: this wave's 64
    // features are in the buffer of step nk-2+wn (the output staging area below lies on the weight tiles only)
    const bf16_t* Ay = reinterpret_cast<const bf16_t*>(smem + ((nk - 2 + wn) & 1) * GBUF_BYTES) + (64 * wm + c32) * GSTR + 4 * g2;
    if (MODE == GP_FORWARD && Gx) __syncthreads();  // every wave has read its last operands: the area is free
    u32x2 e1[2][2][4];
    if (MODE == GP_BWD_INPUT) {
      // dY and g_x at the output positions: whole rows through the staging area (the accumulator layout would
      // ask memory for 8-byte pieces of 32 rows per instruction)
      u32x4 r1[8], r2[8];
      stage_fetch_rows(E1, r1);
      stage_fetch_rows(E2, r2);
      __syncthreads();  // every wave has read its last operands: the area is free
      stage_fetch_put(r1);
#pragma unroll
      for (int ti = 0; ti < 2; ++ti)
#pragma unroll
        for (int fi = 0; fi < 2; ++fi)
#pragma unroll
          for (int q = 0; q < 4; ++q) e1[ti][fi][q] = stage_get(fi, ti, q);
      wave_lds_sync();
      stage_fetch_put(r2);
    }
#pragma unroll
    for (int ti = 0; ti < 2; ++ti) {
#pragma unroll
      for (int fi = 0; fi < 2; ++fi)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (MODE == GP_FORWARD) {
            const u32x2 y = *reinterpret_cast<const u32x2*>(Ay + 32 * ti * GSTR + 32 * fi + 8 * q);
            const float yv[4] = {bf16lo(y[0]), bf16hi(y[0]), bf16lo(y[1]), bf16hi(y[1])};
            float gv[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              gv[e] = sigmoidf_rcp(acc[fi][ti][4 * q + e]);
              out[fi][ti][4 * q + e] = fmaf(gv[e], yv[e], out[fi][ti][4 * q + e]);
            }
            if (Gx) {
              u32x2 w;
              w[0] = pack_bf16(gv[0], gv[1]);
              w[1] = pack_bf16(gv[2], gv[3]);
              stage_put(fi, ti, q, w);
            }
          } else {
            const u32x2 a = e1[ti][fi][q], c = stage_get(fi, ti, q);
            out[fi][ti][4 * q + 0] = fmaf(bf16lo(a[0]), bf16lo(c[0]), acc[fi][ti][4 * q + 0]);
            out[fi][ti][4 * q + 1] = fmaf(bf16hi(a[0]), bf16hi(c[0]), acc[fi][ti][4 * q + 1]);
            out[fi][ti][4 * q + 2] = fmaf(bf16lo(a[1]), bf16lo(c[1]), acc[fi][ti][4 * q + 2]);
            out[fi][ti][4 * q + 3] = fmaf(bf16hi(a[1]), bf16hi(c[1]), acc[fi][ti][4 * q + 3]);
          }
        }
    }
    if (MODE == GP_FORWARD && Gx) stage_flush(Gx);
  }

  __syncthreads();  // every wave has read its last operands (or flushed its last gate rows): the area is free
#pragma unroll
  for (int ti = 0; ti < 2; ++ti)
#pragma unroll
    for (int fi = 0; fi < 2; ++fi)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        u32x2 w;
        w[0] = pack_bf16(out[fi][ti][4 * q + 0], out[fi][ti][4 * q + 1]);
        w[1] = pack_bf16(out[fi][ti][4 * q + 2], out[fi][ti][4 * q + 3]);
        stage_put(fi, ti, q, w);
      }
  stage_flush(reinterpret_cast<bf16_t*>(MODE == GP_BWD_INPUT ? p.Y_out[only] : p.Y));
}

// The same two products in wide tiles: a wave owns 128 tokens x 64 output features as 4 x 2 blocks.  Per 16 contraction indices it
// reads 6 KB of operands from LDS for eight matrix instructions (64 x 64: 4 KB for four), and a workgroup brings in half to three
// quarters of the bytes per product; both are nearly as much time as the matrix work at 64 x 64.  Eight waves, one workgroup per
// CU; tiles arrive by direct global-to-LDS loads, one barrier a step.
//   BOTH (forward of both branches): 256 tokens x 128 features of either branch, four waves each, steps of 32 contraction
//            indices, three buffers.  Neither branch's term of Eq. 5 waits in registers for the other: at the end each wave gives
//            its half of the terms to the wave of the other branch with the same outputs (fp32, through LDS) and writes the other
//            half of Y.
//   else     256 x 256, steps of 64 (whole lines), two buffers: input gradients (the branches are independent parts of the work
//            list) and the forward of a single path.
// Measured at B4, n = 8192, 16 heads of 64, both forms in turn in one process (us): forward of both branches 180 -> 171 (124 without the
// loads: half lines, 64 bytes of a row a step, cost 12 of the rest; two buffers of whole lines do not fit beside either branch's tiles), single
// path 94 -> 78 = 0.88 PFLOP/s, backward of both 460 -> 427 (now 403 with the rest of the call).  bench.py, which times each call by itself,
// reads 189 to 192 for the forward (0.72 PFLOP/s) and 413 to 437 for the backward.  A step's loads go out with the first two operand groups, not all
// behind the barrier: 173 -> 170, 80 -> 78.  Wave priorities around the products: no change.
constexpr int XTM = 256;
constexpr int XNT = 512;
constexpr int XSTR = 64 + 8;                     // bf16 per staged row
constexpr int XAREA = 64 * XSTR * 2;             // staged 64 tokens x 64 features
static_assert(2 * XAREA >= 64 * 64 * 4, "a wave's two staging areas hold 64 x 64 in fp32");

template <bool BOTH>
struct Wide {
  static constexpr int FEATS = BOTH ? 128 : 256;              // output features of a workgroup
  static constexpr int K = BOTH ? 32 : 64;                    // contraction step
  static constexpr int STAGES = BOTH ? 3 : 2;
  static constexpr int ROW = K * 2;                           // bytes of a tile row, 16-byte chunks XORed by swizzle()
  static constexpr int PART = (XTM + FEATS) * ROW;            // a branch's share of a stage: tokens | weights
  static constexpr int STAGE = (BOTH ? 2 : 1) * PART;
  static constexpr int LDS = STAGES * STAGE > 8 * 2 * XAREA ? STAGES * STAGE : 8 * 2 * XAREA;
  static constexpr int ROWS = 1024 / ROW;                     // rows that one instruction of a wave fills
  static constexpr int WAVES = BOTH ? 4 : 8;                  // that load a part
  static constexpr int TLOADS = XTM / ROWS / WAVES, WLOADS = FEATS / ROWS / WAVES;
  // 16 rows x the same chunk are 16 different places of 16 bytes in the 64 banks
  static __device__ int swizzle(int row) { return BOTH ? (row >> 2) & 3 : swz<64>(row); }
};

template <int D, int MODE, bool BOTH>
__global__ __launch_bounds__(XNT, 2) void gate_proj_wide_bf16_kernel(const GateProj p, const int num_tt, const int num_ft,
                                                                     const long total_work) {
  using X = Wide<BOTH>;
  __shared__ __attribute__((aligned(1024))) char smem[X::LDS];
  const long work = xcd_work_index(total_work);
  if (work < 0) return;
  const int ft = (int)(work % num_ft);
  long rest = work / num_ft;
  const int tt = (int)(rest % num_tt);
  rest /= num_tt;
  const int b = (int)(rest % p.B);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int x = BOTH ? wave >> 2 : (MODE == GP_BWD_INPUT ? (int)(rest / p.B) : 0);  // this wave's branch
  const int wl = BOTH ? wave & 3 : wave, wm = wl & 1, wn = wl >> 1;                 // among the branch's waves: token half, 64 features
  const int g2 = lane >> 5, c32 = lane & 31;
  const int n = p.n, H = p.Hq, dm = H * D;
  const int i0 = tt * XTM, o0 = ft * X::FEATS;
  const int nk = dm / X::K;
  const bf16_t* __restrict__ Yb = reinterpret_cast<const bf16_t*>(p.Y_x[x]) + (size_t)b * H * n * D;
  const bf16_t* __restrict__ Wb = reinterpret_cast<const bf16_t*>(p.W_x[x]) + (size_t)o0 * dm;

  // loader: one instruction of a wave fills 1 KB of a tile; the lane delivers one physical chunk of one of its rows
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
  const uint32_t part = lds0 + (BOTH ? x * X::PART : 0);
  constexpr int CH = X::ROW / 16;  // chunks of a row
  uint32_t toff[X::TLOADS], woff[X::WLOADS];
#pragma unroll
  for (int j = 0; j < X::TLOADS; ++j) {
    const int row = X::ROWS * (wl + X::WAVES * j) + lane / CH;
    toff[j] = (uint32_t)min(i0 + row, n - 1) * (uint32_t)(D * 2) + (((lane % CH) ^ X::swizzle(row)) * 16);
  }
#pragma unroll
  for (int j = 0; j < X::WLOADS; ++j) {
    const int row = X::ROWS * (wl + X::WAVES * j) + lane / CH;
    woff[j] = (uint32_t)row * (uint32_t)(dm * 2) + (((lane % CH) ^ X::swizzle(row)) * 16);
  }
  constexpr int LOADS = X::TLOADS + X::WLOADS;
  auto request = [&](int st, int buf, int from, int till) {  // instructions `from` to `till` of a step's LOADS
    const int k0 = st * X::K;
    const bf16_t* ys = Yb + (size_t)(k0 / D) * n * D + k0 % D;
    const bf16_t* ws = Wb + k0;
    const uint32_t to = part + buf * X::STAGE + wl * 1024;
#pragma unroll
    for (int j = from; j < till; ++j)
      load_to_lds_16(j < X::TLOADS ? ys : ws, j < X::TLOADS ? toff[j < X::TLOADS ? j : 0] : woff[j < X::TLOADS ? 0 : j - X::TLOADS], to + X::WAVES * 1024 * j);
  };

  // accumulator 4q + e of block (fi, ti) of lane (g2, c32): token 128 wm + 32 ti + c32, feature 64 wn + 32 fi + 8 q + 4 g2 + e
  f32x16 acc[2][4];
#pragma unroll
  for (int fi = 0; fi < 2; ++fi)
#pragma unroll
    for (int ti = 0; ti < 4; ++ti)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[fi][ti][i] = 0.f;

  typedef __attribute__((address_space(3))) const bf16x8* lds_bf16x8;
  const uint32_t chunk = (uint32_t)((g2 ^ X::swizzle(c32)) * 16);  // chunk g2 of row c32; chunk 2 ks + g2: ^ 32 ks
  const uint32_t tok_at = part + (128 * wm + c32) * X::ROW + chunk, wgt_at = part + (XTM + 64 * wn + c32) * X::ROW + chunk;
  request(0, 0, 0, LOADS);
  if (X::STAGES == 3) request(1, 1, 0, LOADS);
  int buf = 0;
  for (int st = 0; st < nk; ++st) {
    // step st of this wave has landed (the younger one of three buffers may be under way); after the barrier it is whole, and
    // everyone has read the operands of step st - 1, whose buffer is the next to be filled
    static_assert(!BOTH || X::TLOADS + X::WLOADS == 6, "the wait below");
    if (X::STAGES == 3 && st + 1 < nk) asm volatile("s_waitcnt vmcnt(6) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const bool more = st + X::STAGES - 1 < nk;
    const int into = buf == 0 ? X::STAGES - 1 : buf - 1;
    const uint32_t ta = tok_at + buf * X::STAGE, wa = wgt_at + buf * X::STAGE;
    bf16x8 fa[2][2], fb[2][4];
    auto operands = [&](int ks) {
#pragma unroll
      for (int fi = 0; fi < 2; ++fi) fa[ks & 1][fi] = *(lds_bf16x8)(uintptr_t)((wa ^ (32 * ks)) + fi * 32 * X::ROW);
#pragma unroll
      for (int ti = 0; ti < 4; ++ti) fb[ks & 1][ti] = *(lds_bf16x8)(uintptr_t)((ta ^ (32 * ks)) + ti * 32 * X::ROW);
    };
    operands(0);
#pragma unroll
    for (int ks = 0; ks < X::K / 16; ++ks) {
      if (ks + 1 < X::K / 16) operands(ks + 1);
      __builtin_amdgcn_sched_barrier(0);
      if (more && ks < 2) request(st + X::STAGES - 1, into, ks * LOADS / 2, (ks + 1) * LOADS / 2);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int ti = 0; ti < 4; ++ti)
#pragma unroll
        for (int fi = 0; fi < 2; ++fi) acc[fi][ti] = mfma_bf16(fa[ks & 1][fi], fb[ks & 1][ti], acc[fi][ti]);
      __builtin_amdgcn_sched_barrier(0);
    }
    buf = buf == X::STAGES - 1 ? 0 : buf + 1;
  }

  // The epilogue takes the wave's outputs in two halves of 64 tokens; tensors come and go as whole 128-byte pieces of rows
  // through the wave's own two areas.  (rows past n: the last row's values, never stored)
  char* const mine = smem + wave * (2 * XAREA);
  bf16_t* const area[2] = {reinterpret_cast<bf16_t*>(mine), reinterpret_cast<bf16_t*>(mine + XAREA)};
  const int o = o0 + 64 * wn;  // first of the wave's 64 features: inside one head
  const size_t col = ((size_t)b * H + o / D) * n * D + o % D + (lane & 7) * 8;
  const int t0 = i0 + 128 * wm + (lane >> 3);
  auto fetch_rows = [&](const void* src, int half, u32x4* v) {
#pragma unroll
    for (int pass = 0; pass < 8; ++pass)
      v[pass] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const bf16_t*>(src) + col + (size_t)min(t0 + 64 * half + 8 * pass, n - 1) * D);
  };
  auto put_rows = [&](bf16_t* a, const u32x4* v) {
#pragma unroll
    for (int pass = 0; pass < 8; ++pass) *reinterpret_cast<u32x4*>(a + (pass * 8 + (lane >> 3)) * XSTR + (lane & 7) * 8) = v[pass];
  };
  auto flush = [&](void* dst, int half, const bf16_t* a) {
#pragma unroll
    for (int pass = 0; pass < 8; ++pass) {
      const int token = t0 + 64 * half + 8 * pass;
      if (token < n)
        __builtin_nontemporal_store(*reinterpret_cast<const u32x4*>(a + (pass * 8 + (lane >> 3)) * XSTR + (lane & 7) * 8),
                                    reinterpret_cast<u32x4*>(reinterpret_cast<bf16_t*>(dst) + col + (size_t)token * D));
    }
  };
  auto at = [&](bf16_t* a, int fi, int t2, int q) { return reinterpret_cast<u32x2*>(a + (32 * t2 + c32) * XSTR + 32 * fi + 8 * q + 4 * g2); };

  void* const Gx = MODE == GP_FORWARD ? p.G_x[x] : nullptr;
  u32x4 r1[8], r2[8];
  fetch_rows(MODE == GP_FORWARD ? p.Y_x[x] : p.E1, 0, r1);
  if (MODE == GP_BWD_INPUT) fetch_rows(p.E2[x], 0, r2);
  __syncthreads();  // every wave has read its last operands: the areas are free
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    put_rows(area[0], r1);
    if (MODE == GP_BWD_INPUT) put_rows(area[1], r2);
    wave_lds_sync();
    if (half == 0) {
      fetch_rows(MODE == GP_FORWARD ? p.Y_x[x] : p.E1, 1, r1);
      if (MODE == GP_BWD_INPUT) fetch_rows(p.E2[x], 1, r2);
    }
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
      for (int fi = 0; fi < 2; ++fi)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          f32x16& v = acc[fi][2 * half + t2];
          const u32x2 a = *at(area[0], fi, t2, q);
          const float av[4] = {bf16lo(a[0]), bf16hi(a[0]), bf16lo(a[1]), bf16hi(a[1])};
          if (MODE == GP_FORWARD) {
            float gv[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              gv[e] = sigmoidf_rcp(v[4 * q + e]);
              v[4 * q + e] = gv[e] * av[e];
            }
            if (Gx) *at(area[1], fi, t2, q) = u32x2{pack_bf16(gv[0], gv[1]), pack_bf16(gv[2], gv[3])};
          } else {
            const u32x2 c = *at(area[1], fi, t2, q);
            const float r[4] = {fmaf(av[0], bf16lo(c[0]), v[4 * q]), fmaf(av[1], bf16hi(c[0]), v[4 * q + 1]),
                                fmaf(av[2], bf16lo(c[1]), v[4 * q + 2]), fmaf(av[3], bf16hi(c[1]), v[4 * q + 3])};
            *at(area[0], fi, t2, q) = u32x2{pack_bf16(r[0], r[1]), pack_bf16(r[2], r[3])};
          }
        }
    if (MODE == GP_BWD_INPUT || Gx) {
      wave_lds_sync();
      flush(MODE == GP_BWD_INPUT ? p.Y_out[x] : Gx, half, area[MODE == GP_BWD_INPUT ? 0 : 1]);
    }
    wave_lds_sync();
  }
  if (MODE == GP_BWD_INPUT) return;

  // Y: this wave writes the half of its branch's number, with the other branch's terms added (single path: both halves)
  auto terms = [&](int fi, int t2, int q, const char* w) { return reinterpret_cast<const f32x4*>(w + ((fi * 2 + t2) * 4 + q) * 1024 + lane * 16); };
  if (BOTH) {
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
      for (int fi = 0; fi < 2; ++fi)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          f32x4 give;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float lo = acc[fi][t2][4 * q + e], hi = acc[fi][2 + t2][4 * q + e];
            give[e] = x == 0 ? hi : lo;
            acc[fi][t2][4 * q + e] = x == 0 ? lo : hi;
          }
          *const_cast<f32x4*>(terms(fi, t2, q, mine)) = give;
        }
    __syncthreads();
    const char* theirs = smem + (wave ^ 4) * (2 * XAREA);
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
      for (int fi = 0; fi < 2; ++fi)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 got = *terms(fi, t2, q, theirs);
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[fi][t2][4 * q + e] += got[e];
        }
    __syncthreads();  // the partner has read this wave's share
  }
#pragma unroll
  for (int half = 0; half < (BOTH ? 1 : 2); ++half) {
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
      for (int fi = 0; fi < 2; ++fi)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x16& v = acc[fi][2 * half + t2];
          *at(area[0], fi, t2, q) = u32x2{pack_bf16(v[4 * q], v[4 * q + 1]), pack_bf16(v[4 * q + 2], v[4 * q + 3])};
        }
    wave_lds_sync();
    flush(p.Y, BOTH ? x : half, area[0]);
    wave_lds_sync();
  }
}

// The backward's launches serve both branches at once (blockIdx.y, .z or a part of the work list): per branch the three small
// passes cost a launch of 5 us each, and short calls leave the chip idle in the products.
struct GateBwd {
  const uint16_t* Y_x[2];
  const uint16_t* W_x[2];
  const uint16_t* G_x[2];
  const uint16_t* dY;
  uint16_t* dz[2];
  uint16_t* Wt[2];
  float* dWf[2];
  uint16_t* dW[2];
};

// dz = dY * y * g * (1 - g), rounded to bf16; 8 elements per thread, all branches at once: dY is read once for both (bound: HBM; the
// pass was 81 us for two branches at B4, n = 8192, 16 heads of 64, and the call is 13 us shorter without the second reading).
template <int BRANCHES>
__global__ __launch_bounds__(256) void gate_dz_bf16_kernel(const GateBwd p, const size_t vecs) {
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * 256;
  for (; i < vecs; i += stride) {
    const u32x4 a = *reinterpret_cast<const u32x4*>(p.dY + 8 * i);
    u32x4 y[BRANCHES], g[BRANCHES];
#pragma unroll
    for (int x = 0; x < BRANCHES; ++x) {
      y[x] = *reinterpret_cast<const u32x4*>(p.Y_x[x] + 8 * i);
      g[x] = *reinterpret_cast<const u32x4*>(p.G_x[x] + 8 * i);
    }
#pragma unroll
    for (int x = 0; x < BRANCHES; ++x) {
      u32x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float gl = bf16lo(g[x][e]), gh = bf16hi(g[x][e]);
        o[e] = pack_bf16(bf16lo(a[e]) * bf16lo(y[x][e]) * gl * (1.f - gl), bf16hi(a[e]) * bf16hi(y[x][e]) * gh * (1.f - gh));
      }
      *reinterpret_cast<u32x4*>(p.dz[x] + 8 * i) = o;
    }
  }
}

// Wt[k][o] = W[o][k] for a square bf16 matrix (dm a multiple of 64): 64 x 64 tiles through LDS; the same tile of the fp32 sums
// for dW is set to zero.  blockIdx.z = branch.
__global__ __launch_bounds__(256) void gate_bwd_setup_kernel(const GateBwd p, const int dm) {
  __shared__ uint16_t tile[64][66];
  const uint16_t* __restrict__ W = p.W_x[blockIdx.z];
  uint16_t* __restrict__ Wt = p.Wt[blockIdx.z];
  float* __restrict__ sums = p.dWf[blockIdx.z];
  const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
  for (int e = threadIdx.x; e < 64 * 64; e += 256) tile[e / 64][e % 64] = W[(size_t)(r0 + e / 64) * dm + c0 + e % 64];
  for (int e = threadIdx.x; e < 64 * 16; e += 256)
    *reinterpret_cast<f32x4*>(sums + (size_t)(r0 + e / 16) * dm + c0 + 4 * (e % 16)) = f32x4{0.f, 0.f, 0.f, 0.f};
  __syncthreads();
  for (int e = threadIdx.x; e < 64 * 64; e += 256) Wt[(size_t)(c0 + e / 64) * dm + r0 + e % 64] = tile[e % 64][e / 64];
}

// dW[o][k] += sum over a piece of the tokens of dz[t][o] * y[t][k].  Workgroup = 128 x 128 of dW, 4 waves
// as 2 x 2.  The contraction runs over tokens, which is the slow index of both operands in memory, so
// both tiles are brought in as they lie ([token][128 features], by direct global-to-LDS loads, unpadded
// rows with swizzled 16-byte chunks) and both operands are read with the transposing LDS read: a lane
// gets the same 8 tokens of one feature column for the A operand (dz^T) and the B operand (y).
// Steps of 32 tokens, four buffers, three steps in flight.  Tokens past a batch's end are zeroed in
// the dz tile after it has landed.
// A piece of the tokens per workgroup: a run of steps, over the batches one after the other.  A call of one or two batches that pieces
// of WCHUNK tokens cut into one or two is cut into two at most: two additions to zero give the same bits in either order, so dW
// repeats itself.  (It is the faster cut as well for 12 and 16 heads of 64:
// every further piece adds its 64 KB per tile in memory; the whole backward of the gates with 4 and 8 pieces, as many as fill the chip,
// and with two: n = 1100 51.6 / 44.3 us, 2048 65.4 / 48.3, 4096 78.5 / 64.6; with two heads, one tile, n = 8192 28.6 / 56.4.)
// Longer calls add in no fixed order: equal pieces, as many as fill the chip once, with two workgroups per CU where a piece then has WLONG
// tokens and one where not (whole backward, 512 / 256 workgroups, us: 16 heads of 64, B4 n = 8192 409 / 431, B1 n = 16384 203 / 217,
// 9000 145.5 / 144.9, B3 n = 2048 104 / 100; 8 heads, 13 x 476 64 / 55), each of WLEAST at least (3 x 512 of 4 heads 23.8, 256 workgroups 29.3; 13 x 613
// of two heads in pieces of 256 tokens 21.2, of 88 24.7), less where that leaves few workgroups (40 x 31 tokens of two heads in 4 pieces 22.3, in 19
// 20.1, in 38 20.3; of four heads in 4 24.6, in 9 22.7).
// Where tiles do not divide the places, one round stays partly empty and two to four rounds of shorter pieces are taken if they are filled better
// and a piece keeps WMANY tokens (tiles x tokens, pieces of one round / now, us: 288 x 32768 842 / 800, 338 x 32768 1110 / 1030, 200 x 65536 1202 / 1165, 324 x
// 32768 897 / 832, 144 x 65536 820 / 786, 288 x 8192 237 / 232; with 2048 tokens a piece 338 x 6144 213 / 221; more tiles than places, 648 x 32768 in one and
// in three 1710 / 1701, x 6144 340 / 351).
// Half as many pieces again (768 workgroups) 5 % slower and more where the round is full.  Pieces that end with their batch at 4096 tokens took 13 x 613
// tokens of 16 heads 190 us, now 139; 8 x 1024 of 12 heads 105, now 90; 16 x 4096 of 16 heads 840, now 798.
constexpr int WCHUNK = 4096, WLONG = 2048, WMANY = 2560, WLEAST = 256;
constexpr long WTARGET = 256;
constexpr int WSTEP = 32;
constexpr int WSTAGES = 4;
constexpr int WTILE_BYTES = WSTEP * 128 * 2;  // one operand, one step
constexpr int WSTAGE_BYTES = 2 * WTILE_BYTES;
constexpr int WLOADS_PER_STAGE = 4;           // instructions per thread: 2 rows of 16 tokens x 2 operands

template <int D>
__global__ __launch_bounds__(GNT, 2) void gate_dw_bf16_kernel(const GateBwd p, const int B, const int H, const int n, const int num_ft,
                                                               const int piece_steps, const int pieces, const long total_work) {
  __shared__ __attribute__((aligned(16))) char smem[WSTAGES * WSTAGE_BYTES];
  const long work = xcd_work_index(total_work);
  if (work < 0) return;
  const int kt = (int)(work % num_ft);  // input-feature tile (columns of dW)
  long rest = work / num_ft;
  const int ot = (int)(rest % num_ft);  // output-feature tile (rows of dW)
  rest /= num_ft;
  const int piece = (int)(rest % pieces), x = (int)(rest / pieces);  // x = branch
  const bf16_t* __restrict__ dz = reinterpret_cast<const bf16_t*>(p.dz[x]);
  const bf16_t* __restrict__ Yx = reinterpret_cast<const bf16_t*>(p.Y_x[x]);
  float* __restrict__ dW = p.dWf[x];
  const int dm = H * D;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wo = wave & 1, wk = wave >> 1;
  const int g2 = lane >> 5, c32 = lane & 31;
  const int steps_b = (n + WSTEP - 1) / WSTEP;  // steps of a batch
  const int first = piece * piece_steps, nsteps = min(piece_steps, B * steps_b - first);

  // loader: one instruction of a wave fills 4 token rows (256 bytes each) of a tile; the lane delivers
  // physical chunk lane % 16 of token row wave * 4 + lane / 16 (+16 for the second instruction), i.e.
  // fetches the logical chunk (lane % 16) ^ swz(row): 8 features of one head
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
  const int ld_row = wave * 4 + (lane >> 4);
  const int ld_feat = 8 * ((lane & 15) ^ swz<128>(ld_row));
  auto feature_offset = [&](int f) -> uint32_t {  // bytes from the batch's first element to (token 0, feature f)
    return (uint32_t)(((size_t)(f / D) * n * D + f % D) * 2);
  };
  const uint32_t zfeat = feature_offset(ot * 128 + ld_feat), yfeat = feature_offset(kt * 128 + ld_feat);
  int rb = first / steps_b, rrow = first % steps_b * WSTEP;  // batch and first row of the next request
  const size_t batch = (size_t)H * n * D;
  const bf16_t *zb = dz + rb * batch, *yb = Yx + rb * batch;
  auto request_step = [&](int st) {  // past the call's last step: its last row again, never used
    const int buf = st & (WSTAGES - 1);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int token = min(rrow + 16 * j + ld_row, n - 1);
      const uint32_t trow = (uint32_t)token * (uint32_t)(D * 2);
      const uint32_t dst = lds0 + buf * WSTAGE_BYTES + (16 * j + wave * 4) * 256;
      load_to_lds_16(zb, zfeat + trow, dst);
      load_to_lds_16(yb, yfeat + trow, dst + WTILE_BYTES);
    }
    rrow += WSTEP;
  };
  auto next_batch = [&]() {
    if (rrow >= n && rb + 1 < B) { rrow = 0; ++rb; zb += batch; yb += batch; }
  };

  int troff[4][2];
  swizzled_tr_offsets<128>(lane, troff);

  f32x16 acc[2][2];
#pragma unroll
  for (int oi = 0; oi < 2; ++oi)
#pragma unroll
    for (int ki = 0; ki < 2; ++ki)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[oi][ki][i] = 0.f;

  for (int st = 0; st < 3; ++st) {
    request_step(st);
    next_batch();
  }
  // The steps at which something happens beside the products: the request that ends its batch, and a batch's ragged last step.  (Looked for at
  // every step, the calls of few tiles, whose workgroups have a CU each, took 4 % longer: n = 8192 of two heads 53.2 -> 55.5 us.)
  constexpr int NEVER = 0x7fffffff;
  int ends_at = rb + 1 < B ? (n - 1 - rrow) / WSTEP : NEVER, ragged_at = n % WSTEP ? steps_b - 1 - first % steps_b : NEVER;
  int event = min(ends_at, ragged_at);
  for (int st = 0; st < nsteps; ++st) {
    const int buf = st & (WSTAGES - 1);
    // all but the two youngest steps of this wave have landed; after the barrier step st is visible and
    // everyone is done with the buffer of step st - 1, which step st + 3 may now overwrite
    __builtin_amdgcn_s_waitcnt(0x0F70 | (2 * WLOADS_PER_STAGE));  // vmcnt(8)
    __syncthreads();
    request_step(st + 3);
    bf16_t* Zt = reinterpret_cast<bf16_t*>(smem + buf * WSTAGE_BYTES);
    const bf16_t* Yt = reinterpret_cast<const bf16_t*>(smem + buf * WSTAGE_BYTES + WTILE_BYTES);
    if (__builtin_expect(st == event, 0)) {
      if (st == ends_at) {
        next_batch();
        ends_at = rb + 1 < B ? ends_at + steps_b : NEVER;
      }
      if (st == ragged_at) {  // tokens past the end contribute zeros
        const int row = tid >> 3;
        if (row >= n % WSTEP) {
          u32x4* r = reinterpret_cast<u32x4*>(Zt + row * 128 + (tid & 7) * 16);
          r[0] = u32x4{0u, 0u, 0u, 0u};
          r[1] = u32x4{0u, 0u, 0u, 0u};
        }
        ragged_at += steps_b;
        __syncthreads();
      }
      event = min(ends_at, ragged_at);
    }
#pragma unroll
    for (int ks = 0; ks < WSTEP / 16; ++ks) {
      bf16x8 fa[2], fb[2];
#pragma unroll
      for (int oi = 0; oi < 2; ++oi) fa[oi] = lds_read_transposed_swz(Zt + 16 * ks * 128, troff[2 * wo + oi]);
#pragma unroll
      for (int ki = 0; ki < 2; ++ki) fb[ki] = lds_read_transposed_swz(Yt + 16 * ks * 128, troff[2 * wk + ki]);
#pragma unroll
      for (int oi = 0; oi < 2; ++oi)
#pragma unroll
        for (int ki = 0; ki < 2; ++ki) acc[oi][ki] = mfma_bf16(fa[oi], fb[ki], acc[oi][ki]);
    }
  }
  wait_all_loads();  // the surplus steps requested near the end
  // accumulator 4q + x of lane (g2, c32): row o = 64wo + 32oi + 8q + 4g2 + x, column k = 64wk + 32ki + c32
#pragma unroll
  for (int oi = 0; oi < 2; ++oi)
#pragma unroll
    for (int ki = 0; ki < 2; ++ki)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int o = ot * 128 + 64 * wo + 32 * oi + 8 * (i / 4) + 4 * g2 + (i % 4);
        const int k = kt * 128 + 64 * wk + 32 * ki + c32;
        unsafeAtomicAdd(dW + (size_t)o * dm + k, acc[oi][ki][i]);  // hardware fp32 add, device memory
      }
}

// dW in bf16 from its fp32 sums.  blockIdx.y = branch.
__global__ __launch_bounds__(256) void gate_dw_round_kernel(const GateBwd p, const size_t pairs) {
  const float* __restrict__ src = p.dWf[blockIdx.y];
  uint16_t* __restrict__ dst = p.dW[blockIdx.y];
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * 256;
  for (; i < pairs; i += stride) {
    const f32x2 v = *reinterpret_cast<const f32x2*>(src + 2 * i);
    *reinterpret_cast<uint32_t*>(dst + 2 * i) = pack_bf16(v[0], v[1]);
  }
}

// Wide tiles come in rounds of 256 workgroups, one per CU; narrow ones (half a wide one of both branches each, a quarter of a 256 x 256
// one) in half rounds, a second one per CU.  A wide round takes as long as two half rounds of the forward of both branches, and as
// three at least where a wide tile is four narrow ones.  Wide / narrow (us), 16 heads of 64, one sequence, by wide workgroups:
//   both branches forward   112 34.9 / 30.6, 144 35.1 / 40.6, 256 43.7 / 48.0, 272 75.7 / 72.2, 384 77.3 / 75.7, 416 79.6 / 87.9, 512 86.2 / 92.2,
//                           640 119 / 117, 704 123 / 129, 1024 171 / 180
//   backward of both        112 80.2 / 77.4, 144 88.3 / 95.0, 256 124 / 131, 320 159 / 154, 352 165 / 169, 416 183 / 196, 512 207 / 224, 576 272 / 270
//   single path             128 29.3 / 26.6, 136 28.7 / 39.3, 256 38.8 / 49.2, 288 63.5 / 61.0, 352 65.1 / 69.2, 448 69.1 / 86.8
// Short sequences, whose last tile a wide one pads further (batch x tokens, heads of 64): 16 x 300 of 16 38.6 / 40.6, 16 x 513 of 12 54.1 / 34.5,
// 13 x 1030 of 16 109 / 84, backward 10 x 513 of 16 97 / 107, 16 x 513 of 12 109 / 99; 130 x 40 of 2 13.7 / 9.7.
// A wide tile's longer start and end need steps to pay for them.  What that comes to depends on whether the call's inputs are still in the last
// level cache (hot: the same buffers again and again; else 600 MB of buffers in turn, as a program's layers use them).  Wide / narrow:
//   forward of both, dm < 1024: up to 8 % faster hot and as much slower in turn (dm = 768: 4 x 8192 112 / 118 hot, 123 / 124; 2 x 8474 66.9 / 69.5, 76.7 / 70.7; 6 x 8400
//     179 / 188, 200 / 198; 13 x 2774 139 / 133, 152 / 142; dm = 512: 3 x 4096 24.9 / 26.1, 28.8 / 27.7; 2 x 16384 62.5 / 58.4, 67.9 / 63.6; 4 x 14579 112 / 109, 122 /
//     117).  Behind the attention, in sa_dual_path_fwd with buffers in turn, its forward is slower with wide tiles in 66 of 70 such calls, mostly by 1 to 3 %; at dm = 1024 to 1536 level
//     where the tokens are whole tiles and up to 4 % slower where not, at 2048 2 to 4 % faster
//   the others at dm = 768 as from 1024 on (in turn: single path 6 x 8192 93.6 / 94.8, 9 x 3454 58.7 / 61.8, 8 x 8192 106 / 132; backward of both 4 x 6077 218 / 219,
//     9 x 2845 223 / 229, 2 x 8192 160 / 157; single path's 11 x 4096 of 3 whole half rounds a wide one 85.8 / 89.6)
//   at dm = 512 in one round or with half a round to spare (single path 6 x 8192 52.4 / 48.0, 10 x 4427 45.7 / 44.7, 7 x 8192 53.7 / 55.4; backward of both 6 x 3504
//     117 / 117, 14 x 2048 137 / 141)
//   below that the single path's forward in one round (dm = 256: 3 x 16384 18.6 / 21.2, 12 x 2721 15.3 / 18.2, 13 x 4096 20.5 / 23.6; the exception 6 x 8192 21.9 / 20.8;
//     backward of both 17 x 2729 104 / 100, 12 x 4096 107 / 104)
bool wide_is_faster(long wide, long narrow, bool backward, bool dual, long dm) {
  const long rounds = (wide + 255) / 256, halves = (narrow + 255) / 256;
  if (wide < 1) return false;
  if (!backward && dual) return dm >= 1024 && halves >= 2 * rounds;
  if (dm < 512) return !backward && rounds == 1 && halves >= 3;
  return dm >= 768 || rounds == 1 ? halves >= 3 * rounds : 2 * halves >= 7 * rounds;
}

struct Tiles {
  int wide, num_tt, num_ft;  // token tiles, feature tiles
  long total;
};
Tiles gate_tiles(int B, int Hq, int n, int d, bool backward, bool dual) {
  const long dm = (long)Hq * d;
  const int parts = backward && dual ? 2 : 1;  // of the work list
  const bool both = !backward && dual;
  const int feats = both ? Wide<true>::FEATS : Wide<false>::FEATS;
  const int num_tt = (n + TM - 1) / TM, wide_tt = (n + XTM - 1) / XTM;
  const long total = (long)num_tt * (dm / TN) * B * parts, wide = dm % feats ? 0 : (long)wide_tt * (dm / feats) * B * parts;
  if ((size_t)n * d * 2 < ((size_t)1 << 32) && wide_is_faster(wide, total, backward, dual, dm)) return {1, wide_tt, (int)(dm / feats), wide};  // 32-bit offsets inside a head
  return {0, num_tt, (int)(dm / TN), total};
}

template <int MODE>
hipError_t launch_gemm(const GateProj& p, hipStream_t st) {
  const bool dual = p.Y_x[1] != nullptr, both = MODE == GP_FORWARD && dual;
  const Tiles t = gate_tiles(p.B, p.Hq, p.n, p.d, MODE == GP_BWD_INPUT, dual);
  const long blocks = xcd_grid_blocks(t.total);
  if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks), block(t.wide ? XNT : GNT);
  if (t.wide && both) {
    if (p.d == 64) hipLaunchKernelGGL((gate_proj_wide_bf16_kernel<64, GP_FORWARD, true>), grid, block, 0, st, p, t.num_tt, t.num_ft, t.total);
    else hipLaunchKernelGGL((gate_proj_wide_bf16_kernel<128, GP_FORWARD, true>), grid, block, 0, st, p, t.num_tt, t.num_ft, t.total);
  } else if (t.wide) {
    if (p.d == 64) hipLaunchKernelGGL((gate_proj_wide_bf16_kernel<64, MODE, false>), grid, block, 0, st, p, t.num_tt, t.num_ft, t.total);
    else hipLaunchKernelGGL((gate_proj_wide_bf16_kernel<128, MODE, false>), grid, block, 0, st, p, t.num_tt, t.num_ft, t.total);
  } else {
    if (p.d == 64) hipLaunchKernelGGL((gate_proj_fwd_bf16_kernel<64, MODE>), grid, block, 0, st, p, t.num_tt, t.num_ft, t.total);
    else hipLaunchKernelGGL((gate_proj_fwd_bf16_kernel<128, MODE>), grid, block, 0, st, p, t.num_tt, t.num_ft, t.total);
  }
  return hipGetLastError();
}

unsigned capped_blocks(size_t items, size_t per_block) {
  const size_t want = (items + per_block - 1) / per_block;
  return (unsigned)(want < 1 ? 1 : (want > 65536 ? 65536 : want));
}

}  // namespace

bool gate_proj_wide_serves(int B, int Hq, int n, int d, bool backward, bool dual) { return gate_tiles(B, Hq, n, d, backward, dual).wide; }

hipError_t launch_gate_proj_fwd_bf16(int B, int Hq, int n, int d, const void* Y_sa, const void* Y_swa, const void* W_sa,
                                     const void* W_swa, void* Y, void* G_sa, void* G_swa, hipStream_t st) {
  if (B < 1 || Hq < 1 || n < 1 || !Y_sa || !W_sa || !Y) return hipErrorInvalidValue;
  if ((Y_swa == nullptr) != (W_swa == nullptr)) return hipErrorInvalidValue;
  if (!(d == 64 || d == 128)) return hipErrorNotSupported;
  const long dm = (long)Hq * d;
  if (dm % TN != 0 || dm % TK != 0) return hipErrorNotSupported;  // whole feature tiles only
  GateProj p = {};
  p.Y_x[0] = Y_sa; p.Y_x[1] = Y_swa;
  p.W_x[0] = W_sa; p.W_x[1] = W_swa;
  p.G_x[0] = G_sa; p.G_x[1] = G_swa;
  p.Y = Y;
  p.B = B; p.Hq = Hq; p.n = n; p.d = d;
  return launch_gemm<GP_FORWARD>(p, st);
}

size_t gate_proj_bwd_workspace_bytes(int B, int Hq, int n, int d, bool dual) {
  const size_t dm = (size_t)Hq * d, act = (size_t)B * Hq * n * d;
  const size_t per_branch = act * 2 /* dz bf16 */ + dm * dm * 2 /* W^T bf16 */ + dm * dm * 4 /* dW fp32 */;
  return (dual ? 2 : 1) * ((per_branch + 255) / 256 * 256);
}

// Pieces that the tokens of dW are cut into (see gate_dw_bf16_kernel): tiles = those of 128 x 128 of all branches.
long gate_proj_dw_pieces(long tiles, int B, int n) {
  const long tokens = (long)n * B, chunks = (long)((n + WCHUNK - 1) / WCHUNK) * B, places = 2 * WTARGET;
  if (chunks <= 2) return B == 1 && n > WLEAST && tiles * chunks < places ? 2 : chunks;
  long pieces = places / tiles;
  if (pieces * WLONG > tokens) pieces = WTARGET / tiles;
  if (pieces * WLEAST > tokens) {
    const long few = 32 / tiles < 16 ? 32 / tiles : 16, few_short = tokens / 64 < few ? tokens / 64 : few;
    pieces = tokens / WLEAST > few_short ? tokens / WLEAST : few_short;
  }
  if (pieces < 1) pieces = 1;
  // where whole tiles leave places of the one round empty: the rounds, four at most, that are filled best
  long rounds = 1;
  for (long r = 2; r <= 4 && tiles <= places; ++r) {
    const long more = r * places / tiles;
    if (more * WMANY > tokens) break;
    if (more * rounds * 100 > pieces * r * 103) { pieces = more; rounds = r; }
  }
  return pieces;
}

// `branches` branches at once: dz, W^T, dy_x = dY * g_x + dz W_x, dW_x = dz^T y_x.
static hipError_t gate_proj_bwd_branches(int branches, int B, int Hq, int n, int d, const void* const* Y_x, const void* const* W_x,
                                         const void* const* G_x, const void* dY, void* const* dY_x, void* const* dW_x, char* ws,
                                         hipStream_t st) {
  const size_t dm = (size_t)Hq * d, act = (size_t)B * Hq * n * d, per_branch = gate_proj_bwd_workspace_bytes(B, Hq, n, d, false);
  GateBwd p = {};
  GateProj g = {};
  p.dY = reinterpret_cast<const uint16_t*>(dY);
  g.E1 = dY;
  g.B = B; g.Hq = Hq; g.n = n; g.d = d;
  for (int x = 0; x < branches; ++x) {
    char* base = ws + x * per_branch;
    p.Y_x[x] = reinterpret_cast<const uint16_t*>(Y_x[x]);
    p.W_x[x] = reinterpret_cast<const uint16_t*>(W_x[x]);
    p.G_x[x] = reinterpret_cast<const uint16_t*>(G_x[x]);
    p.dz[x] = reinterpret_cast<uint16_t*>(base);
    p.Wt[x] = reinterpret_cast<uint16_t*>(base + act * 2);
    p.dWf[x] = reinterpret_cast<float*>(base + act * 2 + dm * dm * 2);
    p.dW[x] = reinterpret_cast<uint16_t*>(dW_x[x]);
    g.Y_x[x] = p.dz[x]; g.W_x[x] = p.Wt[x];
    g.Y_out[x] = dY_x[x]; g.E2[x] = G_x[x];
  }
  const unsigned blocks64 = (unsigned)(dm / 64);
  hipLaunchKernelGGL(gate_bwd_setup_kernel, dim3(blocks64, blocks64, branches), dim3(256), 0, st, p, (int)dm);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (branches == 2) hipLaunchKernelGGL(gate_dz_bf16_kernel<2>, dim3(capped_blocks(act / 8, 256)), dim3(256), 0, st, p, act / 8);
  else hipLaunchKernelGGL(gate_dz_bf16_kernel<1>, dim3(capped_blocks(act / 8, 256)), dim3(256), 0, st, p, act / 8);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = launch_gemm<GP_BWD_INPUT>(g, st);
  if (e != hipSuccess) return e;
  const int num_ft = (int)(dm / 128);
  const long tiles = (long)num_ft * num_ft * branches, steps = (long)((n + WSTEP - 1) / WSTEP) * B;
  if (steps > 0x7fffffffL) return hipErrorNotSupported;
  long pieces = gate_proj_dw_pieces(tiles, B, n);
  const int piece_steps = (int)((steps + pieces - 1) / pieces);
  pieces = (steps + piece_steps - 1) / piece_steps;
  const long total = tiles * pieces, blocks = xcd_grid_blocks(total);
  if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
  if (d == 64) hipLaunchKernelGGL(gate_dw_bf16_kernel<64>, dim3((unsigned)blocks), dim3(GNT), 0, st, p, B, Hq, n, num_ft, piece_steps, (int)pieces, total);
  else hipLaunchKernelGGL(gate_dw_bf16_kernel<128>, dim3((unsigned)blocks), dim3(GNT), 0, st, p, B, Hq, n, num_ft, piece_steps, (int)pieces, total);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(gate_dw_round_kernel, dim3(capped_blocks((size_t)dm * dm / 2, 256), branches), dim3(256), 0, st, p, (size_t)dm * dm / 2);
  return hipGetLastError();
}

hipError_t launch_gate_proj_bwd_bf16(int B, int Hq, int n, int d, const void* Y_sa, const void* Y_swa, const void* W_sa,
                                     const void* W_swa, const void* G_sa, const void* G_swa, const void* dY, void* dY_sa,
                                     void* dY_swa, void* dW_sa, void* dW_swa, void* ws, hipStream_t st) {
  if (B < 1 || Hq < 1 || n < 1 || !Y_sa || !W_sa || !G_sa || !dY || !dY_sa || !dW_sa || !ws) return hipErrorInvalidValue;
  const bool dual = Y_swa != nullptr;
  if (dual != (W_swa != nullptr) || dual != (G_swa != nullptr) || dual != (dY_swa != nullptr) || dual != (dW_swa != nullptr))
    return hipErrorInvalidValue;
  if (!(d == 64 || d == 128)) return hipErrorNotSupported;
  const long dm = (long)Hq * d;
  if (dm % 128 != 0) return hipErrorNotSupported;
  if ((size_t)dm * n * 2 >= ((size_t)1 << 32)) return hipErrorNotSupported;  // 32-bit byte offsets inside a batch
  const void *const Y_x[2] = {Y_sa, Y_swa}, *const W_x[2] = {W_sa, W_swa}, *const G_x[2] = {G_sa, G_swa};
  void *const dY_x[2] = {dY_sa, dY_swa}, *const dW_x[2] = {dW_sa, dW_swa};
  // Both at once unless an output of one shares memory with what the other still reads (the second branch's gradient in the
  // place of dY, for instance): then one after the other.
  const size_t bytes = (size_t)B * Hq * n * d * 2;
  auto overlap = [&](const void* a, const void* b) {
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return x < y + bytes && y < x + bytes;
  };
  bool apart = true;
  if (dual)
    for (int x = 0; x < 2; ++x)
      apart = apart && !overlap(dY_x[x], dY) && !overlap(dY_x[x], Y_x[1 - x]) && !overlap(dY_x[x], G_x[1 - x]) && !overlap(dY_x[x], dY_x[1 - x]);
  char* base = reinterpret_cast<char*>(ws);
  if (dual && apart) return gate_proj_bwd_branches(2, B, Hq, n, d, Y_x, W_x, G_x, dY, dY_x, dW_x, base, st);
  hipError_t e = gate_proj_bwd_branches(1, B, Hq, n, d, Y_x, W_x, G_x, dY, dY_x, dW_x, base, st);
  if (e != hipSuccess || !dual) return e;
  return gate_proj_bwd_branches(1, B, Hq, n, d, Y_x + 1, W_x + 1, G_x + 1, dY, dY_x + 1, dW_x + 1,
                                base + gate_proj_bwd_workspace_bytes(B, Hq, n, d, false), st);
}

}  // namespace sa
