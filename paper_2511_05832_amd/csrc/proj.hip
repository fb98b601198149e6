// Token-wise linear projections of the layer pipeline, with the head split /
// merge folded into the addressing (Sec. 4.2, input processing: the QKV
// projection follows the Hilbert reordering; Sec. 3.3: the attention output is
// projected back).
//
//   QKV:  y[t, f] = sum_k x[t, k] W[f, k], f in [0, 3C), scattered into
//         q / k / v [B, heads, N, d] by f -> (which, head, e)
//   out:  y[t, f] = sum_k o[b, k/d, n, k%d] W[f, k]  (heads merged on the fly)
//
// Two kernels, both with A = rows of W (features x k) and B = the input rows (k x
// tokens), fp32 accumulation: the streaming one keeps all weights in registers
// (K = 192, the shapes whose weight matrix fits), the tiled one takes any shape.
#include "attn_common.h"

namespace hla {
namespace {

struct ProjArgs {
  const __bf16 *in;   // x [T, K] (QKV) or o [B, heads, N, d] (out)
  // null, or the reordering fused in: QKV reads token n of batch b from input
  // row b*N + order[n]; the output projection writes it to row b*N + order[n]
  const int32_t *order;
  const __bf16 *w;    // [F, K]
  __bf16 *out0, *out1, *out2;  // q, k, v (QKV) or y (out, out0 only)
  int32_t T, N, K, F, heads, d, C;
};

// ---------------------------------------------------------------------------
// Streaming kernel (weights in registers). For the layer's shapes (K = 192,
// F = 576 or 192) the whole weight matrix fits the registers of one workgroup
// of twelve waves: wave w keeps the A operands of its FBW blocks of 16 output
// features for all of K (v_mfma_f32_16x16x32_bf16; FBW * K/32 * 4 VGPRs). The
// workgroup is persistent (one per CU) and streams tiles of 32 tokens:
//  - x rows come into a 5-stage LDS ring by the 16-byte LDS DMA, 1 KiB per
//    instruction, four tiles ahead; the 16-byte chunks of a row are stored XOR-
//    swizzled by (row & 7) (each lane fetches the chunk that belongs in its
//    slot), which puts the B-operand reads (16 rows x one chunk per 16 lanes) on
//    distinct banks;
//  - the results are staged through LDS as [token][feature] rows and written
//    back with non-temporal 16-byte stores in output order: one wave instruction covers 1 KiB
//    of q / k / v (d = 32: 16 consecutive token rows of one head) or of y. (The
//    accumulator layout - four features of one token per lane - stored
//    directly gave 8-byte stores into 32 different rows per instruction and ran
//    at a third of the write bandwidth.)
// Every wave issues the same number of copies and stores per tile (lanes past
// the last token re-read and re-store row T - 1, the same bytes to the same
// place), so each wait leaves an exact number of them in flight: the vmcnt
// counter is in order. With the reordering fused in, the order entries of all
// of the workgroup's tokens are copied into LDS once, before the tiles.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr int kStreamTT = 32;      // tokens per tile
constexpr int kStreamAhead = 4;    // x tiles in flight ahead of the current one
constexpr int kStreamRing = kStreamAhead + 1;
constexpr int kStreamMaxTiles = 64;  // tiles per workgroup (order entries in LDS)
constexpr int kStreamWaves = 12;

struct StreamArgs {
  const __bf16 *in;        // x [T, K] (QKV) or o [B, heads, N, d] (out)
  const int32_t *order;    // null, or the token reordering fused in (see ProjArgs)
  const __bf16 *w;         // [F, K]
  __bf16 *out0, *out1, *out2;
  int32_t T, N, ntiles;
  FastDiv ndiv;            // division by N
};

// LDS writes of this wave done, then barrier (vector memory left in flight).
__device__ __forceinline__ void lds_then_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// KS = K / 32; D head dim; FBW 16-feature blocks per wave; MODE 0 QKV, 1 output
// projection; ORD: an order array is given.
template <int KS, int D, int FBW, int MODE, bool ORD>
__global__ void __launch_bounds__(64 * kStreamWaves, 1) proj_stream_kernel(StreamArgs p) {
  constexpr int NWV = kStreamWaves;
  constexpr int TT = kStreamTT;
  constexpr int A = kStreamAhead;
  constexpr int R = kStreamRing;
  constexpr int K = 32 * KS;
  constexpr int HEADS = K / D;
  constexpr int F = 16 * FBW * NWV;
  constexpr int CPR = K / 8;                        // 16-byte chunks per x row
  constexpr int XTILE = TT * K * 2;                 // bytes of one x tile
  constexpr int CPW = TT * CPR / (64 * NWV);        // x copies per wave and tile
  constexpr int FP = F + 8;                         // staging row pitch, elements
  constexpr int SPW = TT * F / 8 / (64 * NWV);      // 16-byte stores per wave and tile
  constexpr int XR = 0;
  constexpr int ST = XR + R * XTILE;
  constexpr int IX = ST + TT * FP * 2;
  constexpr int LDSB = IX + (ORD ? kStreamMaxTiles * TT * 4 : 0);
  constexpr int MAXN = CPW * (A - 1) + SPW * A;
  static_assert(TT * CPR % (64 * NWV) == 0 && TT * F / 8 % (64 * NWV) == 0, "work must split evenly");
  static_assert(MODE == 0 ? F == 3 * K : true, "QKV: F = 3 C");
  static_assert(CPR % 8 == 0, "the chunk swizzle works within octets");
  static_assert(MAXN < 64, "vmcnt range");

  __shared__ __attribute__((aligned(16))) char lds[LDSB];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g4 = lane >> 4;
  const int fw = wave * FBW * 16;   // this wave's first feature

  // Tiles of this workgroup: blockIdx.x, blockIdx.x + gridDim.x, ... (at most
  // kStreamMaxTiles; the launcher sizes the grid for that).
  const int nt = ((int)blockIdx.x < p.ntiles)
                     ? (p.ntiles - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x
                     : 0;
  auto tile_of = [&](int i) { return (int)blockIdx.x + i * (int)gridDim.x; };
  auto clamp_t = [&](int t) { return t < p.T ? t : p.T - 1; };

  // x tile i into ring stage i % R: slot q of the tile holds row q / CPR, chunk
  // (q % CPR) ^ (row & 7) of the source. QKV with an order: entry r of `rows`
  // is the order entry of the tile's token r (`rows` = the LDS copy of the
  // order entries, or, for the first tiles, registers - see below).
  const int32_t *idx_all = reinterpret_cast<const int32_t *>(lds + IX);
  auto issue_x_from = [&](int i, auto row_of) {
    char *stage = lds + XR + (i % R) * XTILE;
#pragma unroll
    for (int j = 0; j < CPW; ++j) {
      const int q = (j * NWV + wave) * 64 + lane;
      const int r = q / CPR, c = (q % CPR) ^ (r & 7);
      const int t = clamp_t(tile_of(i) * TT + r);
      const int b = (int)fdiv((uint32_t)t, p.ndiv), n = t - b * p.N;
      const __bf16 *src;
      if constexpr (MODE == 0) {
        const int64_t row = ORD ? (int64_t)b * p.N + row_of(j, r) : (int64_t)t;
        src = p.in + row * K + 8 * c;
      } else {
        const int h = (8 * c) / D, e = (8 * c) % D;
        src = p.in + ((int64_t)(b * HEADS + h) * p.N + n) * D + e;
      }
      lds_dma16(src, lds_addr(stage + (j * NWV + wave) * 1024));
    }
  };
  auto issue_x = [&](int i) {
    const int32_t *idx = idx_all + i * TT;
    issue_x_from(i, [&](int, int r) { return idx[r]; });
  };

  // Prologue, all in flight together: (QKV with an order) this lane's order
  // entries for the first A tiles, loaded into registers first; the weights (the
  // A operand of block fb, k-step s = W[fw + 16 fb + l16][32 s + 8 g4 ..]); the
  // order entries of every token of this workgroup's tiles into LDS (entry e =
  // token e % 32 of tile e / 32); the x copies of the first A tiles. Then one
  // wait and a barrier. (The compiler's own wait before the first tiles' x
  // addresses covers only the order loads issued ahead of the weights.)
  int first_rows[A][CPW];
  if constexpr (ORD && MODE == 0) {
#pragma unroll
    for (int i = 0; i < A; ++i)
#pragma unroll
      for (int j = 0; j < CPW; ++j) {
        const int r = ((j * NWV + wave) * 64 + lane) / CPR;
        const int t = clamp_t(min(tile_of(i), p.ntiles - 1) * TT + r);
        const int b = (int)fdiv((uint32_t)t, p.ndiv);
        first_rows[i][j] = p.order[t - b * p.N];
      }
  }
  bf16x8 wr[FBW][KS];
#pragma unroll
  for (int fb = 0; fb < FBW; ++fb)
#pragma unroll
    for (int s = 0; s < KS; ++s)
      wr[fb][s] = *reinterpret_cast<const bf16x8 *>(p.w + (int64_t)(fw + 16 * fb + l16) * K + 32 * s + 8 * g4);
  if constexpr (ORD) {
    for (int c = wave; c * 64 < nt * TT; c += NWV) {
      const int e = min(c * 64 + lane, nt * TT - 1);
      const int t = clamp_t(tile_of(e / TT) * TT + e % TT);
      const int b = (int)fdiv((uint32_t)t, p.ndiv);
      lds_dma4(p.order + (t - b * p.N), lds_addr(lds + IX + c * 256));
    }
  }
#pragma unroll
  for (int i = 0; i < A; ++i)
    if (i < nt) issue_x_from(i, [&](int j, int) { return first_rows[i][j]; });
  wait_vmem_all();
  wait_then_barrier<0>();

  // B-operand byte offsets within a stage: token block tb, k-step s.
  int boff[2][KS];
#pragma unroll
  for (int tb = 0; tb < 2; ++tb)
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int r = 16 * tb + l16, c = (4 * s + g4) ^ (r & 7);
      boff[tb][s] = r * K * 2 + c * 16;
    }

  for (int i = 0; i < nt; ++i) {
    // This wave's operations issued after tile i's x copies: the copies of tiles
    // i + 1 .. i + A - 1 and the stores of tiles i - A .. i - 1 (those that exist).
    wait_n_then_barrier<MAXN>(CPW * min(A - 1, nt - 1 - i) + SPW * min(i, A));
    // (stage (i + A) % R held tile i - 1, which every wave finished before the
    // barrier above)
    if (i + A < nt) issue_x(i + A);

    const char *stage = lds + XR + (i % R) * XTILE;
    f32x4 acc[FBW][2];
#pragma unroll
    for (int fb = 0; fb < FBW; ++fb) acc[fb][0] = acc[fb][1] = f32x4{};
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int tb = 0; tb < 2; ++tb) {
        const bf16x8 xop = *reinterpret_cast<const bf16x8 *>(stage + boff[tb][s]);
#pragma unroll
        for (int fb = 0; fb < FBW; ++fb)
          acc[fb][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wr[fb][s], xop, acc[fb][tb], 0, 0, 0);
      }
    // Stage as [token][feature]: lane (l16, g4) of block (fb, tb) holds token
    // 16 tb + l16, features fw + 16 fb + 4 g4 + 0..3. (The staging area was last
    // read in tile i - 1's stores, before the barrier above.)
#pragma unroll
    for (int fb = 0; fb < FBW; ++fb)
#pragma unroll
      for (int tb = 0; tb < 2; ++tb) {
        bf16x4 o4;
#pragma unroll
        for (int e = 0; e < 4; ++e) o4[e] = (__bf16)acc[fb][tb][e];
        *reinterpret_cast<bf16x4 *>(lds + ST + ((16 * tb + l16) * FP + fw + 16 * fb + 4 * g4) * 2) = o4;
      }
    lds_then_barrier();
    // Stores in output order, 16 bytes per lane.
    const int32_t *idx = idx_all + i * TT;
#pragma unroll
    for (int j = 0; j < SPW; ++j) {
      const int q = (j * NWV + wave) * 64 + lane;
      int r, feat;
      __bf16 *dst;
      if constexpr (MODE == 0) {
        // q -> (block = which * heads + h, token r, 8-feature chunk e8), e8 fastest
        constexpr int E8 = D / 8;
        const int e8 = q % E8;
        r = (q / E8) % TT;
        const int blk = q / (E8 * TT);
        feat = blk * D + 8 * e8;
        const int which = blk / HEADS, h = blk % HEADS;
        const int t = clamp_t(tile_of(i) * TT + r);
        const int b = (int)fdiv((uint32_t)t, p.ndiv), n = t - b * p.N;
        __bf16 *base = which == 0 ? p.out0 : (which == 1 ? p.out1 : p.out2);
        dst = base + ((int64_t)(b * HEADS + h) * p.N + n) * D + 8 * e8;
      } else {
        constexpr int CF = F / 8;
        const int c = q % CF;
        r = q / CF;
        feat = 8 * c;
        const int t = clamp_t(tile_of(i) * TT + r);
        const int b = (int)fdiv((uint32_t)t, p.ndiv), n = t - b * p.N;
        const int64_t row = (int64_t)b * p.N + (ORD ? idx[r] : n);
        dst = p.out0 + row * F + feat;
      }
      // non-temporal: the output streams past the caches (measured 13% faster
      // for the QKV projection, and the attention reading q, k, v next no slower)
      const u32x4 v = *reinterpret_cast<const u32x4 *>(lds + ST + (r * FP + feat) * 2);
      __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(dst));
    }
  }
}

template <int D, int MODE, bool ORD>
hipError_t launch_stream(const ProjArgs &a, hipStream_t s) {
  StreamArgs p;
  p.in = a.in;
  p.order = a.order;
  p.w = a.w;
  p.out0 = a.out0;
  p.out1 = a.out1;
  p.out2 = a.out2;
  p.T = a.T;
  p.N = a.N;
  p.ntiles = (a.T + kStreamTT - 1) / kStreamTT;
  p.ndiv = make_fastdiv((uint32_t)a.N);
  int cus = 0, dev = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
    cus = 256;
  // one workgroup per CU, more when a workgroup would get over kStreamMaxTiles tiles
  int grid = p.ntiles < cus ? p.ntiles : cus;
  const int need = (p.ntiles + kStreamMaxTiles - 1) / kStreamMaxTiles;
  if (need > grid) grid = need;
  // QKV: F = 576 = 12 waves x 3 blocks; output projection: F = 192 = 12 waves x 1
  constexpr int FBW = MODE == 0 ? 3 : 1;
  hipLaunchKernelGGL((proj_stream_kernel<6, D, FBW, MODE, ORD>), dim3(grid), dim3(64 * kStreamWaves), 0, s, p);
  return hipGetLastError();
}

template <int MODE>
hipError_t launch_stream_any(const ProjArgs &p, hipStream_t s) {
  if (p.d == 32) return p.order ? launch_stream<32, MODE, true>(p, s) : launch_stream<32, MODE, false>(p, s);
  return p.order ? launch_stream<64, MODE, true>(p, s) : launch_stream<64, MODE, false>(p, s);
}

// ---------------------------------------------------------------------------
// Tiled kernel: every other shape. y = x W^T as a matrix product of token tiles
// (64 MT tokens) and feature tiles (64 NF features) by four waves, two by two, each
// with MT x NF accumulators of 32 x 32 (v_mfma_f32_32x32x16_bf16, A = W rows, B = x
// rows). What bounds it: the matrix cores and LDS together - a wave reads MT + NF
// operands from LDS per MT * NF products, so a 64 x 96 wave tile (MT = 2, NF = 3)
// keeps the LDS at 5/6 of its rate when the matrix cores are full, while one
// operand read per product (a wave with one token block) fills it.
//  - x and W come in 32 contraction steps at a time, 64-byte rows, by the 16-byte
//    LDS DMA into a ring of three stages, two ahead (60 KiB at 128 x 192, two
//    workgroups per CU; 48 KiB at 128 x 128, three: one's first copies and stores
//    pass under the others' products). A fourth stage was 0-4% slower. Chunks are
//    XOR-swizzled by row / 2, which puts the eight rows of an operand read on
//    distinct banks.
//  - the results are staged through LDS (the ring, once it is drained) as
//    [token][feature] rows and leave with non-temporal 16-byte stores.
//  - the grid gives each XCD a contiguous range of token tiles with all their
//    feature tiles, feature tile fastest: x and W are read from HBM once and come
//    from that XCD's L2 after that.
constexpr int kTileWaves = 4;
constexpr int kTileRing = 3;
constexpr int kTileK = 32;   // contraction elements per stage

struct TileArgs {
  const __bf16 *in;
  const int32_t *order;
  const __bf16 *w;
  __bf16 *out0, *out1, *out2;
  int32_t T, N, K, F, heads, lgd, n_ftiles;
  FastDiv ndiv;   // division by N
  FastDiv fdiv_;  // division by n_ftiles
};

template <int MT, int NF, int MODE>
__global__ void __launch_bounds__(64 * kTileWaves, 2) proj_tile_kernel(TileArgs p) {
  constexpr int NW = kTileWaves, R = kTileRing;
  constexpr int TM = 64 * MT, TF = 64 * NF;        // tokens, features of the tile
  constexpr int ROWB = kTileK * 2;                 // bytes of a staged row
  constexpr int XB = TM * ROWB, STAGE = XB + TF * ROWB;
  constexpr int CX = TM * 4 / (64 * NW), CW = TF * 4 / (64 * NW);  // copies per thread
  constexpr int LPT = CX + CW;
  constexpr int FP = TF + 8;                       // output row pitch, elements
  static_assert(TM * FP * 2 <= R * STAGE, "the output tile must fit the ring");
  static_assert(LPT * (R - 2) < 64, "vmcnt range");
  __shared__ __attribute__((aligned(16))) char lds[R * STAGE];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 31, half = lane >> 5;
  const int wt = wave & 1, wf = wave >> 1;         // this wave's token and feature half
  const int logical = xcd_remap(blockIdx.x, gridDim.x);
  const int tt = (int)fdiv((uint32_t)logical, p.fdiv_);
  const int t0 = tt * TM, f0 = (logical - tt * p.n_ftiles) * TF;

  // Source of this thread's copies at contraction step 0: slot q = (j NW + wave) 64
  // + lane of a tile is row q / 4, chunk (q % 4) ^ (row / 2 % 4). Rows past the last
  // token read row T - 1 and are not stored.
  const __bf16 *xs[CX], *ws[CW];
#pragma unroll
  for (int j = 0; j < CX; ++j) {
    const int q = (j * NW + wave) * 64 + lane, r = q >> 2, c = (q & 3) ^ ((r >> 1) & 3);
    const int t = min(t0 + r, p.T - 1);
    const int b = (int)fdiv((uint32_t)t, p.ndiv), n = t - b * p.N;
    if (MODE == 0) xs[j] = p.in + ((int64_t)b * p.N + (p.order ? p.order[n] : n)) * p.K + 8 * c;
    else xs[j] = p.in + (((int64_t)b * p.heads * p.N + n) << p.lgd) + 8 * c;
  }
#pragma unroll
  for (int j = 0; j < CW; ++j) {
    const int q = (j * NW + wave) * 64 + lane, r = q >> 2, c = (q & 3) ^ ((r >> 1) & 3);
    ws[j] = p.w + (int64_t)(f0 + r) * p.K + 8 * c;
  }
  const int nk = p.K / kTileK;
  auto issue = [&](int i) {
    char *base = lds + (i % R) * STAGE;
    const int k0 = i * kTileK;
    // the input's step: k0 itself, or (heads merged on the fly) head k0 / d
    const int64_t off = MODE == 0 ? (int64_t)k0
                                  : ((int64_t)(k0 >> p.lgd) * p.N << p.lgd) + (k0 & ((1 << p.lgd) - 1));
#pragma unroll
    for (int j = 0; j < CX; ++j) lds_dma16(xs[j] + off, lds_addr(base + (j * NW + wave) * 1024));
#pragma unroll
    for (int j = 0; j < CW; ++j) lds_dma16(ws[j] + k0, lds_addr(base + XB + (j * NW + wave) * 1024));
  };

  // Operand offsets within a stage: step s = 0, 1 of 16 elements, this lane's row
  int xoff[2], woff[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int sw = ((2 * s + half) ^ ((col >> 1) & 3)) * 16;
    xoff[s] = (wt * 32 * MT + col) * ROWB + sw;
    woff[s] = XB + (wf * 32 * NF + col) * ROWB + sw;
  }

  f32x16 acc[NF][MT];
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[f][m] = f32x16{};

  wait_vmem_all();   // the order entries, before the first copy
#pragma unroll
  for (int i = 0; i < R - 1; ++i)
    if (i < nk) issue(i);
  for (int i = 0; i < nk; ++i) {
    // stage i has landed in every wave, and every wave is done with stage i - 1
    wait_tiles_then_barrier<LPT, R - 2>(min(R - 2, nk - 1 - i));
    if (i + R - 1 < nk) issue(i + R - 1);
    const char *base = lds + (i % R) * STAGE;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      bf16x8 x[MT], w[NF];
#pragma unroll
      for (int m = 0; m < MT; ++m) x[m] = *reinterpret_cast<const bf16x8 *>(base + xoff[s] + m * 32 * ROWB);
#pragma unroll
      for (int f = 0; f < NF; ++f) w[f] = *reinterpret_cast<const bf16x8 *>(base + woff[s] + f * 32 * ROWB);
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int m = 0; m < MT; ++m)
          acc[f][m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[f], x[m], acc[f][m], 0, 0, 0);
    }
  }

  // Stage as [token][feature]: lane (col, half) of block (f, m) holds token
  // 32 m + col, slots 4g .. 4g + 3 features 8g + 4 half ..
  wait_then_barrier<0>();   // every wave is done with the ring
  __bf16 *st = reinterpret_cast<__bf16 *>(lds);
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 o4;
#pragma unroll
        for (int e = 0; e < 4; ++e) o4[e] = (__bf16)acc[f][m][4 * g + e];
        *reinterpret_cast<bf16x4 *>(st + ((wt * MT + m) * 32 + col) * FP + (wf * NF + f) * 32 + 8 * g + 4 * half) = o4;
      }
  wait_then_barrier<0>();
  // Stores, 16 bytes per lane. QKV: chunk (token, 8 features of one head), so that a
  // wave's consecutive lanes write whole token rows of one head.
  constexpr int CF = TF / 8;
  constexpr int SPW = TM * CF / (64 * NW);
  static_assert(TM * CF % (64 * NW) == 0, "stores must split evenly");
#pragma unroll 4
  for (int j = 0; j < SPW; ++j) {
    const int q = (j * NW + wave) * 64 + lane;
    int r, c;
    if (MODE == 0) {   // (head, token, chunk in the head)
      const int le = p.lgd - 3;
      c = ((q >> le) / TM << le) + (q & ((1 << le) - 1));
      r = (q >> le) % TM;
    } else {
      r = q / CF;
      c = q % CF;
    }
    const int t = t0 + r;
    if (t >= p.T) continue;
    const int b = (int)fdiv((uint32_t)t, p.ndiv), n = t - b * p.N;
    __bf16 *dst;
    if (MODE == 0) {
      const int feat = f0 + 8 * c;
      const int which = (feat >= p.K) + (feat >= 2 * p.K), e = feat - which * p.K;   // C = K
      __bf16 *base = which == 0 ? p.out0 : (which == 1 ? p.out1 : p.out2);
      dst = base + ((((int64_t)b * p.heads + (e >> p.lgd)) * p.N + n) << p.lgd) + (e & ((1 << p.lgd) - 1));
    } else {
      dst = p.out0 + ((int64_t)b * p.N + (p.order ? p.order[n] : n)) * p.F + f0 + 8 * c;
    }
    const u32x4 v = *reinterpret_cast<const u32x4 *>(st + r * FP + 8 * c);
    __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(dst));
  }
}

template <int MT, int NF, int MODE>
hipError_t launch_tile(const ProjArgs &a, hipStream_t s) {
  TileArgs p;
  p.in = a.in;
  p.order = a.order;
  p.w = a.w;
  p.out0 = a.out0;
  p.out1 = a.out1;
  p.out2 = a.out2;
  p.T = a.T;
  p.N = a.N;
  p.K = a.K;
  p.F = a.F;
  p.heads = a.heads;
  p.lgd = a.d == 32 ? 5 : 6;
  p.n_ftiles = a.F / (64 * NF);
  p.ndiv = make_fastdiv((uint32_t)a.N);
  p.fdiv_ = make_fastdiv((uint32_t)p.n_ftiles);
  const int64_t ttiles = ((int64_t)a.T + 64 * MT - 1) / (64 * MT);
  hipLaunchKernelGGL((proj_tile_kernel<MT, NF, MODE>), dim3((uint32_t)(ttiles * p.n_ftiles)),
                     dim3(64 * kTileWaves), 0, s, p);
  return hipGetLastError();
}

// Tile shape: the widest feature tile that divides F, in tiles of 128 tokens;
// 64-token tiles where those would leave CUs without work. One contraction loop
// serves every K, down to two steps (K = 64). Against a kernel that kept a token
// block's rows in registers and walked the feature tiles (K = 64 and 128), 16 x 4096
// tokens: QKV 13.9 -> 7.4 and 24.6 -> 15.6 us, output projection to K features 6.5 ->
// 4.3 and 11.7 -> 7.0; 1024 tokens 5.5 -> 3.9, 9.7 -> 4.4, 4.0 -> 2.8, 5.0 -> 3.9.
template <int MODE>
hipError_t launch_tile_any(const ProjArgs &p, hipStream_t s) {
  const int cus = device_cu_count();
  const int nf = p.F % 192 == 0 ? 3 : (p.F % 128 == 0 ? 2 : 1);
  const bool wide = ((int64_t)p.T + 127) / 128 * (p.F / (64 * nf)) >= cus;
  if (nf == 3) return wide ? launch_tile<2, 3, MODE>(p, s) : launch_tile<1, 3, MODE>(p, s);
  if (nf == 2) return wide ? launch_tile<2, 2, MODE>(p, s) : launch_tile<1, 2, MODE>(p, s);
  return wide ? launch_tile<2, 1, MODE>(p, s) : launch_tile<1, 1, MODE>(p, s);
}

template <int MODE>
hipError_t launch_proj(ProjArgs p, hipStream_t s) {
  // streaming kernel (weights in registers) for K = 192 with F = 576 (QKV) or
  // F = 192 (output projection), d = 32 or 64: 16 x 4096 tokens 22.5 against the
  // tiled kernel's 27 us (QKV) and 10.3 against 11.2 (output); 64 x 4096 tokens 72
  // against 130 and 35 against 56
  if (p.K == 192 && (p.d == 32 || p.d == 64) && (MODE == 0 ? p.F == 576 : p.F == 192))
    return launch_stream_any<MODE>(p, s);
  return launch_tile_any<MODE>(p, s);
}

}  // namespace

hipError_t launch_qkv_proj(const void *x, const void *w, const int32_t *order, void *q, void *k,
                           void *v, int64_t B, int64_t N, int64_t heads, int64_t d,
                           hipStream_t s) {
  ProjArgs p;
  p.in = static_cast<const __bf16 *>(x);
  p.order = order;
  p.w = static_cast<const __bf16 *>(w);
  p.out0 = static_cast<__bf16 *>(q);
  p.out1 = static_cast<__bf16 *>(k);
  p.out2 = static_cast<__bf16 *>(v);
  p.T = (int32_t)(B * N);
  p.N = (int32_t)N;
  p.C = (int32_t)(heads * d);
  p.K = p.C;
  p.F = 3 * p.C;
  p.heads = (int32_t)heads;
  p.d = (int32_t)d;
  return launch_proj<0>(p, s);
}

hipError_t launch_out_proj(const void *o, const void *w, const int32_t *order, void *y, int64_t B,
                           int64_t N, int64_t heads, int64_t d, int64_t c_out, hipStream_t s) {
  ProjArgs p;
  p.in = static_cast<const __bf16 *>(o);
  p.order = order;
  p.w = static_cast<const __bf16 *>(w);
  p.out0 = static_cast<__bf16 *>(y);
  p.out1 = p.out2 = nullptr;
  p.T = (int32_t)(B * N);
  p.N = (int32_t)N;
  p.C = (int32_t)(heads * d);
  p.K = p.C;
  p.F = (int32_t)c_out;
  p.heads = (int32_t)heads;
  p.d = (int32_t)d;
  return launch_proj<1>(p, s);
}

}  // namespace hla
