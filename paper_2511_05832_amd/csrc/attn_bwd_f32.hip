// Block-sparse attention backward in fp32 throughout (fp32 I/O, fp32 products).
//
// Same computation and tile walk as the bf16 backward (gradients of the forward
// over the listed tiles only; P and dP recomputed from the forward's lse and the
// row statistics; no atomics), with every product on the fp32 matrix cores
// (v_mfma_f32_32x32x2_f32: exact fp32 multiply-adds). Both kernels are bound by
// them: a 32 x 32 block takes 3 D/2 (dq) or 4 D/2 (dk/dv) products of 64 cycles
// beside about 100 vector instructions. With one wave per SIMD nothing fills its
// waits: on the band below they are busy 40% (dq) and 51% (dk/dv) of the time. Measured against plain FMAs (band of
// half-width 128 on 64x64, d = 64, 8 heads): dq 163 -> 50 us, dk/dv 239 -> 52 us.
//
// Operands as in the fp32 forward: the walked rows are A operands from LDS (read
// by rows in 16-byte chunks for S and dP, lane half h contracting its half of d;
// read by columns for the products that contract over the walked index, lane m
// giving column m or columns 2m, 2m + 1), the fixed rows are B operands in
// registers, and S and dP come out in the operand layout of the products that
// follow. The walked tiles come in by the 16-byte LDS DMA, 64 rows at a time into
// a two-stage ring, their chunks XOR-swizzled by row so that both reads are free
// of bank conflicts. On partial tiles a wave skips a 32 x 32 block that holds no
// allowed pair.
//
// Rounding: S is summed in four chains of a quarter of d (as in the forward, see
// there), dP in two at d = 64 and one at d = 32: chains of 32 elements. With one
// chain for both, the gradients at d = 64 were up to 25% further from float64 than
// those of the vector-FMA kernels (49-token windows: dq 4.6e-7 against 3.7e-7; now
// about the same). Four chains for both as well spilled 50 registers in dk/dv.
// At d = 32 a second chain of dP takes dk/dv from 153 to 204 registers, three waves
// per SIMD to two, and one was already nearer (dq 3.5e-7 against 3.8e-7).
//
//   dq kernel    one workgroup per (b*h, query tile); wave w owns 32 queries and
//                walks the row list's key tiles; it also computes the rows'
//                statistics (lse * log2 e, -delta; delta = <dout, out>) and stores
//                them for the next kernel.
//   dkdv kernel  one workgroup of four waves per (b*h, key tile): waves 0, 1 take
//                the two 32-key blocks against the first 32 of each 64 query rows,
//                waves 2, 3 against the other 32, and the halves are added through
//                LDS at the end.
// Fused reordering (GATHER): every tensor in grid order, sequence position i in
// row order[i]; the 64 row indices of a step are copied to LDS a step before its
// rows.
#include "attn_common.h"

namespace hla {
namespace {

constexpr int BN = 64;   // keys per key tile, and rows per ring stage

// LDS offsets of this lane's reads of a 32-row block of a swizzled row tile.
template <int D>
struct Reads {
  static constexpr int ROW = D * 4;
  static constexpr int NDB = D / 32;
  int row[D / 8];   // by rows: chunk c of the lane's row, its half of d
  int colm[4];      // by columns: rows 8 half + r, r % 4 = index
  __device__ __forceinline__ void init(int col, int half) {
    const int r = row_perm(col);
#pragma unroll
    for (int c = 0; c < D / 8; ++c) row[c] = r * ROW + (((half * (D / 8) + c) ^ swz_f32(r)) * 16);
    const int e = col * NDB;   // first column
#pragma unroll
    for (int i = 0; i < 4; ++i)
      colm[i] = 8 * half * ROW + (((e >> 2) ^ (i | (half << 2))) * 16) + (e & 3) * 4;
  }
  // acc = rows . b over the lane's half of d
  template <int CHAINS>
  __device__ __forceinline__ void rows_times(const char *blk, const f32x4 (&b)[D / 8], f32x16 &acc) const {
    mfma_rows_f32<D / 8, CHAINS>(blk, row, b, acc);
  }
  // acc += columns . w
  __device__ __forceinline__ void cols_times(const char *blk, const f32x16 &w, f32x16 (&acc)[NDB]) const {
    mfma_cols_f32<NDB>([&](int t) { return blk + colm[t & 3] + (16 * (t >> 3) + (t & 7)) * ROW; }, w, acc);
  }
};

// Store accumulators (rows = columns of d, this lane's tensor row) scaled by mul
// to dst: slots 4g .. 4g + 3 of half h are columns 8g + 4h .. (d = 32) or, the
// two accumulators interleaved, 16g + 8h .. (d = 64).
template <int D>
__device__ __forceinline__ void store_row(const f32x16 (&acc)[D / 32], float mul, float *dst, int half) {
  constexpr int NDB = D / 32;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    float o[4 * NDB];
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int db = 0; db < NDB; ++db) o[NDB * e + db] = acc[db][4 * g + e] * mul;
#pragma unroll
    for (int x = 0; x < NDB; ++x)
      *reinterpret_cast<float4 *>(dst + NDB * (8 * g + 4 * half) + 4 * x) =
          make_float4(o[4 * x], o[4 * x + 1], o[4 * x + 2], o[4 * x + 3]);
  }
}

// The 64 row indices of sequence positions p0 .. p0 + 63 into an index slot, one
// per lane of the calling wave. Positions past the end read entry N - 1.
__device__ __forceinline__ void copy_idx(const AttnBwdArgs &a, int p0, int lane, const void *slot) {
  lds_dma4(a.order + min(p0 + lane, a.N - 1), lds_addr(slot));
}

// 64 rows of X and Y from sequence position p0 on into a stage (X tile, then Y
// tile), rows past the end of the sequence reading row N - 1. rows: their index
// slot (GATHER).
template <int D, int NW, bool GATHER>
__device__ __forceinline__ void copy_rows(const float *X, const float *Y, int p0, int N, char *base,
                                          const int32_t *rows, int wave, int lane) {
  constexpr int CPR = D / 4, CPW = BN * CPR / (64 * NW), TILE = BN * D * 4;
  static_assert(BN * CPR % (64 * NW) == 0, "copies must split evenly");
#pragma unroll
  for (int j = 0; j < CPW; ++j) {
    const int p = (j * NW + wave) * 64 + lane;
    const int r = p / CPR, c = (p % CPR) ^ swz_f32(r);
    const int64_t row = GATHER ? (int64_t)rows[r] : (int64_t)min(p0 + r, N - 1);
    lds_dma16(X + row * D + 4 * c, lds_addr(base + (j * NW + wave) * 1024));
    lds_dma16(Y + row * D + 4 * c, lds_addr(base + TILE + (j * NW + wave) * 1024));
  }
}

// KS = 2: two waves share 32 queries, one per 32-key block of every tile; their
// sums are added at the end through LDS (see the fp32 forward).
template <int D, int NW, int KS, bool GATHER>
__global__ void __launch_bounds__(64 * NW * KS, 2) attn_bwd_dq_f32(AttnBwdArgs a) {
  constexpr int BM = 32 * NW;
  constexpr int NWT = NW * KS;
  constexpr int TILE = BN * D * 4;
  constexpr int STAGE = 2 * TILE;   // K tile then V tile
  constexpr int NDB = D / 32;
  constexpr int IDXK = 2 * STAGE;   // GATHER: four slots of BN indices
  __shared__ __attribute__((aligned(16))) char lds[IDXK + (GATHER ? 4 * BN * 4 : 0)];
  auto idx_k = [&](int i) { return reinterpret_cast<const int32_t *>(lds + IDXK + (i & 3) * BN * 4); };

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wq = wave % NW, ks = wave / NW;   // query block, key block (KS = 2)
  const int col = lane & 31, half = lane >> 5;
  const int logical = xcd_remap(blockIdx.x, gridDim.x);
  const int bh = logical / a.n_qtiles;
  const int qt = logical - bh * a.n_qtiles;
  const int qpos = qt * BM + wq * 32 + col;
  const int64_t slice = (int64_t)bh * a.N * D;
  const float *K = static_cast<const float *>(a.k) + slice;
  const float *V = static_cast<const float *>(a.v) + slice;

  const PatternArgs &P = a.pat;
  const Region R = region_of<true>(P, qpos);
  const int nf = sload(a.n_full + qt), ntot = nf + sload(a.n_part + qt);
  const int32_t *frow = a.full_idx + (int64_t)qt * a.n_ktiles;
  const int32_t *prow = a.part_idx + (int64_t)qt * a.n_ktiles;
  auto tile_of = [&](int i) { return i < nf ? sload(frow + i) : sload(prow + i - nf); };

  // A query row past the end of the sequence (ragged last query tile) reads row
  // N - 1 and stores nothing.
  const int qc = min(qpos, a.N - 1);
  const int64_t qrow = GATHER ? (int64_t)a.order[qc] : (int64_t)qc;
  const int64_t lrow = slice + qrow * D + half * (D / 2);   // the lane's half row
  f32x4 q[D / 8], g[D / 8];
  float dpart = 0.f;
#pragma unroll
  for (int c = 0; c < D / 8; ++c) {
    q[c] = *reinterpret_cast<const f32x4 *>(static_cast<const float *>(a.q) + lrow + 4 * c);
    g[c] = *reinterpret_cast<const f32x4 *>(static_cast<const float *>(a.dout) + lrow + 4 * c);
    const f32x4 o = *reinterpret_cast<const f32x4 *>(static_cast<const float *>(a.out) + lrow + 4 * c);
#pragma unroll
    for (int e = 0; e < 4; ++e) dpart = __builtin_fmaf(o[e], g[c][e], dpart);
  }
  // This query's row statistics, computed here and stored for the dk/dv kernel:
  // (lse * log2 e, +inf for a row with no allowed key; -delta).
  const float lraw = a.lse[(int64_t)bh * a.N + qrow];
  const float lse2 = lraw == -__builtin_inff() ? __builtin_inff() : lraw * 1.4426950408889634f;
  const float ndelta = -(dpart + __shfl_xor(dpart, 32));
  if (half == 0 && ks == 0 && qpos < a.N)
    *reinterpret_cast<float2 *>(a.stats + 2 * ((int64_t)bh * a.N + qrow)) = make_float2(lse2, ndelta);

  Reads<D> rd;
  rd.init(col, half);
  f32x16 acc[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) acc[db] = f32x16{};

  auto block = [&](const char *stage, int kt, int kb, bool masked) {
    const int k0 = kt * BN + 32 * kb;
    if (masked && !__ballot(region_meets(R, P, k0, 32))) return;
    const char *kblk = stage + kb * 32 * D * 4;
    f32x16 s[1], dp;
    rd.template rows_times<4>(kblk, q, s[0]);
    rd.template rows_times<D / 32>(kblk + TILE, g, dp);
    if (masked) mask_blocks<1>(s, R, P, k0 + 8 * half);
#pragma unroll
    for (int v = 0; v < 16; ++v)
      s[0][v] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[0][v], a.scale_log2, -lse2)) * (dp[v] + ndelta);
    rd.cols_times(kblk, s[0], acc);
  };

  if constexpr (GATHER) {
    for (int i = 0; i < 2; ++i)
      if (i < ntot && wave == 0) copy_idx(a, tile_of(i) * BN, lane, idx_k(i));
  }
  // (one wait the compiler sees covers the register loads, so it adds none inside
  // the loop; the barrier publishes the index copies)
  wait_vmem_all();
  if constexpr (GATHER) wait_then_barrier<0>();
  if (ntot > 0) copy_rows<D, NWT, GATHER>(K, V, tile_of(0) * BN, a.N, lds, idx_k(0), wave, lane);
  for (int i = 0; i < ntot; ++i) {
    // tile i (and the indices of entry i + 1) have landed, and every wave is done
    // with tile i - 1's stage
    wait_then_barrier<0>();
    if (i + 1 < ntot)
      copy_rows<D, NWT, GATHER>(K, V, tile_of(i + 1) * BN, a.N, lds + ((i + 1) & 1) * STAGE, idx_k(i + 1),
                               wave, lane);
    if constexpr (GATHER)
      if (i + 2 < ntot && wave == 0) copy_idx(a, tile_of(i + 2) * BN, lane, idx_k(i + 2));
    const char *stage = lds + (i & 1) * STAGE;
    const int kt = tile_of(i);
#pragma unroll 1
    for (int kb = ks; kb < 2; kb += KS) block(stage, kt, kb, i >= nf);
  }
  if constexpr (KS == 2) {
    constexpr int PER = 16 * NDB * 64;
    static_assert(NW * PER * 4 <= 2 * STAGE, "the merge must fit the ring");
    float *ex = reinterpret_cast<float *>(lds) + wq * PER + lane;
    wait_then_barrier<0>();   // every wave is done with the ring
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (ks == 1) ex[(16 * db + v) * 64] = acc[db][v];
    wait_then_barrier<0>();
    if (ks == 1) return;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[db][v] += ex[(16 * db + v) * 64];
  }
  if (qpos < a.N) store_row<D>(acc, a.scale, static_cast<float *>(a.dq) + slice + qrow * D, half);
}

template <int D, int BMQ, bool GATHER>
__global__ void __launch_bounds__(256, 2) attn_bwd_dkdv_f32(AttnBwdArgs a) {
  constexpr int NW = 4;
  constexpr int SPT = BMQ / BN;          // ring steps per query tile
  constexpr int TILE = BN * D * 4;
  constexpr int STAT = 2 * TILE;         // lse2 of the 64 rows, then -delta
  constexpr int STAGE = 2 * TILE + 2 * BN * 4;   // Q tile, dout tile, statistics
  constexpr int NDB = D / 32;
  constexpr int IDXQ = 2 * STAGE;        // GATHER: four slots of BN indices
  __shared__ __attribute__((aligned(16))) char lds[IDXQ + (GATHER ? 4 * BN * 4 : 0)];
  static_assert(2 * 2 * NDB * 64 * 64 <= 2 * STAGE, "the halves' sums must fit the ring");
  auto idx_q = [&](int i) { return reinterpret_cast<const int32_t *>(lds + IDXQ + (i & 3) * BN * 4); };

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 31, half = lane >> 5;
  const int kb = wave & 1, qb = wave >> 1;   // this wave's key block and query half
  const int logical = xcd_remap(blockIdx.x, gridDim.x);
  const int bh = logical / a.n_ktiles;
  const int kt = logical - bh * a.n_ktiles;
  const int kpos = kt * BN + 32 * kb + col;
  const int64_t slice = (int64_t)bh * a.N * D;
  const float *Q = static_cast<const float *>(a.q) + slice;
  const float *G = static_cast<const float *>(a.dout) + slice;
  const float *S = a.stats + 2 * (int64_t)bh * a.N;

  const PatternArgs &P = a.pat;
  const Region R = region_of<false>(P, kpos);
  const int nf = SPT * sload(a.n_full_t + kt), ntot = nf + SPT * sload(a.n_part_t + kt);
  const int32_t *fcol = a.full_idx_t + (int64_t)kt * a.n_qtiles;
  const int32_t *pcol = a.part_idx_t + (int64_t)kt * a.n_qtiles;
  // first query position of step i
  auto pos_of = [&](int i) {
    const int t = i < nf ? sload(fcol + i / SPT) : sload(pcol + (i - nf) / SPT);
    return t * BMQ + (i % SPT) * BN;
  };
  // The next step from i on that holds an allowed pair (half of a partial
  // 128-row query tile may hold none). Lane l looks at key l of the tile, so
  // every wave finds the same step.
  const Region R64 = region_of<false>(P, kt * BN + lane);
  auto next = [&](int i) {
    if constexpr (SPT > 1)
      while (i >= nf && i < ntot && !__ballot(region_meets(R64, P, pos_of(i), BN))) ++i;
    return i;
  };
  // (n: how many steps ran before this one)
  auto issue = [&](int i, int n) {
    const int p0 = pos_of(i);
    char *stage = lds + (n & 1) * STAGE;
    copy_rows<D, NW, GATHER>(Q, G, p0, a.N, stage, idx_q(n), wave, lane);
    if (wave < 2) {   // wave 0: lse2 of the rows, wave 1: -delta
      const int64_t row = GATHER ? (int64_t)idx_q(n)[lane] : (int64_t)min(p0 + lane, a.N - 1);
      lds_dma4(S + 2 * row + wave, lds_addr(stage + STAT + wave * BN * 4));
    }
  };

  // A key row past the end of the sequence (ragged last key tile) reads row N - 1
  // and stores nothing; query rows past it read row N - 1 and are masked.
  const int kc = min(kpos, a.N - 1);
  const int64_t krow = GATHER ? (int64_t)a.order[kc] : (int64_t)kc;
  const int64_t lrow = slice + krow * D + half * (D / 2);
  f32x4 k[D / 8], v[D / 8];
#pragma unroll
  for (int c = 0; c < D / 8; ++c) {
    k[c] = *reinterpret_cast<const f32x4 *>(static_cast<const float *>(a.k) + lrow + 4 * c);
    v[c] = *reinterpret_cast<const f32x4 *>(static_cast<const float *>(a.v) + lrow + 4 * c);
  }
  Reads<D> rd;
  rd.init(col, half);
  f32x16 dk[NDB], dv[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) dk[db] = dv[db] = f32x16{};

  auto block = [&](const char *stage, int p0, bool masked) {
    const int q0 = p0 + 32 * qb;
    if (masked && !__ballot(region_meets(R, P, q0, 32))) return;
    const char *qblk = stage + qb * 32 * D * 4;
    const float *st = reinterpret_cast<const float *>(stage + STAT) + 32 * qb + 8 * half;
    f32x16 s[1], dp;
    rd.template rows_times<4>(qblk, k, s[0]);
    rd.template rows_times<D / 32>(qblk + TILE, v, dp);
    if (masked) mask_blocks<1>(s, R, P, q0 + 8 * half);
#pragma unroll
    for (int x = 0; x < 4; ++x) {   // slots 4x .. 4x + 3: rows 16 (x/2) + 4 (x%2) ..
      const f32x4 l4 = *reinterpret_cast<const f32x4 *>(st + 16 * (x >> 1) + 4 * (x & 1));
      const f32x4 d4 = *reinterpret_cast<const f32x4 *>(st + BN + 16 * (x >> 1) + 4 * (x & 1));
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[0][4 * x + e], a.scale_log2, -l4[e]));
        s[0][4 * x + e] = p;
        dp[4 * x + e] = p * (dp[4 * x + e] + d4[e]);
      }
    }
    rd.cols_times(qblk + TILE, s[0], dv);
    rd.cols_times(qblk, dp, dk);
  };

  // the step at hand, the next and the one after it
  int i0 = next(0), i1 = next(i0 + 1);
  if constexpr (GATHER) {
    if (wave == 0) {
      if (i0 < ntot) copy_idx(a, pos_of(i0), lane, idx_q(0));
      if (i1 < ntot) copy_idx(a, pos_of(i1), lane, idx_q(1));
    }
  }
  wait_vmem_all();
  if constexpr (GATHER) wait_then_barrier<0>();
  if (i0 < ntot) issue(i0, 0);
  for (int n = 0; i0 < ntot; ++n) {
    wait_then_barrier<0>();
    if (i1 < ntot) issue(i1, n + 1);
    const int i2 = next(i1 + 1);
    if constexpr (GATHER)
      if (i2 < ntot && wave == 0) copy_idx(a, pos_of(i2), lane, idx_q(n + 2));
    block(lds + (n & 1) * STAGE, pos_of(i0), i0 >= nf);
    i0 = i1;
    i1 = i2;
  }

  // Add the two query halves through LDS: waves 2, 3 hand over their dk and keep
  // dv, waves 0, 1 the other way round. Slot area of key block kb: dk, then dv.
  wait_then_barrier<0>();   // every wave is done with the ring
  float *ex = reinterpret_cast<float *>(lds) + kb * 2 * NDB * 16 * 64;
  float *give = ex + (qb ? 0 : NDB * 16 * 64), *take = ex + (qb ? NDB * 16 * 64 : 0);
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int x = 0; x < 16; ++x) give[(16 * db + x) * 64 + lane] = qb ? dk[db][x] : dv[db][x];
  wait_then_barrier<0>();
  if (kpos >= a.N) return;
  if (qb == 0) {
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int x = 0; x < 16; ++x) dk[db][x] += take[(16 * db + x) * 64 + lane];
    store_row<D>(dk, a.scale, static_cast<float *>(a.dk) + slice + krow * D, half);
  } else {
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int x = 0; x < 16; ++x) dv[db][x] += take[(16 * db + x) * 64 + lane];
    store_row<D>(dv, 1.f, static_cast<float *>(a.dv) + slice + krow * D, half);
  }
}

template <int D, int BM, bool GATHER>
hipError_t launch_all(const AttnBwdArgs &a, hipStream_t s) {
  // the dq kernel also writes the row statistics the dk/dv kernel reads
  const dim3 grid((uint32_t)((int64_t)a.BH * a.n_qtiles));
  // (four waves, as in the forward)
  hipLaunchKernelGGL((attn_bwd_dq_f32<D, BM / 32, 128 / BM, GATHER>), grid, dim3(256), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((attn_bwd_dkdv_f32<D, BM, GATHER>), dim3((uint32_t)((int64_t)a.BH * a.n_ktiles)),
                     dim3(256), 0, s, a);
  return hipGetLastError();
}

template <int D, int BM>
hipError_t launch_any(const AttnBwdArgs &a, hipStream_t s) {
  return a.order ? launch_all<D, BM, true>(a, s) : launch_all<D, BM, false>(a, s);
}

}  // namespace

hipError_t launch_attn_bwd_f32(const AttnBwdArgs &a, int d, int tile_m, int tile_n,
                               hipStream_t s) {
  if (tile_n != BN) return hipErrorInvalidValue;
  if (d == 32 && tile_m == 64) return launch_any<32, 64>(a, s);
  if (d == 32 && tile_m == 128) return launch_any<32, 128>(a, s);
  if (d == 64 && tile_m == 64) return launch_any<64, 64>(a, s);
  if (d == 64 && tile_m == 128) return launch_any<64, 128>(a, s);
  return hipErrorInvalidValue;
}

}  // namespace hla
