// Block-sparse attention forward in fp32 throughout (fp32 I/O, fp32 products).
//
// Same algorithm as the bf16 kernel (Sec. 3.1; Eq. 1: only the listed key
// tiles are visited, full tiles unmasked, partial tiles masked, online
// softmax), with the products on the fp32 matrix cores
// (v_mfma_f32_32x32x2_f32: exact fp32 multiply-adds, 157 TFLOP/s dense).
//
// What bounds it: the matrix cores. A wave owns 32 queries and takes a key tile
// in two blocks of 32 keys; a block is D/2 + D/2 products of 64 cycles (4096
// at d = 64) beside about 600 cycles of softmax. The operands come from LDS at
// one 16-byte read per four products (K) and one 8-byte read per two (V), far
// below the LDS rate. The softmax's vector work does not hide behind fp32 matrix
// products (measured: 16 FMAs beside 8 products, of any wave of the SIMD, add
// their whole issue time), so 80% of the matrix rate is about the limit. Measured
// against plain FMAs with four lanes per row, which read every K and V element
// from LDS once per 16 FMAs: band of half-width 128 on 64x64 at d = 64, 8 heads
// 128 -> 36 us, 32 heads 293 -> 111 us (113 TFLOP/s over the listed tiles).
// With one wave per SIMD (8 heads there: 256 workgroups) nothing fills its waits:
// the matrix cores are busy 36% of the time.
//
//   S^T = K Q^T     A = K rows from LDS, B = the wave's q in registers. Lane half
//                   h contracts d in [h D/2, (h+1) D/2), so a lane reads its part
//                   of a key row in 16-byte chunks.
//                   The sum runs in four chains of a quarter of d each: one chain
//                   rounds more (64- and 81-key rows at d = 64: 2.9e-7 and
//                   3.1e-7 off float64, four chains 2.0e-7 and 2.2e-7, the vector
//                   FMAs' quads 2.2e-7 and 2.4e-7) and saves 1% of the time.
//   O^T += V^T P^T  the accumulator slot v of lane half h is key
//                   16 (v/8) + 8 h + v%8 of the block (the K rows are fed
//                   permuted, row_perm): product t takes slot t as its B operand
//                   as it stands and V rows 16 (t/8) + 8 h + t%8 as A, lane m
//                   giving column m (d = 32) or columns 2m and 2m + 1 for two
//                   accumulators (d = 64).
//
// K and V tiles come in by the 16-byte LDS DMA, one tile ahead in a two-stage
// ring (64 KiB at d = 64: two workgroups per CU); K rows have their 16-byte
// chunks XOR-swizzled so that the row reads are free of bank conflicts, V rows
// are read whole. On partial tiles a wave skips a 32-key block in which none of
// its queries has an allowed key (it would contribute exact zeros).
//
// MODE ATTN_GATHER: the tensors are stored in grid order and sequence position i
// lives in row a.order[i] (reordering fused into the loads and stores); a tile's
// 64 row indices are copied to LDS one tile before its K/V copies. MODE ATTN_RPB:
// every score gets the global relative position bias of the grid cells order[i],
// order[j] (see the bf16 kernel); the indices come in the same way.
#include "attn_common.h"

namespace hla {
namespace {

constexpr int BN = 64;
constexpr float kRescaleSlack = 8.f;  // log2 units the softmax reference may lag the max

// NW waves of 32 queries, times KS: with KS = 2, two waves share 32 queries, one
// for each block of 32 keys of every tile, and their softmax states are merged at
// the end through LDS.
template <int D, int NW, int KS, int MODE>
__global__ void __launch_bounds__(64 * NW * KS, 2) attn_fwd_f32(AttnArgs a) {
  constexpr bool GATHER = MODE == ATTN_GATHER;
  constexpr bool RPB = MODE == ATTN_RPB;
  constexpr bool IDX = GATHER || RPB;
  constexpr int BM = 32 * NW;
  constexpr int NWT = NW * KS;        // waves of the workgroup
  constexpr int NT = 64 * NWT;
  constexpr int CPR = D / 4;          // 16-byte chunks per row
  constexpr int ROW = D * 4;          // bytes of a row
  constexpr int TILE = BN * ROW;
  constexpr int STAGE = 2 * TILE;     // K tile then V tile
  constexpr int CPW = BN * CPR / NT;  // 16-byte copies per thread per tile (K or V)
  constexpr int NDB = D / 32;         // accumulators of O^T
  constexpr int IDXK = 2 * STAGE;     // IDX: four slots of BN indices (slot i % 4: list entry i)
  constexpr int LDSB = IDXK + (IDX ? 4 * BN * 4 : 0);
  static_assert(BN * CPR % NT == 0, "copies must split evenly");
  __shared__ __attribute__((aligned(16))) char lds[LDSB];
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
  const float *Q = static_cast<const float *>(a.q) + slice;
  const float *K = static_cast<const float *>(a.k) + slice;
  const float *V = static_cast<const float *>(a.v) + slice;

  const PatternArgs &P = a.pat;
  const Region R = region_of<true>(P, qpos);
  const int nf = sload(a.n_full + qt), ntot = nf + sload(a.n_part + qt);
  const int32_t *frow = a.full_idx + (int64_t)qt * a.n_ktiles;
  const int32_t *prow = a.part_idx + (int64_t)qt * a.n_ktiles;
  auto tile_of = [&](int i) { return i < nf ? sload(frow + i) : sload(prow + i - nf); };

  // The row indices of list entry i into its slot (by the first wave). Positions
  // past the end of the sequence read entry N - 1.
  auto issue_idx = [&](int i) {
    if (wave == 0)
      lds_dma4(a.order + min(tile_of(i) * BN + lane, a.N - 1), lds_addr(lds + IDXK + (i & 3) * BN * 4));
  };
  // K and V rows of list entry i into a stage: LDS slot p of a tile holds row
  // p / CPR, chunk (p % CPR) ^ swizzle of K and chunk p % CPR of V. Key rows past
  // the end of the sequence read row N - 1 (such a tile is always partial and
  // every allowed region ends at N - 1).
  auto issue_tile = [&](int i, int stage) {
    char *base = lds + stage * STAGE;
    const int k0 = tile_of(i) * BN;
#pragma unroll
    for (int j = 0; j < CPW; ++j) {
      const int p = (j * NWT + wave) * 64 + lane;
      const int r = p / CPR, c = p % CPR;
      const int64_t row = GATHER ? (int64_t)idx_k(i)[r] : (int64_t)min(k0 + r, a.N - 1);
      lds_dma16(K + row * D + 4 * (c ^ swz_f32(r)), lds_addr(base + (j * NWT + wave) * 1024));
      lds_dma16(V + row * D + 4 * c, lds_addr(base + TILE + (j * NWT + wave) * 1024));
    }
  };

  // A query row past the end of the sequence (ragged last query tile) reads row
  // N - 1 and stores nothing.
  const bool live = qpos < a.N;
  const int qc = min(qpos, a.N - 1);
  const int64_t qrow = GATHER ? (int64_t)a.order[qc] : (int64_t)qc;
  f32x4 q[D / 8];
#pragma unroll
  for (int c = 0; c < D / 8; ++c)
    q[c] = *reinterpret_cast<const f32x4 *>(Q + qrow * D + half * (D / 2) + 4 * c);
  // scores are multiplied by smul to reach log2 units (RPB: already scaled)
  const float smul = RPB ? 1.44269504088896340736f : a.scale_log2;
  int32_t rpb_base = 0;
  const float *rpb_h = nullptr;
  if constexpr (RPB) {
    const int32_t g = a.order[qc];
    rpb_base = (P.H - 1) * (2 * P.W - 1) + (P.W - 1) + g + (P.W - 1) * (int32_t)fdiv((uint32_t)g, P.wdiv);
    rpb_h = a.rpb + (int64_t)(bh % a.heads) * (2 * P.H - 1) * (2 * P.W - 1);
  }

  // K operand chunk c of this lane's row, V operand column(s), within block 0
  int kaddr[D / 8];
#pragma unroll
  for (int c = 0; c < D / 8; ++c) {
    const int r = row_perm(col);
    kaddr[c] = r * ROW + (((half * (D / 8) + c) ^ swz_f32(r)) * 16);
  }
  const int vaddr = TILE + 8 * half * ROW + col * (4 * NDB);

  f32x16 oacc[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) oacc[db] = f32x16{};
  float m_run = -__builtin_inff();  // running reference, in units of log2
  float l_run = 0.f;                // this lane's partial sum (its half of the keys)

  // One block of 32 keys (block kb of the tile at sequence tile kt, list entry i).
  auto block = [&](const char *stage, int i, int kt, int kb, bool masked) {
    const int k0 = kt * BN + 32 * kb;
    if (masked && !__ballot(region_meets(R, P, k0, 32))) return;
    f32x16 s[1];
    const char *kb_base = stage + kb * 32 * ROW;
    mfma_rows_f32<D / 8, 4>(kb_base, kaddr, q, s[0]);
    if constexpr (RPB) {
      const int32_t *ids = idx_k(i) + 32 * kb + 8 * half;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int32_t gk = ids[16 * (v >> 3) + (v & 7)];
        const int32_t koff = gk + (P.W - 1) * (int32_t)fdiv((uint32_t)gk, P.wdiv);
        s[0][v] = __builtin_fmaf(s[0][v], a.scale, rpb_h[rpb_base - koff]);
      }
    }
    if (masked) mask_blocks<1>(s, R, P, k0 + 8 * half);
    float mx = s[0][0];
#pragma unroll
    for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s[0][v]);
    mx = fmaxf(mx, __shfl_xor(mx, 32)) * smul;
    // The reference moves only when the block's max passes it by the slack
    // (weights stay <= 2^8; O and l share the reference).
    const bool need = mx > m_run + kRescaleSlack;
    if (__ballot(need)) {
      const float m_new = need ? mx : m_run;
      const float alpha = need ? __builtin_amdgcn_exp2f(m_run - m_new) : 1.f;
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) oacc[db][v] *= alpha;
      m_run = m_new;
    }
    const float m_use = m_run == -__builtin_inff() ? 0.f : m_run;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      s[0][v] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[0][v], smul, -m_use));
      l_run += s[0][v];
    }
    const char *vb = kb_base + vaddr;
    mfma_cols_f32<NDB>([&](int t) { return vb + (16 * (t >> 3) + (t & 7)) * ROW; }, s[0], oacc);
  };

  // (one wait the compiler sees covers the register loads above, so it adds none
  // inside the loop; it also covers the index copies, which the barrier publishes)
  if constexpr (IDX) {
    for (int i = 0; i < 2; ++i)
      if (i < ntot) issue_idx(i);
  }
  wait_vmem_all();
  if constexpr (IDX) wait_then_barrier<0>();
  if (ntot > 0) issue_tile(0, 0);
  for (int i = 0; i < ntot; ++i) {
    // tile i (and the indices of entry i + 1) have landed, and every wave is done
    // with tile i - 1's stage
    wait_then_barrier<0>();
    if (i + 1 < ntot) issue_tile(i + 1, (i + 1) & 1);
    if constexpr (IDX)
      if (i + 2 < ntot) issue_idx(i + 2);
    const char *stage = lds + (i & 1) * STAGE;
    const int kt = tile_of(i);
#pragma unroll 1
    for (int kb = ks; kb < 2; kb += KS) block(stage, i, kt, kb, i >= nf);
  }

  l_run += __shfl_xor(l_run, 32);
  if constexpr (KS == 2) {
    // Merge the two key halves: waves ks = 1 hand over O, m and l.
    constexpr int PER = (16 * NDB + 2) * 64;   // floats per wave
    static_assert(NW * PER * 4 <= 2 * STAGE, "the merge must fit the ring");
    float *ex = reinterpret_cast<float *>(lds) + wq * PER + lane;
    wait_then_barrier<0>();   // every wave is done with the ring
    if (ks == 1) {
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) ex[(16 * db + v) * 64] = oacc[db][v];
      ex[16 * NDB * 64] = m_run;
      ex[(16 * NDB + 1) * 64] = l_run;
    }
    wait_then_barrier<0>();
    if (ks == 1) return;
    const float m1 = ex[16 * NDB * 64], m_new = fmaxf(m_run, m1);
    const float m_use = m_new == -__builtin_inff() ? 0.f : m_new;
    const float a0 = __builtin_amdgcn_exp2f(m_run - m_use), a1 = __builtin_amdgcn_exp2f(m1 - m_use);
    l_run = l_run * a0 + ex[(16 * NDB + 1) * 64] * a1;
    m_run = m_new;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int v = 0; v < 16; ++v) oacc[db][v] = oacc[db][v] * a0 + ex[(16 * db + v) * 64] * a1;
  }
  if (!live) return;
  // lane half h, slots 4g .. 4g + 3: columns 8g + 4h .. (d = 32), or, the two
  // accumulators interleaved, 16g + 8h .. (d = 64)
  const float inv = l_run > 0.f ? 1.f / l_run : 0.f;
  float *O = static_cast<float *>(a.out) + slice + qrow * D;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    float o[4 * NDB];
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int db = 0; db < NDB; ++db) o[NDB * e + db] = oacc[db][4 * g + e] * inv;
#pragma unroll
    for (int x = 0; x < NDB; ++x)
      *reinterpret_cast<float4 *>(O + NDB * (8 * g + 4 * half) + 4 * x) =
          make_float4(o[4 * x], o[4 * x + 1], o[4 * x + 2], o[4 * x + 3]);
  }
  if (a.lse && half == 0) {
    const float ln2 = 0.69314718055994530942f;
    a.lse[(int64_t)bh * a.N + qrow] =
        l_run > 0.f ? (m_run + __builtin_amdgcn_logf(l_run)) * ln2 : -__builtin_inff();
  }
}

template <int D, int NW>
hipError_t launch(const AttnArgs &a, hipStream_t s) {
  // four waves: at tile_m = 64 two of them share each 32 queries (d = 64 window,
  // 32 x 4096 rows: 94 -> 86 us; 8 x 4096 rows at d = 32, band: 29 -> 18 us); at
  // tile_m = 128 eight waves were slower or no faster (119 -> 131, 43 -> 43.5 us)
  constexpr int KS = 4 / NW;
  const dim3 grid((uint32_t)((int64_t)a.BH * a.n_qtiles)), wg(64 * NW * KS);
  if (a.mode == ATTN_GATHER)
    hipLaunchKernelGGL((attn_fwd_f32<D, NW, KS, ATTN_GATHER>), grid, wg, 0, s, a);
  else if (a.mode == ATTN_RPB)
    hipLaunchKernelGGL((attn_fwd_f32<D, NW, KS, ATTN_RPB>), grid, wg, 0, s, a);
  else
    hipLaunchKernelGGL((attn_fwd_f32<D, NW, KS, ATTN_PLAIN>), grid, wg, 0, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_f32(const AttnArgs &a, int d, int tile_m, int tile_n,
                           hipStream_t s) {
  if (tile_n != BN) return hipErrorInvalidValue;
  if (d == 32 && tile_m == 64) return launch<32, 2>(a, s);
  if (d == 32 && tile_m == 128) return launch<32, 4>(a, s);
  if (d == 64 && tile_m == 64) return launch<64, 2>(a, s);
  if (d == 64 && tile_m == 128) return launch<64, 4>(a, s);
  return hipErrorInvalidValue;
}

}  // namespace hla
