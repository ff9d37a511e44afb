// Fused attention forward for gfx950 (MI355X) with the softmax exponential
// either the hardware exp2 (control) or Rowmax-H15 (Sec. 5.2 Eq. (m-h15),
// App. B.1 "Implementation") and its finer input roundings S(Q_{2^-k})
// (App. B.2), or Rowmax-PoT (App. A.6), behind the C ABI declared in
// h15attn.h.
//
// Kernel structure (one workgroup = 4 wave64s for FP8, 8 or 4 for BF16, 32 query
// rows of one head per wave; or, where the grid leaves compute units idle, 8
// waves for 128 rows; two waves per SIMD, three for FP8 at d = 64):
//   * each wave keeps its 32 query rows of Q in VGPRs as the MFMA B operand,
//     brought in through LDS with whole-row loads;
//   * key tiles of 128 keys are copied HBM -> LDS with buffer loads that
//     write LDS directly (no staging registers), double-buffered (the copy
//     of tile t+1 is in flight while tile t is computed, one barrier per
//     tile) or single-buffered (K(t+1) copied while the weights and PV of
//     tile t run, V(t+1) while QK^T of tile t+1 runs, two barriers per tile:
//     the lattice weights at FP8 d = 128, and the compact BF16 layout);
//   * in the paired layout the even and the odd tiles of a block of rows go
//     to two halves of the workgroup, each single-buffered on its own, one
//     barrier apart; the two waves of a row exchange tile maxima, so that every
//     tile's anchor is the running maximum in tile order, and add up their
//     sums at the end;
//   * scores are computed transposed, S^T = K Q^T, with 32x32 MFMAs (bf16
//     32x32x16, fp8 32x32x64): each lane owns one query row and 64 of the
//     tile's 128 keys, so the row max and row sum are in-lane reductions plus
//     one exchange with lane ^ 32;
//   * the weights are produced in VALU registers (hardware exp2, or the
//     lattice weights finished two at a time in 16-bit lanes), converted to
//     the MFMA operand type and used directly as the B operand of
//     O^T += V^T P^T: the MFMA contraction index is mapped to keys so that
//     the S accumulator layout already is the P operand layout;
//   * V is read from LDS with the transposing reads ds_read_b64_tr_b16 (bf16)
//     and ds_read_b64_tr_b8 (fp8), in the matching key order;
//   * at fp8 the PV MFMAs over the tile's first 64 keys go first, and the
//     weights of the other 64 are finished between them (split P), so that
//     a wave's VALU work overlaps its own matrix-core work;
//   * O leaves through LDS, so that each store covers whole rows.
#include "attn_device.h"

// The file is compiled twice (build.py): with H15_FP8_LATTICE_D128 = 1 it
// holds only the forward kernels of the FP8 lattice weights at d = 128 and
// their launcher, built with the iterative ILP machine scheduler (measured at
// FP8 8K: +1.2% causal, +1.4% non-causal; the exact control and the BF16 and
// d = 64 kernels are better off with the default scheduler, which at d = 64
// keeps three waves per SIMD); with 0, the default, everything else.
#ifndef H15_FP8_LATTICE_D128
#define H15_FP8_LATTICE_D128 0
#endif

namespace h15 {
hipError_t launch_fwd_fp8_lattice128(const Params& p, bool causal, int mode, hipStream_t st, bool probe);
}

namespace {

using namespace h15;

constexpr int MAX_THREADS = 8 * 64;
// LDS operand prefetch distance (in MFMAs) of the QK^T and PV products
constexpr int QK_AHEAD = 3;
constexpr int PV_AHEAD = 3;
// instruction classes of __builtin_amdgcn_sched_group_barrier
constexpr int SG_MFMA = 0x008;
constexpr int SG_DS_READ = 0x100;
constexpr int POT_KMAX = 20;  // tail clamp of Rowmax-PoT

__device__ __forceinline__ void map_block(const Params& p, int L, int& qb, int& b, int& h) {
  const int nbh = p.B * p.Hq;
  if (p.remap) {
    // Hardware workgroup ids go round-robin over the 8 XCDs (id mod 8).  Give
    // each XCD whole key/value-head groups, so the query heads that read the
    // same K/V share one L2, and walk query blocks longest-first.
    const int x = L & 7, j = L >> 3;
    int qi, kvl, gi;
    if (p.remap == 2) {
      // one KV head group at a time per XCD: the K/V working set of the
      // workgroups resident on an XCD is one head's (non-causal, where every
      // query block reads all of it)
      const int span = p.nqb * p.G;
      kvl = j / span;
      const int r = j - kvl * span;
      qi = r / p.G;
      gi = r - qi * p.G;
    } else {
      const int per = nbh >> 3;
      qi = j / per;
      const int loc = j - qi * per;
      kvl = loc / p.G;
      gi = loc - kvl * p.G;
    }
    qb = p.nqb - 1 - qi;
    const int kvg = kvl * 8 + x;
    b = kvg / p.Hkv;
    h = (kvg - b * p.Hkv) * p.G + gi;
  } else {
    const int qi = L / nbh, bh = L - qi * nbh;
    qb = p.nqb - 1 - qi;
    b = bh / p.Hq;
    h = bh - b * p.Hq;
  }
}

// init plus the row sum of a tile's packed weights: one dot product with
// (1, 1) per word, in two chains.
__device__ __forceinline__ float pair_sum(const uint32_t (&w)[4][8], float init) {
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
  float a[2] = {init, 0.0f};
#pragma unroll
  for (int kb = 0; kb < 4; ++kb)
#pragma unroll
    for (int q = 0; q < 8; ++q)
      a[q & 1] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w[kb][q]), ones, a[q & 1], false);
  return a[0] + a[1];
}

// Rowmax-PoT weight of one score (App. A.6 Eq. (rowmax-pot)) against the
// whole-row maximum m: base-two gap x = fp32(fp32(m - s) c1), d = min(K_max,
// floor(x + 1/2)) (exact: x + 1/2 is representable below 2^22), w = 2^-d.
__device__ __forceinline__ float pot_weight(float s, float m, float c1) {
  const float x = (m - s) * c1;
  const float d = __builtin_fminf(__builtin_floorf(x + 0.5f), (float)POT_KMAX);
  return __builtin_amdgcn_ldexpf(1.0f, -(int)d);
}

// y over the scores of a tile whose key offset lies beyond lim
template <int E = 0>
__device__ __forceinline__ void mask_beyond(f32x16 (&v)[4], int lim, float y) {
  if constexpr (E < 64) {
    constexpr int kb = E / 16, j = E % 16;
    v[kb][j] = select_beyond<kb * 32 + 8 * (j >> 2) + (j & 3)>(lim, v[kb][j], y);
    mask_beyond<E + 1>(v, lim, y);
  }
}

// The scores of a tile are next read by inline asm (the v_max3_f32 tree of
// tile_max, and the compare/select of the masking), and the compiler inserts
// no wait states between a matrix-core write and an inline-asm read.  This
// statement does: it takes the four score blocks as in/out operands, so it
// comes after the last QK^T MFMA and every later read of the blocks comes
// after it, and it holds the wave for 24 wait states, more than the 20 that
// gfx950 requires between a 16-pass XDL write of a VGPR and a VALU read of
// it (the shorter MFMAs need fewer).  (Reading a block right after its MFMA,
// with no such wait, was measured to return stale values.)
__device__ __forceinline__ void settle_scores(f32x16 (&v)[4]) {
  asm("s_nop 15\n\ts_nop 7" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]));
}

// Tree reductions over a lane's 64 scores (short dependency chains); the
// reads of the scores come after settle_scores.
__device__ __forceinline__ float tile_max(const f32x16 (&v)[4]) {
  // 64 -> 22 -> 8 -> 3 -> 1
  float a[22], b[8], c[3];
#pragma unroll
  for (int i = 0; i < 21; ++i) {
    const int e0 = 3 * i, e1 = 3 * i + 1, e2 = 3 * i + 2;
    a[i] = max3(v[e0 >> 4][e0 & 15], v[e1 >> 4][e1 & 15], v[e2 >> 4][e2 & 15]);
  }
  a[21] = v[3][15];
#pragma unroll
  for (int i = 0; i < 7; ++i) b[i] = max3(a[3 * i], a[3 * i + 1], a[3 * i + 2]);
  b[7] = a[21];
  c[0] = max3(b[0], b[1], b[2]);
  c[1] = max3(b[3], b[4], b[5]);
  c[2] = max3(b[6], b[7], b[7]);
  return max3(c[0], c[1], c[2]);
}
__device__ __forceinline__ float tile_sum(const f32x16 (&v)[4]) {
  float a[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) a[i] = (v[0][i] + v[1][i]) + (v[2][i] + v[3][i]);
#pragma unroll
  for (int w = 8; w >= 1; w >>= 1)
#pragma unroll
    for (int i = 0; i < w; ++i) a[i] = a[i] + a[i + w];
  return a[0];
}

template <int DT, int D, bool CAUSAL, int MODE, bool PROBE, int LAY>
__device__ __forceinline__ void fwd_body(const Params& p) {
  using C = Cfg<DT, D, LAY>;
  constexpr int NW = C::NW, BR = C::BR, RW = C::RW;
  constexpr bool PAIR = LAY == LAY_PAIRED;
  // K and V tiles, each double-buffered, or single-buffered: compact d = 128,
  // and the lattice weights at FP8 d = 128 (measured at causal and
  // non-causal 8K: H15 +1.7..2.4% single-buffered, the exact control
  // -0.7%, so the control keeps two buffers)
  constexpr int NSTAGE = (LAY == LAY_WIDE && DT == DT_FP8 && D == 128 && mode_lattice(MODE)) ? 1 : C::NSTAGE;
  static_assert(MODE != MODE_ROWMAX_POT || (NSTAGE == 2 && !PAIR), "the Rowmax-PoT first pass double-buffers K");
  // Paired: one K and one V tile for each half of the waves; at the end they
  // take the fp32 halves of O that the pairs exchange, then the bf16 rows,
  // which have their own array where they do not fit behind.
  constexpr int NOB = D / 32 / C::NPAR;  // 32-column blocks of O that a wave writes
  constexpr int OX = NW * NOB * 4096 / 2, OST = NW * WROWS * NOB * 64;
  constexpr bool OWN_OST = PAIR && 2 * C::TILE < OX + OST;
  __shared__ __attribute__((aligned(16))) uint8_t smem[PAIR ? 2 * C::TILE : NSTAGE * C::BUF];
  __shared__ __attribute__((aligned(16))) uint8_t vsm[PAIR ? 2 * C::TILE : 16];
  __shared__ __attribute__((aligned(16))) uint8_t osm[OWN_OST ? OST : 16];
  static_assert(!PAIR || 2 * C::TILE >= OX, "O exchange fits the tiles");
  static_assert(PAIR || NSTAGE * C::BUF >= OST, "O staging fits the tiles");
  // paired: each row's maximum in the last even and odd tile; at the end the
  // waves' anchors and row sums
  __shared__ float mx_lds[2][2][PAIR ? BR : 1];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int i32 = lane & 31;
  const int g = lane >> 5;
  const int G4 = lane >> 4, L16 = lane & 15;

  int qb, b, h;
  map_block(p, blockIdx.x, qb, b, h);
  const int S = p.S;
  const int hk = h / p.G;
  const int q0 = qb * BR;
  // row wave; paired: parity of this wave's tiles
  const int rw = __builtin_amdgcn_readfirstlane(wave % RW);
  const int par = PAIR ? __builtin_amdgcn_readfirstlane(wave / RW) : 0;
  uint8_t* const ktile = smem + par * C::TILE;  // (single-buffered)
  uint8_t* const vtile = PAIR ? vsm + par * C::TILE : smem + C::TILE;
  const int qw0 = q0 + rw * WROWS;
  const int qrow = qw0 + i32;
  const bool wave_live = qw0 < S;
  const int last_key = CAUSAL ? min(q0 + BR - 1, S - 1) : S - 1;
  const int ntiles = last_key / BC + 1;
  const float off = DT == DT_FP8 ? 8.0f : 0.0f;

  const size_t kv_head = (size_t)(b * p.Hkv + hk) * (size_t)S;
  const uint8_t* kg = p.k + kv_head * C::RB;
  const uint8_t* vg = p.v + kv_head * C::RB;
  const size_t q_head = (size_t)(b * p.Hq + h) * (size_t)S;

  // ---- Q block in registers (MFMA B operand: lane holds row i32, k-half g);
  // loaded through LDS below (stage_q, read_q)
  constexpr int NKQ = DT == DT_BF16 ? D / 16 : D / 64;
  bf16x8 qb16[DT == DT_BF16 ? NKQ : 1];
  i32x8 qf8[DT == DT_FP8 ? NKQ : 1];

  // ---- staging: every wave copies WAVE_LOADS x 1 KB of a K or V tile
  // straight into LDS.  LDS slot s (16 bytes) of a tile holds row s / NCH,
  // chunk (s % NCH) ^ swizzle(row).  Buffer (not global) loads are used so
  // that the compiler's wait counting keeps LDS reads pipelined while these
  // copies are in flight.  One head's rows span S * RB < 2^31 bytes.  Tile t
  // uses K buffer t % 2 and V buffer t % 2.
  const __amdgpu_buffer_rsrc_t krsrc = __builtin_amdgcn_make_buffer_rsrc((void*)kg, (short)0, S * C::RB, BUF_DWORD3);
  const __amdgpu_buffer_rsrc_t vrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)vg, (short)0, S * C::RB, BUF_DWORD3);
  auto kbuf = [&](int t) { return smem + (t & 1) * C::BUF; };
  // Each of the waves that share a tile copies its WAVE_LOADS 1 KB blocks.  The lane's byte
  // offset inside the tile is the same for every tile, so it is computed
  // once; a tile then adds only the scalar offset of its first row.  Rows at
  // or beyond S (the ragged last tile) lie outside the resource's
  // num_records = S * RB: the hardware range check reads them as zero without
  // touching memory, and those keys are masked.  The check compares the
  // lane's offset with num_records minus the scalar offset, so the scalar one
  // must not pass num_records (the difference would wrap): it is held there,
  // where every lane is out of range.  The wave index is scalar, so the LDS
  // destinations (M0) are too.
  // (The addresses handed to the LDS-copy builtin are named variables: with
  // an arithmetic expression in those arguments the host side of this
  // compiler drops the kernels' launch stubs without a diagnostic.)
  constexpr int WAVE_LOADS = C::CHUNKS / (RW * 64);
  const uint32_t head_bytes = (uint32_t)S * C::RB;
  const int wave_s = __builtin_amdgcn_readfirstlane(rw);
  // Paired: the chunk swizzles repeat every 16 rows, and the 1 KB blocks
  // advance by a multiple of that, so one lane offset serves all loads and the
  // scalar offset moves; there the registers are short.  (In the other layouts
  // the scalar instructions for that cost 0.5..1%.)
  constexpr int LANE_OFFS = PAIR ? 1 : WAVE_LOADS;
  static_assert(!PAIR || RW * 64 / C::NCH % 16 == 0, "the swizzle repeats from load to load");
  uint32_t koff[LANE_OFFS], voff[LANE_OFFS];
#pragma unroll
  for (int c = 0; c < LANE_OFFS; ++c) {
    const int slot = (c * RW + rw) * 64 + lane;
    const int row = slot / C::NCH, pch = slot % C::NCH;
    koff[c] = (uint32_t)(row * C::RB + ((pch ^ k_swz<DT, D>(row)) << 4));
    voff[c] = (uint32_t)(row * C::RB + ((pch ^ v_swz<DT, D>(row)) << 4));
  }
  auto stage = [&](int t, uint8_t* dst, const __amdgpu_buffer_rsrc_t& rsrc,
                   const uint32_t (&off)[LANE_OFFS]) __attribute__((always_inline)) {
    // Paired: a tile beyond the last is out of the resource's range, so the
    // copies are the same in every step and no branch hides them from the
    // compiler's wait counting (with one, each first read of K waited for the
    // copies of V)
    const uint32_t soff = PAIR && t >= ntiles ? head_bytes : (uint32_t)(t * BC) * C::RB;
#pragma unroll
    for (int c = 0; c < WAVE_LOADS; ++c) {
      const uint32_t so = PAIR ? min(soff + c * RW * 1024, head_bytes) : soff;
      const uint32_t vo = off[PAIR ? 0 : c];
      uint8_t* ldst = dst + (c * RW + wave_s) * 1024;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, LDS_PTR(void, ldst), 16, vo, so, 0, 0);
    }
  };

  // ---- Q through LDS: each wave copies its own 32 rows with the same
  // direct loads (16 contiguous bytes per lane, so each load covers whole
  // rows; rows at or beyond S read as zero), into a region the first K/V
  // copies do not touch (the V buffer when single-buffered, else the second
  // buffer), chunks swizzled as K's so that the operand reads, one chunk of
  // 32 rows per instruction like K's, spread over the banks.  Every wave
  // reads its operands before any wave copies into that region again (a
  // barrier after read_q).
  constexpr int QBYTES = WROWS * C::RB;
  constexpr int QREGION = NSTAGE == 1 ? C::TILE : C::BUF;
  static_assert(QBYTES % 2048 == 0, "Q staging layout");
  static_assert(PAIR ? RW * QBYTES <= (OWN_OST ? OST : 2 * C::TILE) : QREGION + RW * QBYTES <= NSTAGE * C::BUF,
                "Q staging layout");
  const __amdgpu_buffer_rsrc_t qrsrc =
      __builtin_amdgcn_make_buffer_rsrc((void*)(p.q + q_head * C::RB), (short)0, S * C::RB, BUF_DWORD3);
  uint8_t* const qreg = (OWN_OST ? osm : PAIR ? vsm : smem + QREGION) + wave_s * QBYTES;
  auto stage_q = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int c0 = 0; c0 < QBYTES / 1024; c0 += C::NPAR) {
      const int c = c0 + par;  // (paired: each of the two waves copies one half)
      const int slot = c * 64 + lane;
      const int row = slot / C::NCH, pch = slot % C::NCH;
      // (unsigned: rows past S may take the offset past 2^31, where the
      // range check still reads zero)
      const uint32_t voff = (uint32_t)(qw0 + row) * (uint32_t)C::RB + (uint32_t)((pch ^ k_swz<DT, D>(row)) << 4);
      uint8_t* ldst = qreg + c * 1024;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(qrsrc, LDS_PTR(void, ldst), 16, voff, 0, 0, 0);
    }
  };
  auto read_q = [&]() __attribute__((always_inline)) {
    const uint8_t* const qrow_l = qreg + i32 * C::RB;
    const int qswz = k_swz<DT, D>(i32);
    if constexpr (DT == DT_BF16) {
#pragma unroll
      for (int kk = 0; kk < NKQ; ++kk) qb16[kk] = *(const bf16x8*)(qrow_l + (((2 * kk + g) ^ qswz) << 4));
    } else {
#pragma unroll
      for (int kk = 0; kk < NKQ; ++kk) {
        const i32x4 lo = *(const i32x4*)(qrow_l + (((4 * kk + 2 * g) ^ qswz) << 4));
        const i32x4 hi = *(const i32x4*)(qrow_l + (((4 * kk + 2 * g + 1) ^ qswz) << 4));
        qf8[kk] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      }
    }
  };

  // ---- running state (this lane's query row; lanes i and i^32 agree on m)
  constexpr int NDB = D / 32;  // 32-column blocks of O^T
  f32x16 oacc[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) oacc[db] = f32x16{0.0f};
  float m_run = -INFINITY;
  float m_tile = -INFINITY;  // paired: the row's maximum in the open tile
  float l_part = 0.0f;  // this lane's share of the row sum
  // scores, then weights, of the current tile; accumulator value j of block
  // kb holds key 32 kb + 8 (j/4) + 4 g + j%4 of the tile
  f32x16 sacc[4];
  // P of the current tile in the operand type (the MFMA B operand of PV)
  bf16x8 pb[DT == DT_BF16 ? 8 : 1];
  i32x8 pf[DT == DT_FP8 ? 2 : 1];
  // lattice modes: the weights as BF16 pairs, word q of block kb holding keys
  // 2q and 2q + 1 of sacc[kb]
  uint32_t wpk[4][8];
  // FP8 finishes the second half of the tile's P (keys 64..127)
  // between the PV MFMAs of the first half (MFMA i covers block db = i % NDB
  // of O^T and key half i / NDB), which do not depend on it, so
  // that the wave's own VALU work runs while its matrix core is busy; the
  // row sum's partial sums then stay open across the PV product (exact
  // mode: the two halves in lch; lattice modes: eight dot2 chains in lch8,
  // one per word index, none longer than four)
  constexpr bool SPLIT = DT == DT_FP8 && MODE != MODE_ROWMAX_POT;
  constexpr bool PACKED = mode_lattice(MODE);
  float lch[2];
  float lch8[8];
  float nb1_split = 0.0f;  // exact mode: the exponent bias of the open tile

  // ---- S^T = K Q^T for the 128 keys of a tile (4 blocks of 32 keys).
  // MFMA i covers (kk = i / 4, kb = i % 4).  Its K operand is read from LDS
  // QK_AHEAD MFMAs in advance into a ring of registers, and the schedule keeps
  // that order, so each MFMA finds its operand loaded.
  auto qk = [&](const uint8_t* kl) __attribute__((always_inline)) {
    const int krow_off = i32 * C::RB;
    const int kswz = k_swz<DT, D>(i32);  // == k_swz(kb * 32 + i32)
    constexpr int NQK = 4 * NKQ;
    if constexpr (DT == DT_BF16) {
      auto ldk = [&](int i) {
        const uint8_t* rowp = kl + (i & 3) * 32 * C::RB + krow_off;
        return *(const bf16x8*)(rowp + (((2 * (i >> 2) + g) ^ kswz) << 4));
      };
      bf16x8 ring[QK_AHEAD + 1];
#pragma unroll
      for (int i = 0; i < QK_AHEAD; ++i) ring[i] = ldk(i);
      __builtin_amdgcn_sched_barrier(0);  // the prologue reads go first
#pragma unroll
      for (int i = 0; i < NQK; ++i) {
        const int kk = i >> 2, kb = i & 3;
        sacc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[i % (QK_AHEAD + 1)], qb16[kk],
                                                           kk == 0 ? f32x16{0.0f} : sacc[kb], 0, 0, 0);
        if (i + QK_AHEAD < NQK) ring[(i + QK_AHEAD) % (QK_AHEAD + 1)] = ldk(i + QK_AHEAD);
      }
#pragma unroll
      for (int i = 0; i < NQK; ++i) {
        __builtin_amdgcn_sched_group_barrier(SG_MFMA, 1, 0);
        if (i + QK_AHEAD < NQK) __builtin_amdgcn_sched_group_barrier(SG_DS_READ, 1, 0);
      }
    } else {
      auto ldk = [&](int i) {
        const int kk = i >> 2;
        const uint8_t* rowp = kl + (i & 3) * 32 * C::RB + krow_off;
        const i32x4 lo = *(const i32x4*)(rowp + (((4 * kk + 2 * g) ^ kswz) << 4));
        const i32x4 hi = *(const i32x4*)(rowp + (((4 * kk + 2 * g + 1) ^ kswz) << 4));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      };
      i32x8 ring[QK_AHEAD + 1];
#pragma unroll
      for (int i = 0; i < QK_AHEAD; ++i) ring[i] = ldk(i);
      __builtin_amdgcn_sched_barrier(0);  // the prologue reads go first
#pragma unroll
      for (int i = 0; i < NQK; ++i) {
        const int kk = i >> 2, kb = i & 3;
        sacc[kb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
            ring[i % (QK_AHEAD + 1)], qf8[kk], kk == 0 ? f32x16{0.0f} : sacc[kb], 0, 0, 0, 0, 0, 0);
        if (i + QK_AHEAD < NQK) ring[(i + QK_AHEAD) % (QK_AHEAD + 1)] = ldk(i + QK_AHEAD);
      }
#pragma unroll
      for (int i = 0; i < NQK; ++i) {
        __builtin_amdgcn_sched_group_barrier(SG_MFMA, 1, 0);
        if (i + QK_AHEAD < NQK) __builtin_amdgcn_sched_group_barrier(SG_DS_READ, 2, 0);
      }
    }
  };

  // ---- O^T += V^T P^T for the tile whose V sits at vl and whose P is in
  // pb/pf.  The V^T operands are read from LDS PV_AHEAD MFMAs ahead into a
  // ring of registers: pv_begin(vl) sets the lane's addresses and issues the
  // first PV_AHEAD reads (early, so that their latency hides behind the
  // softmax), pv_finish() issues the MFMAs and the remaining reads.  No
  // other LDS access may come between the two (the waits count reads).
  //
  // bf16: lane (d = i32 + 32 db, half g) needs keys 16 ks + 8 (r/4) + 4 g +
  // r%4 (r = 0..7): two 4-key transposing reads; lane L16 of a 16-lane group
  // addresses row 4 g + L16/4 (+8), columns 16 (G4%2) + 4 (L16%4) .. +3 of
  // the 32-column block.  MFMA i covers (db = i / 8, ks = i % 8).
  // fp8: lane (d = i32 + 32 db, half g) needs, for byte r = 8 rd + e, key
  // 32 (2 t2 + rd/2) + 16 (rd%2) + 8 (e/4) + 4 g + e%4: four 8-key
  // transposing reads; lane L16 of a 16-lane group addresses row vrow = base
  // + 8 (L16/8) + (L16/2)%4, columns d0 + 8 (L16%2) .. +7.  MFMA i covers
  // (db = i / 2, t2 = i % 2).
  // In both, the swizzle of the rows a lane reads equals that of vrow, so
  // only the block db moves the lane's address; the key offset is an
  // immediate.
  constexpr int NPV = DT == DT_BF16 ? NDB * 8 : NDB * 2;
  using VOp = std::conditional_t<DT == DT_BF16, bf16x8, i32x8>;
  VOp vring[PV_AHEAD + 1];
  uint32_t vbase[NDB];
  auto ldv = [&](auto ic) -> VOp {
    constexpr int i = decltype(ic)::value;
    if constexpr (DT == DT_BF16) {
      const i32x2v lo = ds_read_tr16<(16 * (i & 7)) * C::RB>(vbase[i >> 3]);
      const i32x2v hi = ds_read_tr16<(16 * (i & 7) + 8) * C::RB>(vbase[i >> 3]);
      return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3));
    } else {
      constexpr int t2 = SPLIT ? i / NDB : i & 1;
      const uint32_t a = vbase[SPLIT ? i % NDB : i >> 1];
      const i32x2v p0 = ds_read_tr8<(64 * t2) * C::RB>(a);
      const i32x2v p1 = ds_read_tr8<(64 * t2 + 16) * C::RB>(a);
      const i32x2v p2 = ds_read_tr8<(64 * t2 + 32) * C::RB>(a);
      const i32x2v p3 = ds_read_tr8<(64 * t2 + 48) * C::RB>(a);
      const i32x4 lo = __builtin_shufflevector(p0, p1, 0, 1, 2, 3);
      const i32x4 hi = __builtin_shufflevector(p2, p3, 0, 1, 2, 3);
      return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
  };
  auto pv_begin = [&](const uint8_t* vl) __attribute__((always_inline)) {
    const uint32_t vla = (uint32_t)(size_t)LDS_PTR(const uint8_t, vl);
    if constexpr (DT == DT_BF16) {
      const int vrow = 4 * (G4 >> 1) + (L16 >> 2);
      const int vcolb = (16 * (G4 & 1) + 4 * (L16 & 3)) * 2;
#pragma unroll
      for (int db = 0; db < NDB; ++db) {
        const int cb = 64 * db + vcolb;
        vbase[db] = vla + vrow * C::RB + (((cb >> 4) ^ v_swz<DT, D>(vrow)) << 4) + (cb & 15);
      }
    } else {
      const int vrow = 4 * (G4 >> 1) + 8 * (L16 >> 3) + ((L16 >> 1) & 3);
      const int vcol = 16 * (G4 & 1) + 8 * (L16 & 1);
#pragma unroll
      for (int db = 0; db < NDB; ++db) {
        const int cb = 32 * db + vcol;
        vbase[db] = vla + vrow * C::RB + (((cb >> 4) ^ v_swz<DT, D>(vrow)) << 4) + (cb & 15);
      }
    }
    static_for<0, PV_AHEAD>([&](auto ic) { vring[decltype(ic)::value] = ldv(ic); });
  };
  // ---- split P (FP8 lattice modes): part c (0..3) of the second half packs
  // words 4 (c % 2) .. +3 of block 2 + c / 2, converts them to P words 2c and
  // 2c + 1 of pf[1] and adds them to the row sum's chains
  auto finish_half = [&](auto cc) __attribute__((always_inline)) {
    if constexpr (SPLIT && !mode_lattice(MODE)) {
      // exact mode: part c takes values 8 (c % 2) .. +7 of block 2 + c / 2
      // through exp2, into P words 2c and 2c + 1, and sums them
      constexpr int c = decltype(cc)::value;
      constexpr int kb = 2 + (c >> 1), j0 = 8 * (c & 1);
#pragma unroll
      for (int j = j0; j < j0 + 8; ++j)
        sacc[kb][j] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[kb][j], p.c1, nb1_split));
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        const int jw = j0 + 4 * w;
        uint32_t word = __float_as_uint(sacc[kb][jw]);
        word = __builtin_amdgcn_cvt_pk_fp8_f32(sacc[kb][jw], sacc[kb][jw + 1], word, false);
        word = __builtin_amdgcn_cvt_pk_fp8_f32(sacc[kb][jw + 2], sacc[kb][jw + 3], word, true);
        pf[1][2 * c + w] = (int)word;
      }
      const float s8 = ((sacc[kb][j0] + sacc[kb][j0 + 1]) + (sacc[kb][j0 + 2] + sacc[kb][j0 + 3])) +
                       ((sacc[kb][j0 + 4] + sacc[kb][j0 + 5]) + (sacc[kb][j0 + 6] + sacc[kb][j0 + 7]));
      if constexpr ((c & 1) == 0) lch[c >> 1] = s8;
      else lch[c >> 1] += s8;
      if constexpr (c == 3) l_part += lch[0] + lch[1];
    } else if constexpr (SPLIT) {
      constexpr int c = decltype(cc)::value;
      constexpr int kb = 2 + (c >> 1), q0 = 4 * (c & 1);
#pragma unroll
      for (int q = q0; q < q0 + 4; ++q)
        wpk[kb][q] = sq_pack<MODE>(__float_as_uint(sacc[kb][2 * q]), __float_as_uint(sacc[kb][2 * q + 1]));
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        i16x2 word = __builtin_bit_cast(i16x2, wpk[kb][q0 + 2 * w]);
        word = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(word, __builtin_bit_cast(bf16x2, wpk[kb][q0 + 2 * w]), 1.0f,
                                                         false);
        word = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(word, __builtin_bit_cast(bf16x2, wpk[kb][q0 + 2 * w + 1]),
                                                         1.0f, true);
        pf[1][2 * c + w] = __builtin_bit_cast(int, word);
      }
#pragma unroll
      for (int q = q0; q < q0 + 4; ++q) lch8[q] = dot2_ones(wpk[kb][q], lch8[q]);
      if constexpr (c == 3)
        l_part += ((lch8[0] + lch8[1]) + (lch8[2] + lch8[3])) + ((lch8[4] + lch8[5]) + (lch8[6] + lch8[7]));
    }
  };
  auto pv_finish = [&]() __attribute__((always_inline)) {
    // reads per operand
    constexpr int RPO = DT == DT_BF16 ? 2 : 4;
    static_for<0, NPV>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      // the reads of the PV_AHEAD - 1 later operands may still be in flight
      lds_wait<RPO * (i + PV_AHEAD <= NPV ? PV_AHEAD - 1 : NPV - 1 - i)>(vring[i % (PV_AHEAD + 1)]);
      if constexpr (DT == DT_BF16)
        oacc[i >> 3] =
            __builtin_amdgcn_mfma_f32_32x32x16_bf16(vring[i % (PV_AHEAD + 1)], pb[i & 7], oacc[i >> 3], 0, 0, 0);
      else {
        constexpr int db = SPLIT ? i % NDB : i >> 1, t2 = SPLIT ? i / NDB : i & 1;
        static_assert(db < NDB && t2 < 2, "PV operand index");
        oacc[db] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(vring[i % (PV_AHEAD + 1)], pf[t2], oacc[db], 0, 0,
                                                                   0, 0, 0, 0);
      }
      // each MFMA issues as soon as its operand is in (not after later reads)
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (i + PV_AHEAD < NPV)
        vring[(i + PV_AHEAD) % (PV_AHEAD + 1)] = ldv(std::integral_constant<int, i + PV_AHEAD>{});
      if constexpr (SPLIT && i < NDB) {
        // parts 4i/NDB .. 4(i+1)/NDB - 1 run while MFMA i executes; MFMAs
        // NDB .. 2 NDB - 1 read what they write
        static_for<4 * i / NDB, 4 * (i + 1) / NDB>([&](auto cc) { finish_half(cc); });
        __builtin_amdgcn_sched_barrier(0);
      }
    });
  };

  // ---- masked keys (causal diagonal, ragged tail) of tile t get score -inf;
  // returns whether the tile needed masking
  auto mask_scores = [&](int t) __attribute__((always_inline)) {
    const int kt0 = t * BC;
    const bool need_mask = (CAUSAL && kt0 + BC - 1 > qw0) || (kt0 + BC > S);
    if (need_mask) {
      const int lim = (CAUSAL ? min(qrow, S - 1) : S - 1) - kt0 - 4 * g;
      mask_beyond(sacc, lim, -INFINITY);
    }
    return need_mask;
  };

  // ---- the probe variant writes tile t's weights and P for its probed rows
  auto probe_weights = [&](int t) __attribute__((always_inline)) {
    if constexpr (PROBE) {
      const int kt0 = t * BC;
      if (b == p.pb && h == p.ph && qrow >= p.prow0 && qrow < p.prow0 + p.pnrows) {
        const size_t rbase = (size_t)(qrow - p.prow0) * S;
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            const int key = kt0 + kb * 32 + 8 * (j >> 2) + 4 * g + (j & 3);
            if (key < S) {
              uint32_t bits;
              if constexpr (DT == DT_BF16) {
                // read the bf16 bits through a 32-bit view of the operand
                const u32x4 pw = __builtin_bit_cast(u32x4, pb[2 * kb + (j >> 3)]);
                bits = (pw[(j & 7) >> 1] >> (16 * (j & 1))) & 0xFFFFu;
              } else {
                bits = ((uint32_t)pf[kb >> 1][4 * (kb & 1) + (j >> 2)] >> (8 * (j & 3))) & 0xFFu;
              }
              p.w_out[rbase + key] =
                  mode_lattice(MODE) ? __uint_as_float(((wpk[kb][j >> 1] >> (16 * (j & 1))) & 0xFFFFu) << 16)
                                     : sacc[kb][j];
              p.p_out[rbase + key] = bits;
            }
          }
      }
    }
  };

  // ---- masking (causal diagonal and the ragged tail only), and the probe's
  // scores; returns whether the tile needed masking
  auto finish_scores = [&](int t) __attribute__((always_inline)) {
    const bool need_mask = mask_scores(t);
    if constexpr (PROBE) {
      if (b == p.pb && h == p.ph && qrow >= p.prow0 && qrow < p.prow0 + p.pnrows) {
        const size_t rbase = (size_t)(qrow - p.prow0) * S;
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            const int key = t * BC + kb * 32 + 8 * (j >> 2) + 4 * g + (j & 3);
            if (key < S) p.s_out[rbase + key] = sacc[kb][j];
          }
      }
    }
    return need_mask;
  };

  // ---- the anchor after a tile whose row maximum is the larger of ma and mb
  auto next_anchor = [&](float m, float ma, float mb) __attribute__((always_inline)) {
    float m_new = max3(m, ma, mb);
    if (DT == DT_BF16 && p.tau > 0.0f) {
      // conditional rescale (App. B.2; FP8 requires tau = 0): the anchor
      // moves only when the row's maximum grows by more than tau octaves
      // (FP32 test); per wave, when any real row of the wave does
      const float grow_by = (__builtin_fmaxf(ma, mb) - m) * p.c1;
      bool move = m == -INFINITY || grow_by > p.tau;
      if (p.tau_wave) move = __builtin_amdgcn_ballot_w64(move && qrow < S) != 0;
      if (!move) m_new = m;
    }
    return m_new;
  };

  // ---- the scores of tile t become weights, the running state moves, and P
  // is left in pb/pf for the PV product
  // (softmax_exponents, then softmax_weights; V sits at vl)
  float alpha = 1.0f;  // rescale factor of the open tile
  auto softmax_exponents = [&](int t, const uint8_t* vl, bool need_mask) __attribute__((always_inline)) {
    const int kt0 = t * BC;

    // running maximum (threshold 0: moves to the maximum so far); Rowmax-PoT
    // keeps the whole-row maximum of its first pass
    float m_new = m_run;
    if constexpr (PAIR) {
      // the tile before, which the other wave of the pair has, then this one
      const float mp = t > 0 ? mx_lds[0][1 - par][rw * WROWS + i32] : -INFINITY;
      m_new = next_anchor(m_run, mp, mp);
      m_new = next_anchor(m_new, m_tile, m_tile);
    } else if constexpr (MODE != MODE_ROWMAX_POT) {
      float ma, mb;
      with_partner(tile_max(sacc), ma, mb);
      m_new = next_anchor(m_run, ma, mb);
    }
    alpha = __builtin_amdgcn_exp2f((m_run - m_new) * p.c1);
    m_run = m_new;
    // the first V^T operands of this tile load while the weights are computed
    if constexpr (!PAIR) pv_begin(vl);
    // weights, in place over the scores (the lattice modes: as BF16 pairs)
    if constexpr (PACKED) {
      const float nbk = __builtin_fmaf(-m_new, p.ck, (float)(1 << mode_order(MODE)) * off);
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int j = 0; j < 16; ++j) sacc[kb][j] = __uint_as_float(sq_pre<MODE>(sacc[kb][j], p.ck, nbk));
      if (need_mask) {
        // masked keys carry weight 0 (the clamp alone would give 2^-126)
        if constexpr (mode_narrow(MODE)) {
          // their scores are -inf, so t = -inf here; every real t lies in
          // (0x1.8p23 - 2^15, 0x1.8p23 + 2^7), so one max lifts exactly the
          // masked keys to a value below all of them whose low half is the
          // masked-key lane value (v_max3: fmaxf would first canonicalise)
          const float lift = __uint_as_float(0x4B3F0000u | sq_masked<MODE>());
#pragma unroll
          for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int j = 0; j < 16; ++j) sacc[kb][j] = max3(sacc[kb][j], lift, lift);
        } else {
          const int lim = (CAUSAL ? min(qrow, S - 1) : S - 1) - kt0 - 4 * g;
          mask_beyond(sacc, lim, __uint_as_float(sq_masked<MODE>()));
        }
      }
    }
  };
  auto softmax_weights = [&](int t, const uint8_t* vl, bool need_mask) __attribute__((always_inline)) {
    const int kt0 = t * BC;
    if constexpr (PAIR) pv_begin(vl);
    if constexpr (PACKED) {
#pragma unroll
      for (int kb = 0; kb < (SPLIT ? 2 : 4); ++kb)
#pragma unroll
        for (int q = 0; q < 8; ++q)
          wpk[kb][q] = sq_pack<MODE>(__float_as_uint(sacc[kb][2 * q]), __float_as_uint(sacc[kb][2 * q + 1]));
      if constexpr (SPLIT) {
        // eight chains, continued by finish_half
        l_part = l_part * alpha;
#pragma unroll
        for (int q = 0; q < 8; ++q) lch8[q] = dot2_ones(wpk[1][q], dot2_ones(wpk[0][q], 0.0f));
      } else {
        l_part = pair_sum(wpk, l_part * alpha);
      }
    } else {
      if constexpr (MODE == MODE_ROWMAX_POT) {
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
          for (int j = 0; j < 16; ++j) sacc[kb][j] = pot_weight(sacc[kb][j], m_run, p.c1);
        if (need_mask) {
          const int lim = (CAUSAL ? min(qrow, S - 1) : S - 1) - kt0 - 4 * g;
          mask_beyond(sacc, lim, 0.0f);
        }
      } else {
        const float nb1 = __builtin_fmaf(-m_run, p.c1, off);
#pragma unroll
        for (int kb = 0; kb < (SPLIT ? 2 : 4); ++kb)
#pragma unroll
          for (int j = 0; j < 16; ++j) sacc[kb][j] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[kb][j], p.c1, nb1));
        nb1_split = nb1;
      }
      if constexpr (SPLIT) {
        // keys 0..63 now, 64..127 in finish_half
        float a[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) a[i] = sacc[0][i] + sacc[1][i];
#pragma unroll
        for (int w = 8; w >= 1; w >>= 1)
#pragma unroll
          for (int i = 0; i < w; ++i) a[i] = a[i] + a[i + w];
        l_part = l_part * alpha + a[0];
      } else {
        l_part = l_part * alpha + tile_sum(sacc);
      }
    }
    // skipping the rescale is exact when no row of the wave moved its max
    if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int j = 0; j < 16; ++j) oacc[db][j] *= alpha;
    }

    // P in the operand type
    if constexpr (DT == DT_BF16) {
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        if constexpr (PACKED) {
          const int kb = ks >> 1, q0 = 4 * (ks & 1);
          pb[ks] = __builtin_bit_cast(bf16x8, u32x4{wpk[kb][q0], wpk[kb][q0 + 1], wpk[kb][q0 + 2], wpk[kb][q0 + 3]});
        } else {
#pragma unroll
          for (int r = 0; r < 8; ++r) pb[ks][r] = (__bf16)sacc[ks >> 1][8 * (ks & 1) + r];
        }
      }
    } else {
#pragma unroll
      for (int t2 = 0; t2 < (SPLIT ? 1 : 2); ++t2)
#pragma unroll
        for (int w4 = 0; w4 < 8; ++w4) {
          const int kb = 2 * t2 + (w4 >> 2), j0 = 4 * (w4 & 3);
          if constexpr (PACKED) {
            // BF16 -> e4m3 with unit scale (the weights are exact in BF16);
            // the old value is fully overwritten by the two halves
            i16x2 word = __builtin_bit_cast(i16x2, wpk[kb][j0 / 2]);
            word = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(word, __builtin_bit_cast(bf16x2, wpk[kb][j0 / 2]), 1.0f,
                                                             false);
            word = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(word, __builtin_bit_cast(bf16x2, wpk[kb][j0 / 2 + 1]),
                                                             1.0f, true);
            pf[t2][w4] = __builtin_bit_cast(int, word);
          } else {
            // the old value is fully overwritten by the two halves
            uint32_t word = __float_as_uint(sacc[kb][j0]);
            word = __builtin_amdgcn_cvt_pk_fp8_f32(sacc[kb][j0], sacc[kb][j0 + 1], word, false);
            word = __builtin_amdgcn_cvt_pk_fp8_f32(sacc[kb][j0 + 2], sacc[kb][j0 + 3], word, true);
            pf[t2][w4] = (int)word;
          }
        }
    }
    if constexpr (!SPLIT) probe_weights(t);
  };

  // last tile holding a valid key for some row of this wave (-1: none)
  const int last_act = !wave_live ? -1 : (CAUSAL ? min(ntiles - 1, (qw0 + WROWS - 1) / BC) : ntiles - 1);
  if constexpr (MODE == MODE_ROWMAX_POT) {
    // ---- Rowmax-PoT anchors every weight at the whole-row maximum: a first
    // pass over the key tiles computes it (QK^T and the masked row max only)
    stage_q();
    stage(0, kbuf(0), krsrc, koff);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    read_q();
    __syncthreads();
    for (int t = 0; t < ntiles; ++t) {
      if (t + 1 < ntiles) stage(t + 1, kbuf(t + 1), krsrc, koff);
      if (t <= last_act) {
        __builtin_amdgcn_s_setprio(1);
        qk(kbuf(t));
        __builtin_amdgcn_s_setprio(0);
        settle_scores(sacc);
        mask_scores(t);
        const float mt = tile_max(sacc);
        float ma, mb;
        with_partner(mt, ma, mb);
        m_run = max3(m_run, ma, mb);
      }
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
    }
  }

  // ---- one tile per step: copy in the next tile, then QK^T, weights, PV.
  // Steps come in pairs so that each one's LDS buffers are fixed at compile
  // time and their addresses fold into the reads' immediate offsets.
  // Single-buffered tiles: the next K is copied in once every wave has read
  // K, during the weights and PV, and the next V once every wave has read V,
  // during the next QK^T; each wait for a copy comes just before the barrier
  // that makes it visible.
  // Paired: the waves of the odd tiles run one barrier behind those of the
  // even ones, so of the two waves of a SIMD one is in the first half of its
  // step (QK^T, maximum, anchor, exponents) while the other is in the second
  // (weights, O rescale, PV), and each tile's maximum is there when the next
  // tile's anchor needs it.
  auto scores = [&](const uint8_t* kl) __attribute__((always_inline)) {
    __builtin_amdgcn_s_setprio(1);
    qk(kl);
    __builtin_amdgcn_s_setprio(0);
    settle_scores(sacc);
  };
  auto weights_pv = [&](int t, const uint8_t* vl, bool need_mask) __attribute__((always_inline)) {
    softmax_weights(t, vl, need_mask);
    __builtin_amdgcn_s_setprio(1);
    pv_finish();
    __builtin_amdgcn_s_setprio(0);
    if constexpr (SPLIT) probe_weights(t);
  };
  // this wave's copy of V(t) has landed and its reads of K(t) are done
  auto turn_k = [&](int t) __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (PAIR || t + 1 < ntiles) stage(t + C::NPAR, ktile, krsrc, koff);
  };
  // this wave's copy of the next K has landed and its reads of V(t) are done
  auto turn_v = [&](int t) __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (PAIR || t + 1 < ntiles) stage(t + C::NPAR, vtile, vrsrc, voff);
  };
  auto step_single = [&](int t) __attribute__((always_inline)) {
    if (t <= last_act) scores(ktile);
    turn_k(t);
    if (t <= last_act) {
      const bool need_mask = finish_scores(t);
      softmax_exponents(t, vtile, need_mask);
      weights_pv(t, vtile, need_mask);
    }
    turn_v(t);
  };
  auto step_paired = [&](int t, auto active) __attribute__((always_inline)) {
    float* const mx = &mx_lds[0][par][rw * WROWS + i32];
    if constexpr (decltype(active)::value) {
      scores(ktile);
      const bool need_mask = finish_scores(t);
      float ma, mb;
      with_partner(tile_max(sacc), ma, mb);
      m_tile = __builtin_fmaxf(ma, mb);
      if (g == 0) *mx = m_tile;
      softmax_exponents(t, vtile, need_mask);
      turn_k(t);
      weights_pv(t, vtile, need_mask);
    } else {
      if (g == 0) *mx = -INFINITY;
      turn_k(t);
    }
    turn_v(t);
  };
  auto step = [&](int t, auto buf) __attribute__((always_inline)) {
    constexpr int P = decltype(buf)::value;
    uint8_t* const kl = smem + P * C::BUF;
    if (t + 1 < ntiles) {
      stage(t + 1, smem + (1 - P) * C::BUF, krsrc, koff);
      stage(t + 1, smem + (1 - P) * C::BUF + C::TILE, vrsrc, voff);
    }
    if (t <= last_act) {
      scores(kl);
      const bool need_mask = finish_scores(t);
      softmax_exponents(t, kl + C::TILE, need_mask);
      weights_pv(t, kl + C::TILE, need_mask);
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
  };
  if constexpr (PAIR) {
    // Q where the rows of O go at the end, or in the V tiles
    stage_q();
    stage(par, ktile, krsrc, koff);
    if constexpr (OWN_OST) {
      __builtin_amdgcn_sched_barrier(0);
      stage(par, vtile, vrsrc, voff);
      // Q and K are there before the first step, V at its middle
      wait_vmcnt<WAVE_LOADS>();
      lds_barrier();
      read_q();
    } else {
      wait_vmcnt<0>();
      lds_barrier();
      read_q();
      lds_barrier();
      stage(par, vtile, vrsrc, voff);
    }
    // (both halves cross the same number of barriers)
    if (par != 0) lds_barrier();
    int t = par;
    for (; t <= last_act; t += 2) step_paired(t, std::true_type{});
    for (; t < (ntiles + 1) / 2 * 2; t += 2) step_paired(t, std::false_type{});
    if (par == 0) lds_barrier();
    // (the last copies, of no tile, have landed before the tiles are reused)
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
  } else if constexpr (NSTAGE == 1) {
    stage_q();
    stage(0, ktile, krsrc, koff);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    read_q();
    __syncthreads();
    stage(0, vtile, vrsrc, voff);
    for (int t = 0; t < ntiles; ++t) step_single(t);
  } else {
    if constexpr (MODE != MODE_ROWMAX_POT) stage_q();
    stage(0, smem, krsrc, koff);
    stage(0, smem + C::TILE, vrsrc, voff);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if constexpr (MODE != MODE_ROWMAX_POT) {
      read_q();
      __syncthreads();
    }
    for (int t = 0; t < ntiles; t += 2) {
      step(t, std::integral_constant<int, 0>{});
      if (t + 1 < ntiles) step(t + 1, std::integral_constant<int, 1>{});
    }
  }

  // ---- epilogue: O = acc / l * v_descale (bf16), LSE.  A wave writes blocks
  // DB0 .. DB0 + NOB - 1 of its rows' columns (paired: one half each).
  float la, lb;
  with_partner(l_part, la, lb);
  float l = la + lb, m_end = m_run;
  uint8_t* const ost = (OWN_OST ? osm : PAIR ? smem + OX : smem) + wave * (WROWS * NOB * 64);
  if constexpr (PAIR) {
    // the two waves of a pair hold sums relative to their own anchors: each
    // sends the other its part of the other's columns through LDS, which is
    // free once every wave has passed the last barrier
    // ([row wave][block][quarter][lane], the even half's in smem, the odd
    // half's in vsm)
    const int exo = rw * (NOB * 4 * 64) + lane;
    auto send = [&](auto other, f32x4* ex) __attribute__((always_inline)) {
#pragma unroll
      for (int o = 0; o < NOB; ++o)
#pragma unroll
        for (int jq = 0; jq < 4; ++jq) {
          const f32x16& a = oacc[decltype(other)::value * NOB + o];
          ex[exo + (o * 4 + jq) * 64] = f32x4{a[4 * jq], a[4 * jq + 1], a[4 * jq + 2], a[4 * jq + 3]};
        }
    };
    if (par == 0) send(std::integral_constant<int, 1>{}, (f32x4*)smem);
    else send(std::integral_constant<int, 0>{}, (f32x4*)vsm);
    if (g == 0) {
      mx_lds[0][par][rw * WROWS + i32] = m_run;
      mx_lds[1][par][rw * WROWS + i32] = l;
    }
    __syncthreads();
    if (!wave_live) return;
    const float m_other = mx_lds[0][1 - par][rw * WROWS + i32];
    m_end = __builtin_fmaxf(m_run, m_other);
    // (a wave without a visible key has m = -inf, l = 0, O = 0)
    const float fm = m_run == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f((m_run - m_end) * p.c1);
    const float fo = m_other == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f((m_other - m_end) * p.c1);
    l = fm * l + fo * mx_lds[1][1 - par][rw * WROWS + i32];
    auto merge = [&](auto half, const f32x4* ex) __attribute__((always_inline)) {
#pragma unroll
      for (int o = 0; o < NOB; ++o)
#pragma unroll
        for (int jq = 0; jq < 4; ++jq) {
          const f32x4 x = ex[exo + (o * 4 + jq) * 64];
#pragma unroll
          for (int e = 0; e < 4; ++e)
            oacc[o][4 * jq + e] = fm * oacc[decltype(half)::value * NOB + o][4 * jq + e] + fo * x[e];
        }
    };
    if (par == 0) merge(std::integral_constant<int, 0>{}, (const f32x4*)vsm);
    else merge(std::integral_constant<int, 1>{}, (const f32x4*)smem);
  } else {
    if (!wave_live) return;
  }
  const float inv = p.vd / l;
  // O leaves through LDS, which is free once every wave has passed the last
  // barrier: the lanes write their four-column pieces into the wave's own
  // 32-row block there (16-byte chunks XOR-swizzled by row: the reads are
  // free of bank conflicts, the writes of rows r and r + 16 share banks) and
  // read back 16 contiguous bytes of a row, so that each global store covers
  // whole rows (paired: whole halves) instead of 8 bytes in each of 32 rows
  constexpr int ORB = NOB * 64, ONC = ORB / 16;  // bytes and 16-byte chunks per staged row
  auto oswz = [](int row) { return ONC == 16 ? (row & 15) : ONC == 8 ? ((row >> 1) & 7) : ((row >> 2) & 3); };
#pragma unroll
  for (int db = 0; db < NOB; ++db)
#pragma unroll
    for (int jq = 0; jq < 4; ++jq) {
      const __bf16 a0 = (__bf16)(oacc[db][4 * jq + 0] * inv);
      const __bf16 a1 = (__bf16)(oacc[db][4 * jq + 1] * inv);
      const __bf16 a2 = (__bf16)(oacc[db][4 * jq + 2] * inv);
      const __bf16 a3 = (__bf16)(oacc[db][4 * jq + 3] * inv);
      const uint32_t w01 = (uint32_t)__builtin_bit_cast(uint16_t, a0) |
                           ((uint32_t)__builtin_bit_cast(uint16_t, a1) << 16);
      const uint32_t w23 = (uint32_t)__builtin_bit_cast(uint16_t, a2) |
                           ((uint32_t)__builtin_bit_cast(uint16_t, a3) << 16);
      // columns 32 db + 8 jq + 4 g .. +3: chunk 4 db + jq, half g
      *(u32x2*)(ost + i32 * ORB + (((4 * db + jq) ^ oswz(i32)) << 4) + 8 * g) = u32x2{w01, w23};
    }
  // the wave reads what its other lanes wrote (LDS keeps a wave's order)
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  constexpr int RPI = 64 / ONC;  // rows per store
  const int rsub = lane / ONC, csub = lane % ONC;
  uint8_t* const obase = (uint8_t*)p.o + (q_head + qw0) * (size_t)(D * 2) + par * ORB + csub * 16;
  u32x4 orows[WROWS / RPI];
#pragma unroll
  for (int k = 0; k < WROWS / RPI; ++k) {
    const int r = RPI * k + rsub;
    orows[k] = *(const u32x4*)(ost + r * ORB + ((csub ^ oswz(r)) << 4));
  }
  if (qw0 + WROWS <= S) {
#pragma unroll
    for (int k = 0; k < WROWS / RPI; ++k) *(u32x4*)(obase + (size_t)(RPI * k + rsub) * (D * 2)) = orows[k];
  } else {
#pragma unroll
    for (int k = 0; k < WROWS / RPI; ++k)
      if (qw0 + RPI * k + rsub < S) *(u32x4*)(obase + (size_t)(RPI * k + rsub) * (D * 2)) = orows[k];
  }
  if (p.lse && par == 0 && g == 0 && qrow < S)
    p.lse[q_head + qrow] = 0.69314718055994531f * (m_end * p.c1 + log2f(l) - off);
}

// Two waves per SIMD, three for fp8 at d = 64 (163 VGPRs, 32 KB of LDS per
// workgroup: three workgroups fit a CU, and the third wave hides more of the
// VALU latency in that VALU-bound case).
template <int DT, int D, bool CAUSAL, int MODE, bool PROBE, bool CMP>
__global__ __launch_bounds__(MAX_THREADS) __attribute__((amdgpu_waves_per_eu(2, (DT == DT_FP8 && D == 64) ? 3 : 2))) void
attn_fwd_kernel(Params p) {
  fwd_body<DT, D, CAUSAL, MODE, PROBE, CMP ? LAY_COMPACT : LAY_WIDE>(p);
}

// Bound by the chain of one wave's tiles rather than by the chip: from 4K to 8K
// rows (FP8 H15, causal, 256 blocks) a tile of the longest chain costs 1.72 us
// with a lone wave on each SIMD and 1.12 with two (about 4,000 and 2,600 cycles;
// with both halves in step 3,300, with the barrier right after QK^T 2,750).  GPU
// time, causal: 4 heads of 8K FP8 H15 119 -> 81 us, BF16 144 -> 110; 16 heads of
// 2K 34.6 -> 25.9, 41.6 -> 33.2; 16 heads of 1K 19.7 -> 15.7, 23.8 -> 19.8.
template <int DT, int D, bool CAUSAL, int MODE, bool PROBE>
__global__ __launch_bounds__(MAX_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_fwd_paired_kernel(
    Params p) {
  fwd_body<DT, D, CAUSAL, MODE, PROBE, LAY_PAIRED>(p);
}

#if !H15_FP8_LATTICE_D128
// Probe support: pre-fill the probe buffers (s = -inf, w = 0, P = 0).
__global__ void probe_fill(float* s, float* w, uint32_t* pbits, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    s[i] = -INFINITY;
    w[i] = 0.0f;
    pbits[i] = 0u;
  }
}
#endif

template <int DT, int D, bool CAUSAL, int MODE, bool PROBE>
hipError_t launch_one(const Params& p, hipStream_t st) {
  const unsigned grid = (unsigned)(p.nqb * p.B * p.Hq);
  if constexpr (MODE != MODE_ROWMAX_POT) {
    if (p.layout == LAY_PAIRED) {
      hipLaunchKernelGGL((attn_fwd_paired_kernel<DT, D, CAUSAL, MODE, PROBE>), dim3(grid),
                         dim3(Cfg<DT, D, LAY_PAIRED>::NW * 64), 0, st, p);
      return hipGetLastError();
    }
  }
  if constexpr (DT == DT_BF16 && MODE != MODE_ROWMAX_POT) {
    if (p.layout == LAY_COMPACT) {
      hipLaunchKernelGGL((attn_fwd_kernel<DT, D, CAUSAL, MODE, PROBE, true>), dim3(grid),
                         dim3(Cfg<DT, D, LAY_COMPACT>::NW * 64), 0, st, p);
      return hipGetLastError();
    }
  }
  if (p.layout != LAY_WIDE) return hipErrorInvalidValue;  // not offered for this weight or type
  hipLaunchKernelGGL((attn_fwd_kernel<DT, D, CAUSAL, MODE, PROBE, false>), dim3(grid), dim3(Cfg<DT, D>::NW * 64), 0,
                     st, p);
  return hipGetLastError();
}

#if H15_FP8_LATTICE_D128
template <bool CAUSAL, bool PROBE>
hipError_t launch_lattice128(const Params& p, int mode, hipStream_t st) {
  switch (mode) {
    case 1: return launch_one<DT_FP8, 128, CAUSAL, 1, PROBE>(p, st);
    case 2: return launch_one<DT_FP8, 128, CAUSAL, 2, PROBE>(p, st);
    case 3: return launch_one<DT_FP8, 128, CAUSAL, 3, PROBE>(p, st);
    case 4: return launch_one<DT_FP8, 128, CAUSAL, 4, PROBE>(p, st);
    case 5: return launch_one<DT_FP8, 128, CAUSAL, 5, PROBE>(p, st);
    case 6: return launch_one<DT_FP8, 128, CAUSAL, 6, PROBE>(p, st);
    default: return hipErrorInvalidValue;
  }
}
#else
template <int DT, int D, bool CAUSAL, bool PROBE>
hipError_t launch_mode(const Params& p, int mode, hipStream_t st) {
  if (mode == MODE_EXACT) return launch_one<DT, D, CAUSAL, MODE_EXACT, PROBE>(p, st);
  if constexpr (DT == DT_FP8 && D == 128) {
    // the FP8 lattice weights at d = 128 live in the other compilation of
    // this file
    return h15::launch_fwd_fp8_lattice128(p, CAUSAL, mode, st, PROBE);
  } else {
    switch (mode) {
      case 1: return launch_one<DT, D, CAUSAL, 1, PROBE>(p, st);
      case 3: return launch_one<DT, D, CAUSAL, 3, PROBE>(p, st);
      case 5: return launch_one<DT, D, CAUSAL, 5, PROBE>(p, st);
      default: break;
    }
    if constexpr (DT == DT_BF16) {
      if (mode == MODE_ROWMAX_POT) return launch_one<DT, D, CAUSAL, MODE_ROWMAX_POT, PROBE>(p, st);
    }
    // the narrow-clamp forms are only ever chosen for FP8
    if constexpr (DT == DT_FP8) {
      switch (mode) {
        case 2: return launch_one<DT, D, CAUSAL, 2, PROBE>(p, st);
        case 4: return launch_one<DT, D, CAUSAL, 4, PROBE>(p, st);
        case 6: return launch_one<DT, D, CAUSAL, 6, PROBE>(p, st);
        default: break;
      }
    }
    return hipErrorInvalidValue;
  }
}

template <int DT, int D, bool PROBE>
hipError_t launch_dt_d(const Params& p, int causal, int mode, hipStream_t st) {
  return causal ? launch_mode<DT, D, true, PROBE>(p, mode, st) : launch_mode<DT, D, false, PROBE>(p, mode, st);
}

template <bool PROBE>
hipError_t launch_any(const Params& p, int dtype, int d, int causal, int mode, hipStream_t st) {
  if (dtype == ATTN_BF16)
    return d == 128 ? launch_dt_d<DT_BF16, 128, PROBE>(p, causal, mode, st)
                    : launch_dt_d<DT_BF16, 64, PROBE>(p, causal, mode, st);
  return d == 128 ? launch_dt_d<DT_FP8, 128, PROBE>(p, causal, mode, st)
                  : launch_dt_d<DT_FP8, 64, PROBE>(p, causal, mode, st);
}

#endif  // !H15_FP8_LATTICE_D128

}  // namespace

namespace h15 {

#if H15_FP8_LATTICE_D128
hipError_t launch_fwd_fp8_lattice128(const Params& p, bool causal, int mode, hipStream_t st, bool probe) {
  if (probe) return causal ? launch_lattice128<true, true>(p, mode, st) : launch_lattice128<false, true>(p, mode, st);
  return causal ? launch_lattice128<true, false>(p, mode, st) : launch_lattice128<false, false>(p, mode, st);
}
#else
int launch_fwd(const Params& p, int dtype, int d, int causal, int mode, void* stream, bool probe) {
  hipStream_t st = (hipStream_t)stream;
  const hipError_t e = probe ? launch_any<true>(p, dtype, d, causal, mode, st)
                             : launch_any<false>(p, dtype, d, causal, mode, st);
  return e == hipSuccess ? 0 : 1;
}

int launch_probe_fill(float* s, float* w, uint32_t* pbits, size_t n, void* stream) {
  hipLaunchKernelGGL(probe_fill, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream, s, w, pbits,
                     n);
  return hipGetLastError() == hipSuccess ? 0 : 1;
}
#endif

}  // namespace h15
