// Decode over a key/value cache (attn_decode, attn_decode_noalloc): Sq query
// rows per head against Sk cached keys (bottom-right causal alignment), the
// keys cut into parts of split_keys keys that workgroups take in parallel.
// Within a part the per-tile recurrence of the forward kernel runs, with
// tiles starting at the part's first key and the running maximum starting at
// -inf; the parts' (m, l, O) then merge exactly.
//
// One workgroup = NW = 4 waves for one (batch, KV head, block of 32 query
// rows, part).  The 32 rows are the G * Sq query rows of the KV head's
// query heads (row r: head h = hkv G + r / Sq, position r % Sq), so the K/V
// tiles are read once for all of them.
//
// Decode reads the cache once, so it is bound by HBM, or, when there are few
// keys, by the chain of latencies from the first load to the last store.  The
// split of the work shortens that chain and keeps many bytes in flight:
//   * the unit of a wave is 64 keys, half a tile; a round covers NW / 2 whole
//     tiles, so a part of n tiles takes ceil(2 n / NW) rounds.  Parts of few
//     tiles, where that would leave waves without keys, have units of 32
//     keys and a tile a round (the rule: attn_api.cpp);
//   * a weight is rounded relative to the running maximum at its own tile, the
//     maximum over the tiles up to it, not to the last tile before it in some
//     wave.  The waves therefore exchange the maxima of their units (one
//     barrier a round) and each takes the prefix maximum up to its tile as
//     its anchor, which gives the recurrence's weights; row sums and O are
//     kept per wave relative to the wave's own anchor and brought to the
//     part's last one at the end;
//   * no barrier waits for a copy: a wave loads only its own keys, K straight
//     into its MFMA operand registers (the next round's as soon as this
//     round's scores are computed; or through LDS, see KLDS) and V into its own LDS slots (the next
//     round's once this round's are read).  The barrier is a bare s_barrier
//     after the wait for the LDS writes: the compiler's __syncthreads also
//     waits for every load in flight, which serialised the copies with the
//     tiles (2 us a tile at one workgroup per CU).
// Measured against four waves that shared every tile (32 keys each, a
// __syncthreads a tile), GPU time of one call: one sequence of 32 heads over 8
// KV heads with 32K keys 43.6 -> 30.8 us (BF16), 30.6 -> 17.1 (FP8); 8 KV heads
// with 700 keys 14.0 -> 10.4 (BF16), 11.3 -> 7.5 (FP8); B16 8K 98.3 -> 93.9
// (BF16, 5.7 TB/s), B200 1K 154.5 -> 144.1 (BF16), 88.4 -> 76.6 (FP8).
//
// attn_decode_merge follows where there are several parts.  (Merging in the
// same launch, by the last workgroup of a row block to finish, was measured:
// with agent-scope fences each workgroup writes back and invalidates its
// XCD's L2, +17..25 us a call; with write-through stores and no fences it
// gains 0.3..0.5 us at four query rows a block and loses 4 us at 16.)
#include <mutex>

#include "attn_device.h"

namespace {

constexpr int NW = 4;               // waves per workgroup
// instruction classes of __builtin_amdgcn_sched_group_barrier
constexpr int SG_MFMA = 0x008;
constexpr int SG_DS_READ = 0x100;

// The scores are next read by inline asm (v_max3_f32, the masking's compare
// and select), and the compiler inserts no wait states between a matrix-core
// write and an inline-asm read: this holds the wave for 24, more than the 20
// that gfx950 requires after a 16-pass write.
template <int NB>
__device__ __forceinline__ void settle_unit(f32x16 (&v)[NB]) {
  if constexpr (NB == 2) asm("s_nop 15\n\ts_nop 7" : "+v"(v[0]), "+v"(v[1]));
  else asm("s_nop 15\n\ts_nop 7" : "+v"(v[0]));
}

// y over the scores of a unit (32 or 64 keys) whose key offset lies beyond lim
template <int NB, int E = 0>
__device__ __forceinline__ void mask_unit(f32x16 (&v)[NB], int lim, float y) {
  if constexpr (E < 16 * NB) {
    constexpr int kb = E / 16, j = E % 16;
    v[kb][j] = select_beyond<kb * 32 + 8 * (j >> 2) + (j & 3)>(lim, v[kb][j], y);
    mask_unit<NB, E + 1>(v, lim, y);
  }
}

template <int NB>
__device__ __forceinline__ float unit_max(const f32x16 (&v)[NB]) {
  // 32 -> 11 -> 4 -> 2 -> 1, or 16 -> 6 -> 2 -> 1
  if constexpr (NB == 2) {
    float a[11], b[4];
#pragma unroll
    for (int i = 0; i < 10; ++i) {
      const int e0 = 3 * i, e1 = 3 * i + 1, e2 = 3 * i + 2;
      a[i] = max3(v[e0 >> 4][e0 & 15], v[e1 >> 4][e1 & 15], v[e2 >> 4][e2 & 15]);
    }
    a[10] = max3(v[1][14], v[1][15], v[1][15]);
    b[0] = max3(a[0], a[1], a[2]);
    b[1] = max3(a[3], a[4], a[5]);
    b[2] = max3(a[6], a[7], a[8]);
    b[3] = max3(a[9], a[10], a[10]);
    const float c = max3(b[0], b[1], b[2]);
    return max3(c, b[3], b[3]);
  } else {
    float a[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) a[i] = max3(v[0][3 * i], v[0][3 * i + 1], v[0][3 * i + 2]);
    const float b0 = max3(a[0], a[1], a[2]), b1 = max3(a[3], a[4], v[0][15]);
    return max3(b0, b1, b1);
  }
}

// The transposing LDS reads of V operands, with their wait in the same
// statement: the builtin forms make the compiler wait for every copy into LDS
// that is in flight, also those of the next round's K.
// bf16: two blocks of 32 columns (a0, a1), the eight 8-row steps of 64 keys
template <int RB>
__device__ __forceinline__ void read_v16(i32x2v (&r)[16], uint32_t a0, uint32_t a1) {
  asm volatile(
      "ds_read_b64_tr_b16 %0, %16\n\tds_read_b64_tr_b16 %1, %16 offset:%18\n\t"
      "ds_read_b64_tr_b16 %2, %16 offset:%19\n\tds_read_b64_tr_b16 %3, %16 offset:%20\n\t"
      "ds_read_b64_tr_b16 %4, %16 offset:%21\n\tds_read_b64_tr_b16 %5, %16 offset:%22\n\t"
      "ds_read_b64_tr_b16 %6, %16 offset:%23\n\tds_read_b64_tr_b16 %7, %16 offset:%24\n\t"
      "ds_read_b64_tr_b16 %8, %17\n\tds_read_b64_tr_b16 %9, %17 offset:%18\n\t"
      "ds_read_b64_tr_b16 %10, %17 offset:%19\n\tds_read_b64_tr_b16 %11, %17 offset:%20\n\t"
      "ds_read_b64_tr_b16 %12, %17 offset:%21\n\tds_read_b64_tr_b16 %13, %17 offset:%22\n\t"
      "ds_read_b64_tr_b16 %14, %17 offset:%23\n\tds_read_b64_tr_b16 %15, %17 offset:%24\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7]),
        "=&v"(r[8]), "=&v"(r[9]), "=&v"(r[10]), "=&v"(r[11]), "=&v"(r[12]), "=&v"(r[13]), "=&v"(r[14]), "=&v"(r[15])
      : "v"(a0), "v"(a1), "n"(8 * RB), "n"(16 * RB), "n"(24 * RB), "n"(32 * RB), "n"(40 * RB), "n"(48 * RB),
        "n"(56 * RB)
      : "memory");
}
// the four 8-row steps of 32 keys
template <int RB>
__device__ __forceinline__ void read_v16(i32x2v (&r)[8], uint32_t a0, uint32_t a1) {
  asm volatile(
      "ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %1, %8 offset:%10\n\t"
      "ds_read_b64_tr_b16 %2, %8 offset:%11\n\tds_read_b64_tr_b16 %3, %8 offset:%12\n\t"
      "ds_read_b64_tr_b16 %4, %9\n\tds_read_b64_tr_b16 %5, %9 offset:%10\n\t"
      "ds_read_b64_tr_b16 %6, %9 offset:%11\n\tds_read_b64_tr_b16 %7, %9 offset:%12\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7])
      : "v"(a0), "v"(a1), "n"(8 * RB), "n"(16 * RB), "n"(24 * RB)
      : "memory");
}
// fp8: two blocks of 32 columns, the four 16-row steps of 64 keys
template <int RB>
__device__ __forceinline__ void read_v8(i32x2v (&r)[8], uint32_t a0, uint32_t a1) {
  asm volatile(
      "ds_read_b64_tr_b8 %0, %8\n\tds_read_b64_tr_b8 %1, %8 offset:%10\n\t"
      "ds_read_b64_tr_b8 %2, %8 offset:%11\n\tds_read_b64_tr_b8 %3, %8 offset:%12\n\t"
      "ds_read_b64_tr_b8 %4, %9\n\tds_read_b64_tr_b8 %5, %9 offset:%10\n\t"
      "ds_read_b64_tr_b8 %6, %9 offset:%11\n\tds_read_b64_tr_b8 %7, %9 offset:%12\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7])
      : "v"(a0), "v"(a1), "n"(16 * RB), "n"(32 * RB), "n"(48 * RB)
      : "memory");
}

// the two 16-row steps of 32 keys
template <int RB>
__device__ __forceinline__ void read_v8(i32x2v (&r)[4], uint32_t a0, uint32_t a1) {
  asm volatile(
      "ds_read_b64_tr_b8 %0, %4\n\tds_read_b64_tr_b8 %1, %4 offset:%6\n\t"
      "ds_read_b64_tr_b8 %2, %5\n\tds_read_b64_tr_b8 %3, %5 offset:%6\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3])
      : "v"(a0), "v"(a1), "n"(16 * RB)
      : "memory");
}

// O and LSE of one row from its parts, by one wave: m = max m_p, f_p =
// 2^(c1 (m_p - m)) (0 for a part that saw no key), l = sum f_p l_p,
// O = sum f_p O_p / l * v_descale, LSE = ln2 (m c1 + log2 l - off).  Lane j
// holds four columns and every (64 / (D / 4))th part, and the rows of up to 32
// parts are in flight at once: 4.0 us at 32 parts and 32 rows, where one wave
// reading its parts one after the other took 11.8.  As compiled a row still
// costs two round trips, since the wait for its (m, l) comes before the first
// row load, and, the row not being known to be uniform, each load's resource
// goes through a loop over its values in the wave.
template <int D>
__device__ __forceinline__ void merge_row(const float* ml, const float* po, int nsplit, float c1, float vd, float off,
                                          uint16_t* orow, float* lse) {
  constexpr int LPP = D / 4, PG = 64 / LPP;  // lanes per part, parts at once
  constexpr int U = 32 / PG, U4 = U / 4;     // reads in flight, taken in quarters
  const int lane = threadIdx.x & 63;
  const int pg = lane / LPP, col = 4 * (lane % LPP);
  // parts s0 .. s0 + 31: (m, l) in the lanes, the rows in v (zero, and f 0,
  // beyond the last part)
  f32x2 w;
  f32x4 v[U];
  auto fetch = [&](int s0) __attribute__((always_inline)) {
    w = lane < 32 && s0 + lane < nsplit ? *(const f32x2*)(ml + 2 * (s0 + lane)) : f32x2{-INFINITY, 0.0f};
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(po + (size_t)s0 * D), (short)0, min(nsplit - s0, 32) * D * 4, BUF_DWORD3);
#pragma unroll
    for (int u0 = 0; u0 < U; u0 += U4) {
      if (u0 > 0 && s0 + u0 * PG >= nsplit) break;
#pragma unroll
      for (int u = u0; u < u0 + U4; ++u)
        v[u] = __builtin_bit_cast(
            f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, ((u * PG + pg) * D + col) * 4, 0, 0));
    }
  };
  fetch(0);
  float m = w[0];
#pragma unroll 1
  for (int s = 32 + lane; s < nsplit; s += 64) m = __builtin_fmaxf(m, ml[2 * s]);
#pragma unroll
  for (int x = 32; x >= 1; x >>= 1) m = __builtin_fmaxf(m, __shfl_xor(m, x, 64));
  float l = 0.0f;
  f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
  for (int s0 = 0;;) {
    const float f = w[0] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f((w[0] - m) * c1);
    l += f * w[1];
#pragma unroll
    for (int u0 = 0; u0 < U; u0 += U4) {
      if (u0 > 0 && s0 + u0 * PG >= nsplit) break;
#pragma unroll
      for (int u = u0; u < u0 + U4; ++u) {
        const float fs = __shfl(f, u * PG + pg, 64);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += fs * v[u][e];
      }
    }
    s0 += 32;
    if (s0 >= nsplit) break;
    fetch(s0);
  }
#pragma unroll
  for (int x = 32; x >= 1; x >>= 1) l += __shfl_xor(l, x, 64);
#pragma unroll
  for (int x = LPP; x < 64; x <<= 1)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] += __shfl_xor(acc[e], x, 64);
  if (pg == 0) {
    const float inv = vd / l;
    uint32_t w[2];
#pragma unroll
    for (int e = 0; e < 2; ++e)
      w[e] = (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)(acc[2 * e] * inv)) |
             ((uint32_t)__builtin_bit_cast(uint16_t, (__bf16)(acc[2 * e + 1] * inv)) << 16);
    *(u32x2*)(orow + col) = u32x2{w[0], w[1]};
  }
  if (lse && lane == 0) *lse = 0.69314718055994531f * (m * c1 + log2f(l) - off);
}

// UNIT: keys of a wave and round.  ONE: the parts have one round, so there is
// nothing to copy for a next one (one tile, B200, BF16: 22.4 -> 20.6 us; left
// out of longer parts' last round by a branch, the rest of the loop schedules
// worse: +2..25%).
// KLDS: K of a round comes through LDS like V, in copies of whole rows, else
// straight into the MFMA operand registers, in loads of 32 rows with 32 bytes
// each.  The rules between the forms stand where they are applied
// (attn_api.cpp).
template <int DT, int D, int UNIT, bool ONE, bool KLDS, bool CAUSAL, int MODE, bool PROBE>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_decode_kernel(DecParams p) {
  using C = Cfg<DT, D>;
  constexpr int NDB = D / 32;
  constexpr int NKQ = DT == DT_BF16 ? D / 16 : D / 64;
  constexpr int SLOT = UNIT * C::RB;                            // one wave's K or V rows of a round
  constexpr int LOADS = SLOT / 1024;                            // 1 KB LDS copies per wave and round
  constexpr int NB = UNIT / 32;                                 // 32-key score blocks of a unit
  constexpr int TPR = NW * UNIT / BC;                           // tiles per round
  constexpr int KLOADS = KLDS ? LOADS : NB * (DT == DT_BF16 ? NKQ : 2 * NKQ);  // K loads per lane and round
  static_assert(TPR == 1 || TPR == 2, "the anchors of a round");
  // the final reduction takes rows 0..15 of every wave's O in vsm, rows 16..31
  // in ksm (K in registers: behind the others in vsm)
  constexpr int RHALF = 16, RBYTES = NW * RHALF * D * 4, RMIN = KLDS ? RBYTES : 2 * RBYTES;
  constexpr int SLOTS = NW * SLOT > RMIN ? NW * SLOT : RMIN;
  __shared__ __attribute__((aligned(16))) uint8_t vsm[SLOTS];
  // (an array of its own, so that the compiler tells the copies apart)
  __shared__ __attribute__((aligned(16))) uint8_t ksm[KLDS ? SLOTS : 16];
  __shared__ __attribute__((aligned(16))) float mx_lds[2][32][NW];
  __shared__ __attribute__((aligned(16))) float m_lds[32][NW], l_lds[32][NW];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i32 = lane & 31;
  const int g = lane >> 5;
  const int G4 = lane >> 4, L16 = lane & 15;

  int rb = 0, unit = blockIdx.x;  // unit: (batch, KV head, part)
  if (p.nrb > 1) {
    // the row blocks that read the same keys run on one XCD (workgroup ids go
    // round-robin over the 8 XCDs), so that its L2 serves all but the first
    // (two row blocks, B8 4K: 51.4 -> 42.9 us BF16, 33.1 -> 22.7 FP8)
    const int n8 = p.B * p.Hkv * p.nsplit / 8 * 8 * p.nrb, L = blockIdx.x;
    if (L < n8) {
      rb = (L >> 3) % p.nrb;
      unit = (L >> 3) / p.nrb * 8 + (L & 7);
    } else {
      rb = (L - n8) % p.nrb;
      unit = n8 / p.nrb + (L - n8) / p.nrb;
    }
  }
  const int bkv = unit / p.nsplit, split = unit - bkv * p.nsplit;
  const int b = bkv / p.Hkv, hkv = bkv - b * p.Hkv;
  // output row (over [B][Hq][Sq]) of row r of this block of rows
  const int nrows = min(WROWS, p.R - rb * WROWS);
  const size_t orow0 = ((size_t)b * p.Hq + (size_t)hkv * p.G) * (size_t)p.Sq + (size_t)rb * WROWS;
  const int rowc = min(i32, nrows - 1);
  const int iq = (rb * WROWS + rowc) % p.Sq;
  const bool row_ok = i32 < nrows;
  const int Sk = p.Sk;
  const int limit = CAUSAL ? Sk - p.Sq + iq : Sk - 1;  // last key this row sees
  const int j0 = split * p.split_keys;
  const int j1 = min(j0 + p.split_keys, Sk);
  const int ntiles = (j1 - j0 + BC - 1) / BC;
  const float off = DT == DT_FP8 ? 8.0f : 0.0f;

  // ---- Q rows (MFMA B operand: lane holds row i32, k-half g)
  const uint8_t* qptr = p.q + (orow0 + rowc) * C::RB;
  bf16x8 qb16[DT == DT_BF16 ? NKQ : 1];
  i32x8 qf8[DT == DT_FP8 ? NKQ : 1];
  if constexpr (DT == DT_BF16) {
#pragma unroll
    for (int kk = 0; kk < NKQ; ++kk) qb16[kk] = *(const bf16x8*)(qptr + (16 * kk + 8 * g) * 2);
  } else {
#pragma unroll
    for (int kk = 0; kk < NKQ; ++kk) qf8[kk] = *(const i32x8*)(qptr + 64 * kk + 32 * g);
  }

  // ---- the part's K and V rows through buffer resources that hold just
  // them: rows beyond read as zero without touching memory (those keys are
  // masked), so every wave issues the same loads in every round and the
  // waits can count them.  The range check compares a lane's offset with the
  // resource's size minus the scalar offset, so scalar offsets stop at the
  // size (part_off), where every lane is out of range.
  const uint8_t* kg = p.k + ((size_t)bkv * (size_t)p.Sk_cap + (size_t)j0) * C::RB;
  const uint8_t* vg = p.v + ((size_t)bkv * (size_t)p.Sk_cap + (size_t)j0) * C::RB;
  const __amdgpu_buffer_rsrc_t krsrc =
      __builtin_amdgcn_make_buffer_rsrc((void*)kg, (short)0, (j1 - j0) * C::RB, BUF_DWORD3);
  const __amdgpu_buffer_rsrc_t vrsrc =
      __builtin_amdgcn_make_buffer_rsrc((void*)vg, (short)0, (j1 - j0) * C::RB, BUF_DWORD3);

  const uint32_t part_bytes = (uint32_t)(j1 - j0) * C::RB;
  auto part_off = [&](uint32_t byte) { return min(byte, part_bytes); };
  // this wave's first key of round c within the part
  const int wt = TPR == 1 ? 0 : wave >> 1;  // tile of the round
  auto first_key = [&](int c) { return c * (TPR * BC) + wave * UNIT; };

  // K of this wave's 64 keys straight into the MFMA A operand (block kb, lane:
  // key 32 kb + i32; bf16: 16 bytes at 32 kk + 16 g of the row; fp8: 32 bytes
  // at 64 kk + 32 g)
  using KOp = std::conditional_t<DT == DT_BF16, bf16x8, i32x8>;
  KOp kreg[NB][NKQ];
  uint8_t* const kslot = ksm + (KLDS ? wave * SLOT : 0);
  const int kswz = k_swz<DT, D>(i32);  // == k_swz(32 kb + i32)
  // the chunk swizzle of K rows repeats after every fourth 1 KB copy
  uint32_t koff_c[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = (i * 64 + lane) / C::NCH, pch = lane % C::NCH;
    koff_c[i] = (uint32_t)((r - i * (64 / C::NCH)) * C::RB + ((pch ^ k_swz<DT, D>(r)) << 4));
  }
  auto load_k = [&](int c) __attribute__((always_inline)) {
    if constexpr (KLDS) {
#pragma unroll
      for (int i = 0; i < LOADS; ++i) {
        const uint32_t soff = part_off((uint32_t)first_key(c) * C::RB + i * 1024);
        const uint32_t voff = koff_c[i & 3];
        uint8_t* ldst = kslot + i * 1024;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(krsrc, LDS_PTR(void, ldst), 16, voff, soff, 0, 0);
      }
      return;
    }
    const int krow = i32 * C::RB;
#pragma unroll
    for (int kb = 0; kb < NB; ++kb) {
      const int soff = (int)part_off((uint32_t)(first_key(c) + 32 * kb) * C::RB);
#pragma unroll
      for (int kk = 0; kk < NKQ; ++kk) {
        if constexpr (DT == DT_BF16) {
          kreg[kb][kk] = __builtin_bit_cast(
              bf16x8, __builtin_amdgcn_raw_buffer_load_b128(krsrc, krow + 32 * kk + 16 * g, soff, 0));
        } else {
          const i32x4 lo = __builtin_bit_cast(
              i32x4, __builtin_amdgcn_raw_buffer_load_b128(krsrc, krow + 64 * kk + 32 * g, soff, 0));
          const i32x4 hi = __builtin_bit_cast(
              i32x4, __builtin_amdgcn_raw_buffer_load_b128(krsrc, krow + 64 * kk + 32 * g + 16, soff, 0));
          kreg[kb][kk] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        }
      }
    }
  };
  // V of this wave's 64 keys into its LDS slot: slot byte s holds row s / RB
  // with the forward kernel's chunk swizzle, which repeats after every second
  // 1 KB copy, so two lane offsets serve all of them
  uint32_t voff_c[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = (i * 64 + lane) / C::NCH, pch = lane % C::NCH;
    voff_c[i] = (uint32_t)((r - i * (64 / C::NCH)) * C::RB + ((pch ^ v_swz<DT, D>(r)) << 4));
  }
  uint8_t* const vslot = vsm + wave * SLOT;
  auto stage_v = [&](int c) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const uint32_t soff = part_off((uint32_t)first_key(c) * C::RB + i * 1024);
      const uint32_t voff = voff_c[i & 1];
      uint8_t* ldst = vslot + i * 1024;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(vrsrc, LDS_PTR(void, ldst), 16, voff, soff, 0, 0);
    }
  };

  // ---- V^T operand addresses within the slot (as the forward kernel's)
  uint32_t vaddr[NDB];
  const uint32_t vla = (uint32_t)(size_t)LDS_PTR(const uint8_t, vslot);
  if constexpr (DT == DT_BF16) {
    const int vrow = 4 * (G4 >> 1) + (L16 >> 2);
    const int vcolb = (16 * (G4 & 1) + 4 * (L16 & 3)) * 2;
#pragma unroll
    for (int db = 0; db < NDB; ++db) {
      const int cb = 64 * db + vcolb;
      vaddr[db] = vla + vrow * C::RB + (((cb >> 4) ^ v_swz<DT, D>(vrow)) << 4) + (cb & 15);
    }
  } else {
    const int vrow = 4 * (G4 >> 1) + 8 * (L16 >> 3) + ((L16 >> 1) & 3);
    const int vcol = 16 * (G4 & 1) + 8 * (L16 & 1);
#pragma unroll
    for (int db = 0; db < NDB; ++db) {
      const int cb = 32 * db + vcol;
      vaddr[db] = vla + vrow * C::RB + (((cb >> 4) ^ v_swz<DT, D>(vrow)) << 4) + (cb & 15);
    }
  }

  f32x16 oacc[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) oacc[db] = f32x16{0.0f};
  float m_seen = -INFINITY;  // running maximum over the rounds done
  float m_wave = -INFINITY;  // this wave's anchor: what its l_part and O are relative to
  float l_part = 0.0f;
  const bool probe_row = PROBE && row_ok && b == p.pb && iq == p.pi && hkv * p.G + (rb * WROWS + rowc) / p.Sq == p.ph;

  // (in this order: what is needed first is waited for first)
  __builtin_amdgcn_sched_barrier(0);
  load_k(0);
  __builtin_amdgcn_sched_barrier(0);
  stage_v(0);
  __builtin_amdgcn_sched_barrier(0);
  // wait for Q here, where the copies behind it can be counted
#pragma unroll
  for (int kk = 0; kk < NKQ; ++kk) {
    if constexpr (DT == DT_BF16) asm volatile("" : "+v"(qb16[kk]));
    else asm volatile("" : "+v"(qf8[kk]));
  }
  const int nrounds = ONE ? 1 : (ntiles + TPR - 1) / TPR;
#pragma unroll 1
  for (int c = 0; c < nrounds; ++c) {
    const int kw0 = j0 + first_key(c);  // first key of this wave's unit
    const bool need_mask = (CAUSAL && kw0 + UNIT - 1 > Sk - p.Sq) || (kw0 + UNIT > j1);
    const int lim = min(limit, j1 - 1) - kw0 - 4 * g;

    // ---- S^T of this wave's keys, and their maximum for each row
    f32x16 sv[NB];
    if constexpr (KLDS) {
      // this round's K copies have landed once at most the V copies issued
      // after them are outstanding
      if constexpr (PROBE) wait_vmcnt<0>();
      else wait_vmcnt<LOADS>();
    }
#pragma unroll
    for (int kk = 0; kk < NKQ; ++kk)
#pragma unroll
      for (int kb = 0; kb < NB; ++kb) {
        if constexpr (KLDS) {
          const uint8_t* kr = kslot + (32 * kb + i32) * C::RB;
          if constexpr (DT == DT_BF16) {
            kreg[kb][kk] = *(const bf16x8*)(kr + (((2 * kk + g) ^ kswz) << 4));
          } else {
            const i32x4 lo = *(const i32x4*)(kr + (((4 * kk + 2 * g) ^ kswz) << 4));
            const i32x4 hi = *(const i32x4*)(kr + (((4 * kk + 2 * g + 1) ^ kswz) << 4));
            kreg[kb][kk] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
          }
        }
        if constexpr (DT == DT_BF16)
          sv[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kreg[kb][kk], qb16[kk], kk == 0 ? f32x16{0.0f} : sv[kb],
                                                           0, 0, 0);
        else
          sv[kb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
              kreg[kb][kk], qf8[kk], kk == 0 ? f32x16{0.0f} : sv[kb], 0, 0, 0, 0, 0, 0);
      }
    if constexpr (KLDS) {
      // K operands are read four MFMAs ahead, and all of them before the next
      // copy goes into the slot
      constexpr int RK = DT == DT_BF16 ? 1 : 2, NQK = NB * NKQ, AHEAD = NQK < 4 ? NQK : 4;
      __builtin_amdgcn_sched_group_barrier(SG_DS_READ, RK * AHEAD, 0);
#pragma unroll
      for (int i = 0; i < NQK; ++i) {
        __builtin_amdgcn_sched_group_barrier(SG_MFMA, 1, 0);
        if (i + AHEAD < NQK) __builtin_amdgcn_sched_group_barrier(SG_DS_READ, RK, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!ONE) load_k(c + 1);
    settle_unit(sv);
    // keys beyond the row's limit or the cache
    if (need_mask) mask_unit(sv, lim, -INFINITY);
    if constexpr (PROBE) {
      if (probe_row) {
#pragma unroll
        for (int kb = 0; kb < NB; ++kb)
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            const int key = kw0 + 32 * kb + 8 * (j >> 2) + 4 * g + (j & 3);
            if (key < j1) p.s_out[key] = sv[kb][j];
          }
      }
    }
    float ma, mb;
    with_partner(unit_max(sv), ma, mb);
    const float um = __builtin_fmaxf(ma, mb);
    if (g == 0) mx_lds[c & 1][i32][wave] = um;
    // (the two copies of mx_lds alternate, so a wave that runs ahead writes
    // the other one: every wave has read this one before the next barrier)
    lds_barrier();
    float anchor = m_seen;
    {
      const float* mx = &mx_lds[c & 1][i32][0];
      const f32x4 x = *(const f32x4*)mx;
      const float t0 = __builtin_fmaxf(x[0], x[1]), t1 = __builtin_fmaxf(x[2], x[3]);
      m_seen = max3(m_seen, t0, t1);
      anchor = TPR == 2 && wt == 0 ? __builtin_fmaxf(anchor, t0) : m_seen;
    }
    // a row that has seen no key yet keeps m = -inf, l = 0, O = 0
    const float alpha = anchor == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f((m_wave - anchor) * p.c1);
    const float m_use = anchor == -INFINITY ? 0.0f : anchor;
    m_wave = anchor;

    // ---- weights (in place), row sum
    uint32_t wpk[NB][8];
    constexpr bool PACKED = mode_lattice(MODE);
    if constexpr (PACKED) {
      const float nbk = __builtin_fmaf(-m_use, p.ck, (float)(1 << mode_order(MODE)) * off);
#pragma unroll
      for (int kb = 0; kb < NB; ++kb)
#pragma unroll
        for (int j = 0; j < 16; ++j) sv[kb][j] = __uint_as_float(sq_pre<MODE>(sv[kb][j], p.ck, nbk));
      if (need_mask) {
        if constexpr (mode_narrow(MODE)) {
          // as the forward kernel: one max lifts exactly the masked keys
          const float lift = __uint_as_float(0x4B3F0000u | sq_masked<MODE>());
#pragma unroll
          for (int kb = 0; kb < NB; ++kb)
#pragma unroll
            for (int j = 0; j < 16; ++j) sv[kb][j] = max3(sv[kb][j], lift, lift);
        } else {
          mask_unit(sv, lim, __uint_as_float(sq_masked<MODE>()));
        }
      }
      float a[4] = {l_part * alpha, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int kb = 0; kb < NB; ++kb)
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          wpk[kb][q] = sq_pack<MODE>(__float_as_uint(sv[kb][2 * q]), __float_as_uint(sv[kb][2 * q + 1]));
          a[q & 3] = dot2_ones(wpk[kb][q], a[q & 3]);
        }
      l_part = (a[0] + a[1]) + (a[2] + a[3]);
    } else {
      const float nb1 = __builtin_fmaf(-m_use, p.c1, off);
#pragma unroll
      for (int kb = 0; kb < NB; ++kb)
#pragma unroll
        for (int j = 0; j < 16; ++j) sv[kb][j] = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[kb][j], p.c1, nb1));
      float a[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) a[i] = NB == 2 ? sv[0][i] + sv[NB - 1][i] : sv[0][i];
#pragma unroll
      for (int w = 8; w >= 1; w >>= 1)
#pragma unroll
        for (int i = 0; i < w; ++i) a[i] = a[i] + a[i + w];
      l_part = l_part * alpha + a[0];
    }
    if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int j = 0; j < 16; ++j) oacc[db][j] *= alpha;
    }

    // ---- P in the operand type: bf16 as 16-key operands, fp8 as one 64-key
    // operand (a unit of 32 keys: P = 0 and V = 0 in its other half)
    bf16x8 pb[2 * NB];
    i32x8 pf = {0, 0, 0, 0, 0, 0, 0, 0};
    if constexpr (DT == DT_BF16) {
#pragma unroll
      for (int ks = 0; ks < 2 * NB; ++ks) {
        const int kb = ks >> 1;
        if constexpr (PACKED) {
          const int q0 = 4 * (ks & 1);
          pb[ks] =
              __builtin_bit_cast(bf16x8, u32x4{wpk[kb][q0], wpk[kb][q0 + 1], wpk[kb][q0 + 2], wpk[kb][q0 + 3]});
        } else {
#pragma unroll
          for (int r = 0; r < 8; ++r) pb[ks][r] = (__bf16)sv[kb][8 * (ks & 1) + r];
        }
      }
    } else {
#pragma unroll
      for (int w8 = 0; w8 < 4 * NB; ++w8) {
        const int kb = w8 >> 2, j4 = 4 * (w8 & 3);
        if constexpr (PACKED) {
          i16x2 word = __builtin_bit_cast(i16x2, wpk[kb][j4 / 2]);
          word = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(word, __builtin_bit_cast(bf16x2, wpk[kb][j4 / 2]), 1.0f,
                                                           false);
          word = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(word, __builtin_bit_cast(bf16x2, wpk[kb][j4 / 2 + 1]),
                                                           1.0f, true);
          pf[w8] = __builtin_bit_cast(int, word);
        } else {
          uint32_t word = __float_as_uint(sv[kb][j4]);
          word = __builtin_amdgcn_cvt_pk_fp8_f32(sv[kb][j4], sv[kb][j4 + 1], word, false);
          word = __builtin_amdgcn_cvt_pk_fp8_f32(sv[kb][j4 + 2], sv[kb][j4 + 3], word, true);
          pf[w8] = (int)word;
        }
      }
    }
    if constexpr (PROBE) {
      if (probe_row) {
#pragma unroll
        for (int kb = 0; kb < NB; ++kb)
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            const int key = kw0 + 32 * kb + 8 * (j >> 2) + 4 * g + (j & 3);
            if (key < j1 && key <= limit) {
              uint32_t bits;
              if constexpr (DT == DT_BF16) {
                const u32x4 pw4 = __builtin_bit_cast(u32x4, pb[2 * kb + (j >> 3)]);
                bits = (pw4[(j & 7) >> 1] >> (16 * (j & 1))) & 0xFFFFu;
              } else {
                bits = ((uint32_t)pf[4 * kb + (j >> 2)] >> (8 * (j & 3))) & 0xFFu;
              }
              p.w_out[key] = PACKED ? __uint_as_float(((wpk[kb][j >> 1] >> (16 * (j & 1))) & 0xFFFFu) << 16)
                                    : sv[kb][j];
              p.p_out[key] = bits;
            }
          }
      }
    }

    // ---- O^T += V^T P^T over this wave's keys: its copy of V has landed
    // once at most the next round's K loads, issued after it, are
    // outstanding (the probe's stores count too, so the probe waits for
    // all)
    if constexpr (PROBE || ONE) wait_vmcnt<0>();
    else wait_vmcnt<KLOADS>();
#pragma unroll
    for (int db = 0; db < NDB; db += 2) {
      if constexpr (DT == DT_BF16) {
        i32x2v r[8 * NB];
        read_v16<C::RB>(r, vaddr[db], vaddr[db + 1]);
#pragma unroll
        for (int ks = 0; ks < 2 * NB; ++ks)
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int r0 = 4 * NB * h + 2 * ks;
            const bf16x8 vop = __builtin_bit_cast(bf16x8, __builtin_shufflevector(r[r0], r[r0 + 1], 0, 1, 2, 3));
            oacc[db + h] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vop, pb[ks], oacc[db + h], 0, 0, 0);
          }
      } else {
        i32x2v r[4 * NB];
        read_v8<C::RB>(r, vaddr[db], vaddr[db + 1]);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int r0 = 2 * NB * h;
          const i32x4 lo = __builtin_shufflevector(r[r0], r[r0 + 1], 0, 1, 2, 3);
          i32x4 hi = {0, 0, 0, 0};
          if constexpr (NB == 2) hi = __builtin_shufflevector(r[r0 + 2], r[r0 + 3], 0, 1, 2, 3);
          const i32x8 vop = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
          oacc[db + h] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(vop, pf, oacc[db + h], 0, 0, 0, 0, 0, 0);
        }
      }
    }
    // (the slot has been read: the reads are waited for above)
    if constexpr (!ONE) stage_v(c + 1);
  }
  // every copy has landed (the last round's went to no key) and every wave is
  // done with its V slots before they are reused for the reduction
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  // ---- the waves' partial sums, each relative to its own anchor, added up
  // through LDS in one pass (chunks of four columns, XOR-swizzled by row).
  // With 32 rows in two passes of 16, a barrier between them, a full block of
  // rows took 0.7..0.9 us longer; bringing the sums to one anchor in registers
  // beforehand costs 0.3 us where O sits in accumulation registers.
  {
    float la, lb;
    with_partner(l_part, la, lb);
    if (g == 0) {
      m_lds[i32][wave] = m_wave;
      l_lds[i32][wave] = la + lb;
    }
  }
  uint8_t* const upper = KLDS ? ksm : vsm + RBYTES;
  if (row_ok) {
    const int ri = i32 & (RHALF - 1);
    float* red = (float*)(i32 < RHALF ? vsm : upper) + (wave * RHALF + ri) * D;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int jq = 0; jq < 4; ++jq)
        *(f32x4*)(red + 4 * ((8 * db + 2 * jq + g) ^ ri)) =
            f32x4{oacc[db][4 * jq], oacc[db][4 * jq + 1], oacc[db][4 * jq + 2], oacc[db][4 * jq + 3]};
  }
  lds_barrier();
  for (int r0 = 0; r0 < nrows; r0 += RHALF) {
    const float* red = (const float*)(r0 == 0 ? vsm : upper);
#pragma unroll
    for (int i = 0; i < RHALF * (D / 4) / (NW * 64); ++i) {
      const int idx = i * NW * 64 + tid, rr = idx / (D / 4), ch = idx % (D / 4), r = r0 + rr;
      if (r >= nrows) continue;
      const f32x4 mw = *(const f32x4*)m_lds[r], lw = *(const f32x4*)l_lds[r];
      const float m = __builtin_fmaxf(__builtin_fmaxf(mw[0], mw[1]), __builtin_fmaxf(mw[2], mw[3]));
      float l = 0.0f;
      f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        // (one tile a round: one anchor, and no exponential: 1, but NaN for an
        // infinite anchor and 0 for a row without one, as the exponential has it)
        const float fw = TPR == 1 ? 1.0f + (mw[w] - m) : __builtin_amdgcn_exp2f((mw[w] - m) * p.c1);
        const float f = mw[w] == -INFINITY ? 0.0f : fw;
        l += f * lw[w];
        const f32x4 o = *(const f32x4*)(red + (w * RHALF + rr) * D + 4 * (ch ^ rr));
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += f * o[e];
      }
      const size_t orow = orow0 + r;
      if (p.nsplit == 1) {
        const float inv = p.vd / l;
        uint32_t w[2];
#pragma unroll
        for (int e = 0; e < 2; ++e)
          w[e] = (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)(acc[2 * e] * inv)) |
                 ((uint32_t)__builtin_bit_cast(uint16_t, (__bf16)(acc[2 * e + 1] * inv)) << 16);
        *(u32x2*)(p.o + orow * (size_t)D + 4 * ch) = u32x2{w[0], w[1]};
        if (p.lse && ch == 0) p.lse[orow] = 0.69314718055994531f * (m * p.c1 + log2f(l) - off);
      } else {
        *(f32x4*)(p.part_o + (orow * (size_t)p.nsplit + (size_t)split) * (size_t)D + 4 * ch) = acc;
        if (ch == 0) *(f32x2*)(p.part_ml + (orow * (size_t)p.nsplit + (size_t)split) * 2) = f32x2{m, l};
      }
    }
  }
}

struct MergeParams {
  const float* part_o;
  const float* part_ml;
  uint16_t* o;
  float* lse;
  int rows, nsplit;
  float c1, vd, off;
};

template <int D>
__global__ __launch_bounds__(256) void attn_decode_merge(MergeParams p) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= p.rows) return;
  merge_row<D>(p.part_ml + (size_t)row * p.nsplit * 2, p.part_o + (size_t)row * p.nsplit * D, p.nsplit, p.c1, p.vd,
               p.off, p.o + (size_t)row * D, p.lse ? p.lse + row : nullptr);
}

template <int DT, int D, int UNIT, bool ONE, bool KLDS, bool CAUSAL, int MODE, bool PROBE>
hipError_t launch_dec_kernel(const DecParams& p, hipStream_t st) {
  const unsigned grid = (unsigned)(p.B * p.Hkv * p.nrb * p.nsplit);
  hipLaunchKernelGGL((attn_decode_kernel<DT, D, UNIT, ONE, KLDS, CAUSAL, MODE, PROBE>), dim3(grid), dim3(NW * 64), 0,
                     st, p);
  return hipGetLastError();
}

template <int DT, int D, bool CAUSAL, int MODE, bool PROBE>
hipError_t launch_dec_one(const DecParams& p, hipStream_t st) {
  if (p.unit == 32) {
    return p.split_keys == BC ? launch_dec_kernel<DT, D, 32, true, true, CAUSAL, MODE, PROBE>(p, st)
                              : launch_dec_kernel<DT, D, 32, false, true, CAUSAL, MODE, PROBE>(p, st);
  }
  if constexpr (DT == DT_BF16 && D == 128) {
    if (!p.k_lds) return launch_dec_kernel<DT, D, 64, false, false, CAUSAL, MODE, PROBE>(p, st);
  }
  return launch_dec_kernel<DT, D, 64, false, true, CAUSAL, MODE, PROBE>(p, st);
}

template <int DT, int D, bool CAUSAL, bool PROBE>
hipError_t launch_dec_mode(const DecParams& p, int mode, hipStream_t st) {
  switch (mode) {
    case MODE_EXACT: return launch_dec_one<DT, D, CAUSAL, MODE_EXACT, PROBE>(p, st);
    case 1: return launch_dec_one<DT, D, CAUSAL, 1, PROBE>(p, st);
    case 3: return launch_dec_one<DT, D, CAUSAL, 3, PROBE>(p, st);
    case 5: return launch_dec_one<DT, D, CAUSAL, 5, PROBE>(p, st);
    default: break;
  }
  if constexpr (DT == DT_FP8) {
    switch (mode) {
      case 2: return launch_dec_one<DT, D, CAUSAL, 2, PROBE>(p, st);
      case 4: return launch_dec_one<DT, D, CAUSAL, 4, PROBE>(p, st);
      case 6: return launch_dec_one<DT, D, CAUSAL, 6, PROBE>(p, st);
      default: break;
    }
  }
  return hipErrorInvalidValue;
}

template <bool PROBE>
hipError_t launch_dec_any(const DecParams& p, int dtype, int d, int causal, int mode, hipStream_t st) {
  if (dtype == ATTN_BF16) {
    if (d == 128)
      return causal ? launch_dec_mode<DT_BF16, 128, true, PROBE>(p, mode, st)
                    : launch_dec_mode<DT_BF16, 128, false, PROBE>(p, mode, st);
    return causal ? launch_dec_mode<DT_BF16, 64, true, PROBE>(p, mode, st)
                  : launch_dec_mode<DT_BF16, 64, false, PROBE>(p, mode, st);
  }
  if (d == 128)
    return causal ? launch_dec_mode<DT_FP8, 128, true, PROBE>(p, mode, st)
                  : launch_dec_mode<DT_FP8, 128, false, PROBE>(p, mode, st);
  return causal ? launch_dec_mode<DT_FP8, 64, true, PROBE>(p, mode, st)
                : launch_dec_mode<DT_FP8, 64, false, PROBE>(p, mode, st);
}

hipError_t launch_merge(const DecParams& dp, int dtype, int d, hipStream_t st) {
  MergeParams mp;
  mp.part_o = dp.part_o;
  mp.part_ml = dp.part_ml;
  mp.o = dp.o;
  mp.lse = dp.lse;
  mp.rows = dp.B * dp.Hq * dp.Sq;
  mp.nsplit = dp.nsplit;
  mp.c1 = dp.c1;
  mp.vd = dp.vd;
  mp.off = dtype == ATTN_FP8_E4M3 ? 8.0f : 0.0f;
  const unsigned grid = (unsigned)((mp.rows + 3) / 4);
  if (d == 128) hipLaunchKernelGGL(attn_decode_merge<128>, dim3(grid), dim3(256), 0, st, mp);
  else hipLaunchKernelGGL(attn_decode_merge<64>, dim3(grid), dim3(256), 0, st, mp);
  return hipGetLastError();
}

// Built-in workspace of attn_decode_noalloc: the parts' (m, l, O) of one
// decode call, for callers that cannot allocate.  Each GPU the library runs
// on holds its own copy until the process ends.  In host code the name is
// only a stand-in for the device address: the address each device uses is
// looked up once per device (scratch_address) and only that is passed on.
constexpr size_t SCRATCH_BYTES = (size_t)16 << 20;
static __device__ __align__(256) uint8_t scratch[SCRATCH_BYTES];
}  // namespace

namespace h15 {

size_t scratch_capacity() { return SCRATCH_BYTES; }

int scratch_address(void* stream, void** ptr) {
  constexpr int MAX_DEVICES = 64;
  static std::mutex mu;
  static void* addr[MAX_DEVICES] = {};
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return 1;
  if (stream) {
    // the kernels run on the stream's device: its buffer is the one to use,
    // and it is looked up with the current device, so the two must agree
    hipDevice_t sdev = -1;
    if (hipStreamGetDevice((hipStream_t)stream, &sdev) != hipSuccess) return 1;
    if (sdev != dev) return 2;
  }
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    // with the device current: this device's copy of the array
    void* a = nullptr;
    if (hipGetSymbolAddress(&a, HIP_SYMBOL(scratch)) != hipSuccess || !a) return 1;
    addr[dev] = a;
  }
  *ptr = addr[dev];
  return 0;
}

int launch_decode(const DecParams& p, int dtype, int d, int causal, int mode, void* stream, bool probe) {
  hipStream_t st = (hipStream_t)stream;
  hipError_t e = probe ? launch_dec_any<true>(p, dtype, d, causal, mode, st)
                       : launch_dec_any<false>(p, dtype, d, causal, mode, st);
  if (e == hipSuccess && p.nsplit > 1) e = launch_merge(p, dtype, d, st);
  return e == hipSuccess ? 0 : 1;
}

}  // namespace h15
