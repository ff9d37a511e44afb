// Device code that the forward kernels (h15attn.hip) and the decode kernels
// (h15decode.hip) share: operand types, tile layouts and swizzles, the
// lattice weights, masking, the transposing LDS reads and the small
// reductions.  Everything has internal linkage; each file includes it once.
#ifndef H15ATTN_DEVICE_H
#define H15ATTN_DEVICE_H

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "attn_params.h"
#include "h15attn.h"

namespace {

using namespace h15;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x2v __attribute__((__vector_size__(2 * sizeof(int))));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short i16x2 __attribute__((ext_vector_type(2)));

#define LDS_PTR(T, p) ((__attribute__((address_space(3))) T*)(p))

enum { DT_BF16 = 0, DT_FP8 = 1 };

// Waves per workgroup in the default layout: 4 for FP8 (two workgroups
// share a CU, so one's barrier and prologue stalls overlap the other's
// work), 8 for BF16 (whose double-buffered tiles at d = 128 leave LDS for
// only one workgroup per CU; the compact layout, Cfg below, has 4).
template <int DT>
constexpr int waves_per_group() {
  return DT == DT_FP8 ? 4 : 8;
}
// word 3 of a raw buffer resource on CDNA (32-bit data format, no swizzle)
constexpr int BUF_DWORD3 = 0x00020000;
constexpr float H15_MAGIC = 12582912.0f;  // 0x4B400000 = 2^23 + 2^22
// top half of bits(1.0) in both 16-bit lanes
constexpr uint32_t ONE_BITS16X2 = 0x3F803F80u;

// Kernel weight modes (attn_params.h): the order k of a lattice mode, and its
// clamp form.
constexpr int mode_order(int mode) { return (mode + 1) / 2; }
constexpr bool mode_lattice(int mode) { return mode != MODE_EXACT && mode != MODE_ROWMAX_POT; }
constexpr bool mode_narrow(int mode) { return mode_lattice(mode) && mode % 2 == 0; }

// Layouts of a forward workgroup (which one a call takes is decided on the
// host, attn_api.cpp):
//   LAY_WIDE    waves_per_group waves of 32 query rows each, one key tile a step;
//   LAY_COMPACT BF16: 4 waves and at most 80 KB of LDS, so two groups share a
//               CU and one's prologue, barriers and epilogue overlap the
//               other's work; at d = 128 that means single-buffered tiles;
//   LAY_PAIRED  8 waves for 128 query rows: waves w and w + 4 have the same
//               rows and take the even and the odd key tiles, half a step
//               apart, each four with single-buffered tiles of their own.
template <int DT, int D, int LAY = LAY_WIDE>
struct Cfg {
  static constexpr int EB = DT == DT_BF16 ? 2 : 1;  // operand bytes
  static constexpr int RB = D * EB;                 // bytes per K/V row
  static constexpr int NCH = RB / 16;               // 16-byte chunks per row
  static constexpr int TILE = BC * RB;              // bytes of one K (or V) tile
  static constexpr int BUF = 2 * TILE;              // K then V
  static constexpr int CHUNKS = BC * NCH;           // 16-byte chunks per tile
  static constexpr int NW = LAY == LAY_COMPACT ? 4 : LAY == LAY_PAIRED ? 8 : waves_per_group<DT>();  // waves per group
  static constexpr int NPAR = LAY == LAY_PAIRED ? 2 : 1;  // waves with the same rows
  static constexpr int RW = NW / NPAR;                    // waves that share a tile
  static constexpr int BR = RW * WROWS;                   // query rows per workgroup
  // K/V tile buffers: two (the copy of tile t + 1 overlaps tile t), or one
  // when two would not let two compact groups share a CU's 160 KB of LDS
  static constexpr int NSTAGE = LAY == LAY_PAIRED || (LAY == LAY_COMPACT && 2 * BUF > 80 * 1024) ? 1 : 2;
  static_assert(CHUNKS % (RW * 64) == 0, "tile/staging mismatch");
  static_assert(BR == (LAY != LAY_WIDE ? FWD_ROWS_SMALL : DT == DT_FP8 ? FWD_ROWS_FP8 : FWD_ROWS_BF16),
                "row block of attn_params.h");
};

// Bank-spreading XOR swizzles of the 16-byte chunks of a row.  K rows are read
// as the MFMA A operand (one chunk of 32 consecutive rows per instruction);
// V rows through the transposing reads (4 rows x 2 chunks for bf16, 8 rows x
// 1 chunk for fp8 per 16 lanes).  An fp8 row is 128 bytes, half the banks'
// width, so rows r and r + 1 start on different bank halves; the K swizzle
// then varies with r / 2, so that 16 consecutive rows reading one logical
// chunk cover every bank once (with r % NCH, rows r and r + 8 shared banks;
// the counter read 2,080 conflict cycles per wave at d = 128, now zero).
template <int DT, int D>
__device__ __forceinline__ int k_swz(int row) {
  using C = Cfg<DT, D>;
  if constexpr (DT == DT_BF16) return row % C::NCH;
  else return (row >> 1) % C::NCH;
}
template <int DT, int D>
__device__ __forceinline__ int v_swz(int row) {
  using C = Cfg<DT, D>;
  if constexpr (DT == DT_BF16) return ((C::NCH >= 16 ? 4 : 2) * (row & 3)) % C::NCH;
  else return ((row & 3) | (((row >> 3) & 1) << 2)) % C::NCH;
}

// Weight of one score, S(Q_{2^-k}(x)) with k = mode_order(MODE) (App. B.1
// "Implementation" for k = 1, App. B.2 "Exponential-map ablation" for k = 2,
// 3): y = 2^k x = fma(s, 2^k c1, nb), clamp at -126 * 2^k, RNE add of
// 0x4B400000 (n = RNE(y) lands in the low mantissa bits), left shift by
// 23 - k (the low k bits of n become the top mantissa bits, the rest the
// exponent), plus the bits of 1.0, all modulo 2^32.
//
// Such a weight has at most k <= 3 mantissa bits, so the low 16 bits of its
// FP32 pattern are zero and its top 16 bits, (n << (7 - k)) + 0x3F80 modulo
// 2^16, are its exact BF16 pattern.  The kernel finishes the weights two at
// a time in the 16-bit lanes of one register: the row sum takes one
// two-element dot product per pair, and the pair is already a BF16 operand
// (or one packed conversion away from FP8).
//
// sq_pre: the 32-bit value whose low half carries n: bits(max(y, -126 2^k) +
// magic), or for the narrow clamp bits(y + magic) (the magic's low half is
// zero, so the low half is n modulo 2^16).
template <int MODE>
__device__ __forceinline__ uint32_t sq_pre(float s, float ck, float nbk) {
  constexpr int K = mode_order(MODE);
  const float y = __builtin_fmaf(s, ck, nbk);
  if constexpr (mode_narrow(MODE)) return __float_as_uint(y + H15_MAGIC);
  else return __float_as_uint(__builtin_fmaxf(y, -126.0f * (float)(1 << K)) + H15_MAGIC);
}

// The BF16 weights of two keys in one word (u0 in the low lane): the low
// halves of their sq_pre values, the narrow clamp max(n, -126 2^k) on int16
// lanes (n is then n itself: the launcher selects the narrow mode only when
// every |y| is provably below 2^15), and n 2^(7-k) + 0x3F80 per lane modulo
// 2^16 in one packed multiply-add.
template <int MODE>
__device__ __forceinline__ uint32_t sq_pack(uint32_t u0, uint32_t u1) {
  constexpr int K = mode_order(MODE);
  uint32_t x = __builtin_amdgcn_perm(u1, u0, 0x05040100u);
  if constexpr (mode_narrow(MODE)) {
    constexpr short lo = (short)(-126 * (1 << K));
    x = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(i16x2, x), i16x2{lo, lo}));
  }
  // the multiplier is an inline constant read from its low half in both
  // lanes (op_sel_hi 0); the addend comes from a scalar register
  uint32_t r;
  asm("v_pk_mad_u16 %0, %1, %2, %3 op_sel_hi:[1,0,1]" : "=v"(r) : "v"(x), "n"(1 << (7 - K)), "s"(ONE_BITS16X2));
  return r;
}

// sq_pre value of a masked key: its packed weight is +0.  n = 385 * 2^k gives
// n 2^(7-k) = 0xC080 = -0x3F80 modulo 2^16, and lies above the narrow clamp.
template <int MODE>
constexpr uint32_t sq_masked() {
  return 385u << mode_order(MODE);
}
// (0x4B3F0000 | sq_masked) = 0x1.8p23 - 2^16 + sq_masked lies below
// 0x1.8p23 - 2^15 for every mode
static_assert((385u << 3) < (1u << 15), "the lift stays below every narrow-mode t");

// acc plus the two weights of a packed pair: one dot product with (1, 1)
__device__ __forceinline__ float dot2_ones(uint32_t w, float acc) {
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w), ones, acc, false);
}

// x, or y where key offset C lies beyond this lane's last valid offset lim.
// Compare and select go through VCC together (C as an immediate): written
// as plain C the compiler keeps all 64 masks of a tile live in scalar
// registers at once.
template <int C>
__device__ __forceinline__ float select_beyond(int lim, float x, float y) {
  float r;
  // volatile: keeps the masking inside the branch that needs it
  asm volatile("v_cmp_gt_i32 vcc, %1, %2\n\tv_cndmask_b32 %0, %3, %4, vcc"
               : "=v"(r)
               : "n"(C), "v"(lim), "v"(x), "v"(y)
               : "vcc");
  return r;
}
// This lane's value and that of lane i ^ 32 (in an order that depends on the
// lane), exchanged on the VALU rather than through LDS.
__device__ __forceinline__ void with_partner(float x, float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}

// Compile-time loop: f(integral_constant<int, I>) for I in [B, E).
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// Transposing LDS reads written as inline asm.  The compiler's wait counting
// would make the intrinsic forms wait for every LDS copy in flight (it cannot
// tell that those copies land in other buffers); here the caller waits for
// the reads itself with lds_wait, which also orders the uses after the wait.
template <int OFF>
__device__ __forceinline__ i32x2v ds_read_tr8(uint32_t addr) {
  static_assert(OFF >= 0 && OFF < 65536, "ds offset");
  i32x2v r;
  asm volatile("ds_read_b64_tr_b8 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF));
  return r;
}
template <int OFF>
__device__ __forceinline__ i32x2v ds_read_tr16(uint32_t addr) {
  static_assert(OFF >= 0 && OFF < 65536, "ds offset");
  i32x2v r;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF));
  return r;
}
// Wait until at most N LDS operations of this wave are outstanding (they
// complete in order), then hand x on as produced after the wait.
template <int N, typename T>
__device__ __forceinline__ void lds_wait(T& x) {
  static_assert(N >= 0 && N < 16, "lgkmcnt range");
  asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(x) : "n"(N));
}

// s_waitcnt for vmcnt <= N only (gfx9 encoding: vmcnt in bits 3:0 and 15:14;
// expcnt 6:4 and lgkmcnt 11:8 at their maxima, so not waited for)
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
  asm volatile("" ::: "memory");
}

// Barrier that makes this workgroup's LDS writes visible and leaves loads
// from memory in flight (fences, also those of LDS alone, wait for the copies
// into LDS).
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// v_max3_f32 directly: fmaxf on matrix-core results would first canonicalize
// every input (one extra instruction per score).
__device__ __forceinline__ float max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

}  // namespace

#endif  // H15ATTN_DEVICE_H
