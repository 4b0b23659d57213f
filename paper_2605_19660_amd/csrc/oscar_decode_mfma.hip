// oscar_decode_attn, matrix-core path for gfx950 (v_mfma_f32_16x16x32_f16).
//
// Why matrix cores: at 86 bytes per token and kv head, 70 % of 8 TB/s leaves about 600
// plain-ALU lane operations per token and kv head on 256 CUs; the two GQA-batched
// contractions alone (q K^T and P V, 4..8 query heads per kv head) need 1024..2048 fused
// multiply-adds.  Everything that is a contraction therefore runs on MFMA; unpacking,
// softmax and scale folding stay on the vector ALU.
//
//   logit[h][t] = n_t * ( sum_j (Q_h[h][j] Delta_k[j]) c_k[t][j]  -  sum_j Q_h[h][j] Delta_k[j] z_k[j] )
//   out[h][c]   = sum_t (p[h][t] Delta_v[t][G(c)]) c_v[t][c]  -  sum_t p[h][t] Delta_v[t][G(c)] z_v[t][G(c)]
// (logits of App. "Implementation Details", "Overall Design"; dequantization of Eq. 3-4.)
//
// Exactness devices:
//  * Codes become fp16 operands with one AND per register and no offset: a code parked at
//    bit offset s of an fp16 lane's mantissa (exponent field zero) is the subnormal number
//    c * 2^s * 2^-24, and the MFMA keeps fp16 subnormals.  2^s is divided out of the other
//    operand.  Offsets stay near the top of the mantissa (see slot_bitpos).
//  * The other operand (Q_h*Delta_k, resp. p*Delta_v) is carried as fp16 hi + lo limbs in two
//    rows of the 16-row MFMA tile (rows are otherwise idle for GQA <= 8): hi + lo equals the
//    fp32 product to ~2^-21, the MFMA's products with the codes are exact and accumulation
//    is fp32.  The limbs come from packed fp16 arithmetic on a multiplicand split once
//    (mul_limbs_packed; mul_split_hi_lo is the mixed-precision form it replaced, still built
//    with OSCAR_LIMBS_PACKED = 0).
//  * Zero-points are subtracted analytically in fp32 (the two right-hand sums above).
//
// Work decomposition: grid (split, kv head, sequence); 4 waves per workgroup (8 in launches that leave
// compute units to spare, see eight_waves_built), every wave
// owns whole pages (no barriers in the page loop) and keeps its own online-softmax state;
// the wave states and the workgroup's slice of the 16-bit residual tokens (plain ALU code,
// the window is dealt to the splits in multiples of 16 tokens) are merged through LDS at
// the end.
// Tile roles: q K^T uses M = query-head limb rows, N = 16 tokens, K = 128 channels;
// P V uses M = query-head limb rows, N = 16 channels, K = 128 tokens.  A lane of the logit
// tile is (token n, head group q4), which is also the lane that owns the 8-token operand
// vector (k-step n/4, quarter n%4) of the P V contraction: probabilities go to LDS as
// 16-byte vectors and come back as MFMA A-operands without any shuffle.
#include <atomic>

#include "oscar_decode_common.h"

#include <type_traits>

// This file is compiled six times: as it stands for the integer zero-point of Eq. 3-4, and through
// oscar_decode_mfma_zpmin.hip with OSCAR_MFMA_ZPMIN = 1 for the float zero-point form; the
// zero-point form is a compile-time constant of the kernel (no branches in the page loop), and
// the two sets of variants compile side by side.
#ifndef OSCAR_MFMA_ZPMIN
#define OSCAR_MFMA_ZPMIN 0
#endif
// and both forms once more with OSCAR_MFMA_META32 = 1: step sizes, zero-points and norms stored
// as fp32 (oscar_decode_mfma_meta32.hip, oscar_decode_mfma_meta32_zpmin.hip).
#ifndef OSCAR_MFMA_META32
#define OSCAR_MFMA_META32 0
#endif
// OSCAR_MFMA_STEP = 1 (oscar_decode_step.hip, oscar_decode_step_zpmin.hip): the decode step's kernel,
// which appends the step's new token on the way (fp16 metadata).
#ifndef OSCAR_MFMA_STEP
#define OSCAR_MFMA_STEP 0
#endif
#include "oscar_rowops.h"
#if OSCAR_MFMA_STEP
#include "oscar_append_kernel.h"
#pragma clang fp contract(fast)
#endif

// A prefetch that refills registers in place must not be moved, by the instruction scheduler,
// above the last read of the registers' old contents: the arriving data then lands in other
// registers and is copied home, and the copy waits for a load that was only just issued.
// The fence keeps vector-ALU and vector-memory instructions on their side of it; scalar,
// matrix and LDS instructions may still cross.
#ifndef OSCAR_PREFETCH_FENCE_MASK
#define OSCAR_PREFETCH_FENCE_MASK 0x38C
#endif
#define OSCAR_PREFETCH_FENCE() __builtin_amdgcn_sched_barrier(OSCAR_PREFETCH_FENCE_MASK)

#ifndef OSCAR_DECODE_PRIORITY
#define OSCAR_DECODE_PRIORITY 1
#endif

// Phase time stamps (measurement aid, off in the library proper: build.py --stamps makes a
// second library with them, phase_profile.py runs it).  Lane 0 of every wave of the first and
// the last four workgroups of the grid writes the constant-rate counter (100 MHz, the same on
// every CU) at the phase boundaries below; indices are masked, the array is fixed.
#ifdef OSCAR_DECODE_STAMPS
namespace {
__device__ unsigned long long g_stamps[8][4][32];
}
#define OSCAR_STAMP(i)                                                                  \
  do {                                                                                  \
    if (stamp_on && wave < 4 && lane == 0) g_stamps[stamp_slot & 7][wave & 3][(i) & 31] = wall_clock64(); \
  } while (0)
#else
#define OSCAR_STAMP(i)
#endif

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// wave-local LDS hand-off: LDS operations of one wave execute in order; this only stops
// the compiler from moving accesses across the hand-off point.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Reductions over the 16 lanes of a DPP row (= one head group): xor-1 and xor-2 inside
// quads, then the two mirrors; every lane ends with the same bits.
template <int CTRL> __device__ __forceinline__ float dpp_mov(float v) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float row16_max(float v) {
  v = fmaxf(v, dpp_mov<0xB1>(v));   // quad_perm [1,0,3,2]
  v = fmaxf(v, dpp_mov<0x4E>(v));   // quad_perm [2,3,0,1]
  v = fmaxf(v, dpp_mov<0x141>(v));  // row_half_mirror
  v = fmaxf(v, dpp_mov<0x140>(v));  // row_mirror
  return v;
}
// The same reductions with the permutation folded into the max itself, for the page loop
// (the compiler's form is a move, a canonicalizing max and the max: three instructions a step).
// A DPP operand must not be read in the two issue slots after the register was written: each
// step starts with that wait, which the compiler cannot add inside the block.
#define OSCAR_DPP_MAX_STEPS(OP)                                                              \
  asm volatile("s_nop 1\n\t" OP " %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t" \
               "s_nop 1\n\t" OP " %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t" \
               "s_nop 1\n\t" OP " %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"     \
               "s_nop 1\n\t" OP " %0, %0, %0 row_mirror row_mask:0xf bank_mask:0xf"                \
               : "+v"(v))
__device__ __forceinline__ float row16_max_fast(float v) {   // no NaN among the inputs
  OSCAR_DPP_MAX_STEPS("v_max_f32_dpp");
  return v;
}
__device__ __forceinline__ uint32_t row16_max_u32(uint32_t v) {
  OSCAR_DPP_MAX_STEPS("v_max_u32_dpp");
  return v;
}
__device__ __forceinline__ float row16_sum(float v) {
  v += dpp_mov<0xB1>(v);
  v += dpp_mov<0x4E>(v);
  v += dpp_mov<0x141>(v);
  v += dpp_mov<0x140>(v);
  return v;
}

__device__ __forceinline__ void halves_to_f32(const uint4& r, float (&x)[8]) {
  const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    x[2 * i] = __half2float(__ushort_as_half((unsigned short)(w[i] & 0xffffu)));
    x[2 * i + 1] = __half2float(__ushort_as_half((unsigned short)(w[i] >> 16)));
  }
}

// fp16 hi[8] + lo[8] limbs of the exact products x[i] * y[i] (y = 8 packed fp16 values):
// hi = f16(x*y), lo = f16(fma(x, y, -hi)), each a single mixed-precision FMA that reads its
// fp16 sources in place and writes one half of the destination register, so neither the
// multiplier nor the limbs are ever widened, subtracted or packed separately.
// hi + lo equals the product to ~2^-22.
// One block of 16 instructions: a half-register write must not be followed directly by a
// vector instruction that reads the register (the compiler cannot see into the block to
// insert the wait state itself); here every such read comes four instructions after the
// write, and the block ends with a wait state of its own.
__device__ __forceinline__ void mul_split_hi_lo(const float (&x)[8], const uint4& y, uint4& hi,
                                                uint4& lo) {
  uint32_t h0, h1, h2, h3, l0, l1, l2, l3;
  asm volatile("v_fma_mixlo_f16 %0, %8, %16, 0 op_sel_hi:[0,1,0]\n\t"
      "v_fma_mixlo_f16 %1, %10, %17, 0 op_sel_hi:[0,1,0]\n\t"
      "v_fma_mixlo_f16 %2, %12, %18, 0 op_sel_hi:[0,1,0]\n\t"
      "v_fma_mixlo_f16 %3, %14, %19, 0 op_sel_hi:[0,1,0]\n\t"
      "v_fma_mixhi_f16 %0, %9, %16, 0 op_sel:[0,1,0] op_sel_hi:[0,1,0]\n\t"
      "v_fma_mixhi_f16 %1, %11, %17, 0 op_sel:[0,1,0] op_sel_hi:[0,1,0]\n\t"
      "v_fma_mixhi_f16 %2, %13, %18, 0 op_sel:[0,1,0] op_sel_hi:[0,1,0]\n\t"
      "v_fma_mixhi_f16 %3, %15, %19, 0 op_sel:[0,1,0] op_sel_hi:[0,1,0]\n\t"
      "v_fma_mixlo_f16 %4, %8, %16, -%0 op_sel_hi:[0,1,1]\n\t"
      "v_fma_mixlo_f16 %5, %10, %17, -%1 op_sel_hi:[0,1,1]\n\t"
      "v_fma_mixlo_f16 %6, %12, %18, -%2 op_sel_hi:[0,1,1]\n\t"
      "v_fma_mixlo_f16 %7, %14, %19, -%3 op_sel_hi:[0,1,1]\n\t"
      "v_fma_mixhi_f16 %4, %9, %16, -%0 op_sel:[0,1,1] op_sel_hi:[0,1,1]\n\t"
      "v_fma_mixhi_f16 %5, %11, %17, -%1 op_sel:[0,1,1] op_sel_hi:[0,1,1]\n\t"
      "v_fma_mixhi_f16 %6, %13, %18, -%2 op_sel:[0,1,1] op_sel_hi:[0,1,1]\n\t"
      "v_fma_mixhi_f16 %7, %15, %19, -%3 op_sel:[0,1,1] op_sel_hi:[0,1,1]\n\t"
      "s_nop 0"
      : "=&v"(h0), "=&v"(h1), "=&v"(h2), "=&v"(h3), "=&v"(l0), "=&v"(l1), "=&v"(l2), "=&v"(l3)
      : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]), "v"(x[6]), "v"(x[7]),
        "v"(y.x), "v"(y.y), "v"(y.z), "v"(y.w));
  hi = make_uint4(h0, h1, h2, h3);
  lo = make_uint4(l0, l1, l2, l3);
}

// The same limbs from packed fp16 arithmetic, for a multiplicand that serves several
// multipliers (the probabilities of a page against the step sizes of every value group, the
// queries against the step sizes of every page): x is split once into fp16 xh + xl (xl holds
// what the rounding of xh left over: x = xh + xl to 2^-22), and per multiplier
//   hi = xh * y,  e = fma(xh, y, -hi)  (the rounding error of that product, an fp16 number
//   unless it falls below the subnormal range),  lo = fma(xl, y, e)
// -- three packed instructions per two elements where the mixed-precision form takes four of
// twice the issue time.  hi + lo equals the product to ~2^-21.
#ifndef OSCAR_LIMBS_PACKED
#define OSCAR_LIMBS_PACKED 1
#endif
__device__ __forceinline__ void split_to_halves(const float (&x)[8], uint4& xh, uint4& xl) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  uint32_t h[4], l[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const f32x2 v = {x[2 * i], x[2 * i + 1]};
    const half2v hh = __builtin_convertvector(v, half2v);
    const f32x2 r = {x[2 * i] - (float)hh[0], x[2 * i + 1] - (float)hh[1]};   // exact
    h[i] = __builtin_bit_cast(uint32_t, hh);
    l[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, half2v));
  }
  xh = make_uint4(h[0], h[1], h[2], h[3]);
  xl = make_uint4(l[0], l[1], l[2], l[3]);
}
__device__ __forceinline__ uint4 scale_halves(const uint4& y, half2v k) {
  const uint32_t c[4] = {y.x, y.y, y.z, y.w};
  uint32_t r[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2v, c[i]) * k);
  return make_uint4(r[0], r[1], r[2], r[3]);
}
// Two fp16 limbs of t[i], |t[i]| < 2^13 * u[i] with u a power of two per slot, on a common grid:
// hi[i] is t rounded to the grid 4 * u[i] (adding and subtracting 1.5 * 2^23 grids rounds to nearest
// even), lo[i] what is left of it, the pair 2^-24 of the range off at most.  g and r are the two
// limbs widened, for the sums that have to cancel the limbs' own.
__device__ __forceinline__ void grid_limbs(const float (&t)[8], const float (&u)[8], float (&g)[8],
                                           float (&r)[8], uint4& hi, uint4& lo) {
#pragma clang fp contract(off)
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  constexpr float magic = 12582912.0f * 4.0f;
  uint32_t h[4], l[4];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float m = u[i] * magic;
    g[i] = (t[i] + m) - m;
    r[i] = t[i] - g[i];
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const f32x2 gv = {g[2 * i], g[2 * i + 1]}, rv = {r[2 * i], r[2 * i + 1]};
    const half2v lv = __builtin_convertvector(rv, half2v);
    h[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(gv, half2v));
    l[i] = __builtin_bit_cast(uint32_t, lv);
    r[2 * i] = (float)lv[0];
    r[2 * i + 1] = (float)lv[1];
  }
  hi = make_uint4(h[0], h[1], h[2], h[3]);
  lo = make_uint4(l[0], l[1], l[2], l[3]);
}
__device__ __forceinline__ void mul_limbs_packed(const uint4& xh, const uint4& xl, const uint4& y,
                                                 uint4& hi, uint4& lo) {
  const uint32_t a[4] = {xh.x, xh.y, xh.z, xh.w}, b[4] = {xl.x, xl.y, xl.z, xl.w};
  const uint32_t c[4] = {y.x, y.y, y.z, y.w};
  uint32_t h[4], l[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const half2v ah = __builtin_bit_cast(half2v, a[i]), al = __builtin_bit_cast(half2v, b[i]);
    const half2v yy = __builtin_bit_cast(half2v, c[i]);
    const half2v p = ah * yy;
    const half2v e = __builtin_elementwise_fma(ah, yy, -p);
    const half2v q = __builtin_elementwise_fma(al, yy, e);
    h[i] = __builtin_bit_cast(uint32_t, p);
    l[i] = __builtin_bit_cast(uint32_t, q);
  }
  hi = make_uint4(h[0], h[1], h[2], h[3]);
  lo = make_uint4(l[0], l[1], l[2], l[3]);
}

// Products of packed fp16 pairs in fp32, and fp16 * fp32, without widening instructions:
// the mixed-precision FMA reads fp16 sources in place.  (The wrong logits that a (32,32)-group
// build once showed with these blocks as plain asm came from an output register placed on the
// destination of a matrix instruction in flight, see keep_tuple; with that fixed they work as
// plain asm too, and stay volatile only because nothing is gained by letting them move.)
__device__ __forceinline__ void mix_mul_pair(uint32_t a, uint32_t b, float& lo, float& hi) {
  asm volatile("v_fma_mix_f32 %0, %1, %2, 0 op_sel_hi:[1,1,0]" : "=v"(lo) : "v"(a), "v"(b));
  asm volatile("v_fma_mix_f32 %0, %1, %2, 0 op_sel:[1,1,0] op_sel_hi:[1,1,0]" : "=v"(hi) : "v"(a), "v"(b));
}
// -(fp16 value), widened: the zero-point term of the float zero-point mode
__device__ __forceinline__ void neg_widen8(const uint4& a, float (&x)[8]) {
  const uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    x[2 * i] = -__half2float(__ushort_as_half((unsigned short)(w[i] & 0xffffu)));
    x[2 * i + 1] = -__half2float(__ushort_as_half((unsigned short)(w[i] >> 16)));
  }
}
__device__ __forceinline__ void mix_mul8(const uint4& a, const uint4& b, float (&x)[8]) {
  mix_mul_pair(a.x, b.x, x[0], x[1]);
  mix_mul_pair(a.y, b.y, x[2], x[3]);
  mix_mul_pair(a.z, b.z, x[4], x[5]);
  mix_mul_pair(a.w, b.w, x[6], x[7]);
}
// x * (fp16 half `hi_half` of packed h)
template <int HI> __device__ __forceinline__ float mix_scale(float x, uint32_t h) {
  float r;
  if (HI) asm volatile("v_fma_mix_f32 %0, %1, %2, 0 op_sel:[0,1,0] op_sel_hi:[0,1,0]" : "=v"(r) : "v"(x), "v"(h));
  else asm volatile("v_fma_mix_f32 %0, %1, %2, 0 op_sel_hi:[0,1,0]" : "=v"(r) : "v"(x), "v"(h));
  return r;
}

// The unpack masks live in vector registers.  Measured on gfx950 with two or more waves per
// SIMD: a v_and_b32 or v_lshrrev_b32 whose operands are vector registers (or a literal) issues in
// about 2.6 clocks per wave, the same instruction with a scalar-register operand in 4.5 -- so the
// masks are kept out of scalar registers (where the compiler puts such loop constants).
template <int BITS> struct Masks {
  uint32_t m0, m1, m2;
  __device__ __forceinline__ void init() {
    m0 = BITS == 2 ? 0x00300030u : 0x003C003Cu;
    m1 = BITS == 2 ? 0x00C000C0u : 0x03C003C0u;
    m2 = 0x03000300u;
    asm volatile("" : "+v"(m0), "+v"(m1));
    if (BITS == 2) asm volatile("" : "+v"(m2));
  }
};

// All four registers of a matrix-instruction result stay allocated up to this point, also the
// ones nobody reads (rows of absent heads).  Without it the register allocator hands such a
// register to the next value while the instruction that will still write it is in flight; for
// its own instructions the compiler then inserts the wait states the hardware asks for, for the
// instructions inside an asm block it cannot -- and the result of a block placed there was
// overwritten when the matrix instruction retired (seen as run-to-run differences of a build
// whose only change was the order of the matrix instructions).
__device__ __forceinline__ void keep_tuple(const float4v& t) { asm volatile("" ::"v"(t)); }

// One 32-code chunk -> the four B-operand vectors (k-steps 0..3) of a 16x16x32 MFMA.
template <int BITS> struct Chunk;
template <> struct Chunk<2> {
  uint32_t w[2];
  __device__ __forceinline__ void operands(u32x4 (&b)[4], const Masks<2>& m) const {
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      // bit pairs 0,1 via << 4 (-> positions 4, 6), pairs 2,3,4 in place, pairs 5,6,7 via >> 6
      const uint32_t x = w[d], y = x >> 6, z = x << 4;
      b[2 * d] = (u32x4){z & m.m0, z & m.m1, x & m.m0, x & m.m1};
      b[2 * d + 1] = (u32x4){x & m.m2, y & m.m0, y & m.m1, y & m.m2};
    }
  }
};
template <> struct Chunk<4> {
  uint32_t w[4];
  __device__ __forceinline__ void operands(u32x4 (&b)[4], const Masks<4>& m) const {
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      // nibbles 0,1 via << 2 (-> bit offsets 2, 6), nibbles 2,3 via >> 6
      const uint32_t x = w[d], y = x >> 6, z = x << 2;
      b[d] = (u32x4){z & m.m0, z & m.m1, y & m.m0, y & m.m1};
    }
  }
};

// Page loads go through raw buffer resources, one per pool.  The resource's base is fixed for
// the whole kernel (pool + kv head * page bytes) and spans one page; the page itself is
// selected by the scalar offset of the load (physical page * kv heads * page bytes), so a new
// page costs a scalar multiply and add per pool instead of a 64-bit address computation.  The
// hardware's range check compares the per-lane offset with (number of records - scalar
// offset), so the record count of a live resource is the end of its page.  The per-lane offset is a loop constant, and a resource of
// zero length turns the prefetch past a wave's last page into loads that return zeros without
// touching memory -- the prefetch needs no branch, so the loaded registers are plain
// loop-carried values (a conditional load made the compiler copy the whole register set, and
// wait for it, at the end of every iteration).  A single wave issues one instruction about
// every five clocks whatever its kind, so scalar bookkeeping in the page loop is not free.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t pool_rsrc(const uint8_t* base, uint32_t page_off,
                                                            int bytes, bool valid) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(base), 0,
                                           valid ? (int)(page_off + (uint32_t)bytes) : 0, 0x00020000);
}
// Loads are marked non-temporal (streaming): every byte of the cache is read once per launch,
// and keeping it out of the way of the small kernels around this one took 3 us off a decode
// step on the 32K-context workload (1 us off this kernel).
__device__ __forceinline__ uint4 buf_load16(__amdgpu_buffer_rsrc_t r, int off, uint32_t soff = 0) {
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, off, (int)soff, 2));
}

// 16 bytes a lane from memory straight into LDS, lane after lane from byte `dst` of LDS (uniform) on.  In asm, as
// are the reads of what it brings (read_staged): the compiler would wait for every load in flight in front of each
// LDS access that might touch it, the operand tables' in the page loop included.  It does not count this one, so
// its own waits can only come out longer.  (The wait states: the descriptor may come from vector instructions, and
// m0 is read a slot after it was written.)
__device__ __forceinline__ u32x4 lds_load_rsrc(const void* base, uint32_t bytes) {
  const unsigned long long p = reinterpret_cast<unsigned long long>(base);
  return (u32x4){(uint32_t)p, (uint32_t)(p >> 32) & 0xffffu, bytes, 0x00020000u};
}
__device__ __forceinline__ void load_to_lds(const u32x4& rsrc, uint32_t dst, int off) {
  asm volatile("s_nop 4\n\ts_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen nt lds"
               :: "s"(dst), "v"(off), "s"(rsrc) : "memory", "m0");
}
// Four times 16 bytes of LDS, 256 bytes apart, and the wait for them.
__device__ __forceinline__ void read_staged(uint32_t at, u32x4 (&x)[4]) {
  asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:256\n\tds_read_b128 %2, %4 offset:512\n\t"
               "ds_read_b128 %3, %4 offset:768\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]) : "v"(at) : "memory");
}
__device__ __forceinline__ uint32_t lds_byte(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

// Eight consecutive metadata values (element `elem` of the resource onwards), held as stored.
template <bool M32> struct Meta8;
template <> struct Meta8<false> {
  uint4 a;
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, int elem, uint32_t so) {
    a = buf_load16(r, elem * 2, so);
  }
};
template <> struct Meta8<true> {
  uint4 a, b;
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, int elem, uint32_t so) {
    a = buf_load16(r, elem * 4, so);
    b = buf_load16(r, elem * 4 + 16, so);
  }
  __device__ __forceinline__ void floats(float (&x)[8]) const {
    x[0] = __uint_as_float(a.x); x[1] = __uint_as_float(a.y);
    x[2] = __uint_as_float(a.z); x[3] = __uint_as_float(a.w);
    x[4] = __uint_as_float(b.x); x[5] = __uint_as_float(b.y);
    x[6] = __uint_as_float(b.z); x[7] = __uint_as_float(b.w);
  }
};
// What one unit of the other operand takes off per element: Delta*z, or -zero when the zero-point
// is the float group minimum (x = Delta*c + zero).
template <bool ZPMIN>
__device__ __forceinline__ void zero_terms(const Meta8<true>& d, const Meta8<true>& z, float (&dz)[8]) {
  float zf[8];
  z.floats(zf);
  if constexpr (ZPMIN) {
#pragma unroll
    for (int i = 0; i < 8; ++i) dz[i] = -zf[i];
  } else {
    float df[8];
    d.floats(df);
#pragma unroll
    for (int i = 0; i < 8; ++i) dz[i] = df[i] * zf[i];
  }
}
template <bool ZPMIN>
__device__ __forceinline__ void zero_terms(const Meta8<false>& d, const Meta8<false>& z, float (&dz)[8]) {
  if constexpr (ZPMIN) neg_widen8(z.a, dz);
  else mix_mul8(d.a, z.a, dz);
}

// A lane's two chunks of a tile pair: 16 bytes (2-bit) or 32 bytes (4-bit) of pair tp.
template <int BITS> struct TilePair;
template <> struct TilePair<2> {
  uint4 v;
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, int tp, int lane, uint32_t so) {
    v = buf_load16(r, (tp * 64 + (lane & 15) * 4 + (lane >> 4)) * 16, so);
  }
  __device__ __forceinline__ Chunk<2> chunk(int i) const {
    Chunk<2> c;
    c.w[0] = i ? v.z : v.x;
    c.w[1] = i ? v.w : v.y;
    return c;
  }
};
// A lane's 32 bytes as two loads of their halves ask for every cache line twice: the 16 lanes of a quarter are 128
// bytes apart, a load takes half of what it touches, and by the second load the lines of the first are gone again
// (a request to the L2 for every 69 bytes, 9.2 million in a launch over 64 x 8K tokens).  So the 16 lanes of a
// quarter read 32 bytes of eight places in one load: lane n = m + 8*h of the first load the half h (tile
// 2*tp + h) of place m, of the second the half 1 - h of place 8 + m: 127 bytes a request, 5.0 million.  A register
// holds the even tile in one half of its lanes and the odd one in the other; three DPP moves a word put both in
// order where they are used (step of 64 x 8K tokens 118.9 -> 106.0 us, 5.3 -> 6.0 TB/s).  With the two halves in
// neighbouring lanes the requests are the same and the accesses inside the CU's cache 0.57 times as many, and
// nothing is gained by it (104.5 against 103.6 us): memory is the bound.
template <> struct TilePair<4> {
  uint4 a, b;
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, int tp, int lane, uint32_t so) {
    const int m = lane & 7, h = (lane >> 3) & 1, q4 = lane >> 4;
    a = buf_load16(r, (tp * 64 + m * 4 + q4) * 32 + 16 * h, so);
    b = buf_load16(r, (tp * 64 + (m + 8) * 4 + q4) * 32 + 16 * (1 - h), so);
  }
  static __device__ __forceinline__ uint32_t word(uint32_t x, uint32_t y, int i) {
    if (i == 0)   // lanes 0 .. 7 of a row from a, 8 .. 15 from b, where they are
      return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)y, 0xE4 /* quad_perm:[0,1,2,3] */, 0xf, 0xc, false);
    // lanes 0 .. 7 from lanes 8 .. 15 of a, 8 .. 15 from 0 .. 7 of b
    const int t = __builtin_amdgcn_update_dpp((int)x, (int)x, 0x128 /* row_ror:8 */, 0xf, 0x3, false);
    return (uint32_t)__builtin_amdgcn_update_dpp(t, (int)y, 0x128, 0xf, 0xc, false);
  }
  __device__ __forceinline__ Chunk<4> chunk(int i) const {
    Chunk<4> c;
    c.w[0] = word(a.x, b.x, i);
    c.w[1] = word(a.y, b.y, i);
    c.w[2] = word(a.z, b.z, i);
    c.w[3] = word(a.w, b.w, i);
    return c;
  }
};

// The pools' bases for one kv head and the byte strides between physical pages (wave-uniform).
struct PoolBases {
  const uint8_t *kcodes, *kmeta, *knorm, *vcodes, *vmeta;
  uint32_t s_kcodes, s_kmeta, s_knorm, s_vcodes, s_vmeta;
  __device__ __forceinline__ void make(const DecodeParams& P, int kvh) {
    const uint32_t Hkv = (uint32_t)P.c.cfg.n_kv_heads;
    kcodes = static_cast<const uint8_t*>(P.c.k_codes) + (size_t)kvh * P.g.k_codes_bytes;
    kmeta = static_cast<const uint8_t*>(P.c.k_meta) + (size_t)kvh * P.g.k_meta_bytes;
    knorm = static_cast<const uint8_t*>(P.c.k_norms) + (size_t)kvh * P.g.k_norms_bytes;
    vcodes = static_cast<const uint8_t*>(P.c.v_codes) + (size_t)kvh * P.g.v_codes_bytes;
    vmeta = static_cast<const uint8_t*>(P.c.v_meta) + (size_t)kvh * P.g.v_meta_bytes;
    s_kcodes = Hkv * (uint32_t)P.g.k_codes_bytes;
    s_kmeta = Hkv * (uint32_t)P.g.k_meta_bytes;
    s_knorm = Hkv * (uint32_t)P.g.k_norms_bytes;
    s_vcodes = Hkv * (uint32_t)P.g.v_codes_bytes;
    s_vmeta = Hkv * (uint32_t)P.g.v_meta_bytes;
  }
};
// The five buffer resources of one page and the page's scalar offsets (wave-uniform).
struct PageRsrc {
  __amdgpu_buffer_rsrc_t kcodes, kmeta, knorm, vcodes, vmeta;
  uint32_t o_kcodes, o_kmeta, o_knorm, o_vcodes, o_vmeta;
  __device__ __forceinline__ void make(const PoolBases& B, const DecodeParams& P, uint32_t phys, bool valid) {
    o_kcodes = phys * B.s_kcodes;
    o_kmeta = phys * B.s_kmeta;
    o_knorm = phys * B.s_knorm;
    o_vcodes = phys * B.s_vcodes;
    o_vmeta = phys * B.s_vmeta;
    kcodes = pool_rsrc(B.kcodes, o_kcodes, P.g.k_codes_bytes, valid);
    kmeta = pool_rsrc(B.kmeta, o_kmeta, P.g.k_meta_bytes, valid);
    knorm = pool_rsrc(B.knorm, o_knorm, P.g.k_norms_bytes, valid);
    vcodes = pool_rsrc(B.vcodes, o_vcodes, P.g.v_codes_bytes, valid);
    vmeta = pool_rsrc(B.vmeta, o_vmeta, P.g.v_meta_bytes, valid);
  }
};

// What one wave needs of one page, in registers, single-buffered: every register is
// reloaded for the wave's next page right after its last use for the current one, so each
// load has a whole iteration to arrive and only one copy of a page is ever live.
template <int BITS, int NGK, bool M32> struct KeyRegs {
  TilePair<BITS> kc[4];
  Meta8<M32> kd[NGK], kz[NGK];  // key Delta / zero of positions 8n..8n+7 (operand order)
  Meta8<M32> nr;                // norms of tokens 16*T+n, T = 0..7
  __device__ __forceinline__ void load_codes(const PageRsrc& r, int tp, int lane) {
    kc[tp].load(r.kcodes, tp, lane, r.o_kcodes);
  }
  __device__ __forceinline__ void load_meta(const PageRsrc& r, int g, int lane) {
    kd[g].load(r.kmeta, g * D + 8 * (lane & 15), r.o_kmeta);
    kz[g].load(r.kmeta, (NGK + g) * D + 8 * (lane & 15), r.o_kmeta);
  }
  __device__ __forceinline__ void load_norm(const PageRsrc& r, int lane) {
    nr.load(r.knorm, 8 * (lane & 15), r.o_knorm);
  }
  __device__ __forceinline__ void load(const PageRsrc& r, int lane) {
#pragma unroll
    for (int tp = 0; tp < 4; ++tp) load_codes(r, tp, lane);
#pragma unroll
    for (int g = 0; g < NGK; ++g) load_meta(r, g, lane);
    load_norm(r, lane);
  }
};
template <int BITS, int NGV, bool M32> struct ValRegs {
  TilePair<BITS> vc[4];
  Meta8<M32> vd[NGV], vz[NGV];  // value Delta / zero of tokens 16*T+n
  __device__ __forceinline__ void load_codes(const PageRsrc& r, int tp, int lane) {
    vc[tp].load(r.vcodes, tp, lane, r.o_vcodes);
  }
  __device__ __forceinline__ void load_delta(const PageRsrc& r, int g, int lane) {
    vd[g].load(r.vmeta, g * R + 8 * (lane & 15), r.o_vmeta);
  }
  __device__ __forceinline__ void load_zero(const PageRsrc& r, int g, int lane) {
    vz[g].load(r.vmeta, (NGV + g) * R + 8 * (lane & 15), r.o_vmeta);
  }
  __device__ __forceinline__ void load(const PageRsrc& r, int lane) {
#pragma unroll
    for (int tp = 0; tp < 4; ++tp) load_codes(r, tp, lane);
#pragma unroll
    for (int g = 0; g < NGV; ++g) {
      load_delta(r, g, lane);
      load_zero(r, g, lane);
    }
  }
};

// Eight consecutive values of the caller's dtype (a run-time property here), held raw.
// Loads are buffer loads without branches: a branch around a load makes the compiler wait
// for every load in flight where the branches join (the start of this kernel was a chain of
// such waits: each residual token's loads completed, behind the whole first page, before the
// next token's were issued).  fp32 needs 32 bytes; the upper 16 come through a second
// resource that is void for the 16-bit types.
struct IoRsrc {
  __amdgpu_buffer_rsrc_t lo, hi;
  int es;   // bytes per element
  __device__ __forceinline__ void make(const void* base, size_t first_elem, int n_elem, int dt,
                                       bool valid) {
    es = dt == OSCAR_F32 ? 4 : 2;
    uint8_t* p = const_cast<uint8_t*>(static_cast<const uint8_t*>(base)) + first_elem * (size_t)es;
    lo = __builtin_amdgcn_make_buffer_rsrc(p, 0, valid ? n_elem * es : 0, 0x00020000);
    hi = __builtin_amdgcn_make_buffer_rsrc(p, 0, (valid && dt == OSCAR_F32) ? n_elem * es : 0, 0x00020000);
  }
};
struct Raw8rt {
  uint4 a, b;
  // elements elem .. elem+7 of the resource (zeros past its end)
  __device__ __forceinline__ void load(const IoRsrc& r, int elem) {
    a = buf_load16(r.lo, elem * r.es);
    b = buf_load16(r.hi, elem * r.es + 16);
  }
  __device__ __forceinline__ void widen(float (&x)[8], int dt) const {
    if (dt == OSCAR_F32) {
      x[0] = __uint_as_float(a.x); x[1] = __uint_as_float(a.y);
      x[2] = __uint_as_float(a.z); x[3] = __uint_as_float(a.w);
      x[4] = __uint_as_float(b.x); x[5] = __uint_as_float(b.y);
      x[6] = __uint_as_float(b.z); x[7] = __uint_as_float(b.w);
    } else if (dt == OSCAR_BF16) {
      x[0] = __uint_as_float(a.x << 16); x[1] = __uint_as_float(a.x & 0xffff0000u);
      x[2] = __uint_as_float(a.y << 16); x[3] = __uint_as_float(a.y & 0xffff0000u);
      x[4] = __uint_as_float(a.z << 16); x[5] = __uint_as_float(a.z & 0xffff0000u);
      x[6] = __uint_as_float(a.w << 16); x[7] = __uint_as_float(a.w & 0xffff0000u);
    } else {
      halves_to_f32(a, x);
    }
  }
};

// One residual token's share for a lane: 8 channels (channel group cg) of K_u (fp16) and of
// V (caller's dtype), and the token norm, as stored.
template <bool M32> struct ResTok {
  uint4 k;
  Raw8rt v;
  uint32_t nrm;
  __device__ __forceinline__ float norm() const {
    return M32 ? __uint_as_float(nrm) : __half2float(__ushort_as_half((unsigned short)nrm));
  }
};
// Step sizes are non-negative fp16 numbers, which order like their bit patterns: packed
// unsigned 16-bit max needs no NaN canonicalization.
typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pk_max_u16(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(ushort2v, a),
                                                                __builtin_bit_cast(ushort2v, b)));
}
__device__ __forceinline__ uint4 pk_max4(const uint4& a, const uint4& b) {
  return make_uint4(pk_max_u16(a.x, b.x), pk_max_u16(a.y, b.y), pk_max_u16(a.z, b.z),
                    pk_max_u16(a.w, b.w));
}

// rows of the 16-row operand tile: head h -> hi row 4*(h%4) + 2*(h/4), lo row + 1, so the
// accumulator lane group q4 (rows 4*q4..4*q4+3) owns heads q4 (slot 0) and q4+4 (slot 1).
__device__ __forceinline__ int row_hi(int h) { return 4 * (h & 3) + 2 * (h >> 2); }

// HP = head slots per accumulator lane group: 1 for up to 4 query heads per kv head, 2 for
// 5..8 (twice the per-head registers).  Two workgroups per CU wherever the registers allow it
// with little or no scratch memory (oscar_decode_mfma_wgs_per_cu lists the variants); the
// rest run one workgroup per CU and their overflow lives in accumulation registers
// (measured: 4-bit, G_k = 32 took 188 us with 65 spilled registers at two per CU, 76 us at
// one).
//
// The step's kernel holds the new token beside all that.  Five variants that run at two per CU without it
// (step_one_per_cu) are built for one, and taken only where a CU gets no second workgroup anyway
// (step_form_pays): at two they kept 64 .. 120 bytes of a lane in scratch as long as the residual window went
// through registers.  At two they would have none today (220 .. 245 registers; (2,2,4,4) 24 bytes).
__host__ __device__ constexpr bool step_one_per_cu(int bits, int hp, int ngk, int ngv) {
  if (bits == 2) return hp == 2 && ngk == 4 && ngv == 4;
  return hp == 1 ? ngk == 4 && ngv < 4 : ngk <= 2 && ngv == 1;
}

// Workgroups of eight waves, for launches of at most one workgroup a CU: with four, the other half of the
// SIMDs' two wave slots stays empty while a wave, held to an instruction every five clocks, walks its two
// pages and its share of the residual window.  Device time of a step over caches that are not in the
// last-level cache, four / eight waves, us: INT2, G_k = 128, G_v = 32, 8 kv heads, batch 1 x 1000 17.6 / 14.1,
// 1 x 4000 12.5 / 11.3, 1 x 32000 13.2 / 12.7, 16 x 1000 19.7 / 15.7; seven query heads a kv head, 1 x 1000
// 23.0 / 18.3, 1 x 16000 16.1 / 14.8; fp32 metadata 1 x 1000 20.9 / 17.4; INT4 1 x 1000 19.1 / 16.5.  At INT4 it
// is one split only (the window is what gains: with several splits, warm, 1 x 8000 12.8 / 13.6, 1 x 16000
// 14.7 / 17.5), with fp32 metadata not at all.  With an empty window the attention alone loses there (1 x 1024
// 9.7 / 10.4, with 104 tokens in it 17.1 / 14.2, with 116 of 500 15.8 / 12.3; the step 11.8 / 11.6, 19.0 / 16.5 and
// 17.7 / 14.4), and the window is as often full as empty.
// (With the residual window straight in LDS, whole step, warm, 1 x 1016, one split: 28 heads on 4, G_k = 128 with
// G_v = 32 16.9 / 14.9, G_k = G_v = 64 16.6 / 14.8, G_k = 64 with G_v = 32 17.3 / 15.2; 32 on 8, 1 x 1000 12.4 / 11.3,
// INT4 13.4 / 12.6.  15 splits of 1 x 16000, 28 on 4, 16.6 / 15.4.)
// At one split count the two forms deal a sequence's pages to different waves: the last bits of its output
// differ between launches on either side of the line.
// Built where two workgroups of four fit a CU in both kernels (the step's and the attention alone
// give the same bits, so they split alike).
__host__ __device__ constexpr bool eight_waves_built(int bits, int hp, int ngk, int ngv, bool m32) {
  return oscar_decode_mfma_wgs_per_cu(bits, hp, ngk, ngv, m32) == 2 &&
         (m32 ? bits == 2 : !step_one_per_cu(bits, hp, ngk, ngv));
}

#if OSCAR_MFMA_STEP
// values of the residual window as the encoder's block quantizer takes them
struct WindowValues {
  Raw8rt raw;
  int dt;
  __device__ __forceinline__ void widen(float (&x)[8]) const { raw.widen(x, dt); }
};

// One lane's 8 channels of a token into slot `at` of the residual window.
__device__ __forceinline__ void store_new_token(const DecodeParams& P, size_t at, const uint4& k, const Raw8rt& v,
                                                uint32_t nrm, int cg) {
  *reinterpret_cast<uint4*>(reinterpret_cast<__half*>(P.c.res_k) + at * D + 8 * cg) = k;
  if (P.c.cfg.io_dtype == OSCAR_F32) {
    uint4* o = reinterpret_cast<uint4*>(reinterpret_cast<float*>(P.c.res_v) + at * D + 8 * cg);
    o[0] = v.a;
    o[1] = v.b;
  } else {
    *reinterpret_cast<uint4*>(reinterpret_cast<uint16_t*>(P.c.res_v) + at * D + 8 * cg) = v.a;
  }
  if (cg == 0) reinterpret_cast<uint16_t*>(P.c.res_norm)[at] = (uint16_t)nrm;
}

// The full window of (b, kvh) into page `page` of the sequence, then the new token into slot 0: what
// oscar_append_kernel does for this call, by one workgroup.
template <int BITS, int KG, int NP>
__device__ __forceinline__ void flush_window(EncoderLds<__half, BITS, KG, NP>& lds, const DecodeParams& P, int b, int kvh,
                                             int page, int tid, int cg) {
  const int Hkv = P.c.cfg.n_kv_heads, slot = NP == 8 ? tid >> 4 : (tid >> 4) & 15, grp = NP == 8 ? 0 : tid >> 8;
  const size_t rb = ((size_t)b * Hkv + kvh) * R;
  const int phys = P.c.block_table[(size_t)b * P.c.max_pages_per_seq + page];
  const __half* res_norm = reinterpret_cast<const __half*>(P.c.res_norm) + rb;
  const auto win_k = __builtin_amdgcn_make_buffer_rsrc(static_cast<uint8_t*>(P.c.res_k) + rb * D * 2, 0, R * D * 2, 0x00020000);
  IoRsrc win_v;
  win_v.make(P.c.res_v, rb * D, R * D, P.c.cfg.io_dtype, true);
  uint4 ku[NP];
  WindowValues vw[NP];
  float nrm[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int t = 16 * (NP == 8 ? p : 2 * p + grp) + slot;
    ku[p] = buf_load16(win_k, (t * D + 8 * cg) * 2);
    vw[p].raw.load(win_v, t * D + 8 * cg);
    vw[p].dt = P.c.cfg.io_dtype;
    nrm[p] = __half2float(res_norm[t]);
  }
  IoRsrc kn, vn;
  const size_t e0 = ((size_t)b * Hkv + kvh) * D;
  kn.make(P.k_new, e0, D, P.c.cfg.io_dtype, true);
  vn.make(P.v_new, e0, D, P.c.cfg.io_dtype, true);
  Raw8rt kraw, vraw;
  kraw.load(kn, 8 * cg);
  vraw.load(vn, 8 * cg);
  float x[8], nf;
  kraw.widen(x, P.c.cfg.io_dtype);
  uint32_t sg[4];
  butterfly_signs(cg, sg);
  const uint4 k = key_transform8<__half>(x, sg, nf);
  // every read of the old window has returned before slot 0 is written
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (slot == 0 && grp == 0) store_new_token(P, rb, k, vraw, half_bits(nf), cg);
  const float nrm_q[NP / 4] = {};
  const size_t pg = (size_t)phys * Hkv + kvh;
  quantize_keys<__half, BITS, KG, NP>(lds, ku, false, nrm, nrm_q, P.c, P.g, pg, OSCAR_MFMA_ZPMIN != 0, tid, cg);
  quantize_values<__half, BITS, KG, NP>(lds, vw, P.c, P.g, pg, OSCAR_MFMA_ZPMIN != 0, tid, cg);
}
#endif

// STEP: the launch is a whole decode step under the decode rule of oscar_quantize_append (one token per
// sequence, rotation on, L2 norm per head), then the attention over the cache that results.  As launches
// of their own the append cost 4 .. 9 us of a step for a token row per sequence and kv head.
//  * Every workgroup that owns part of the residual window transforms the new token itself (the 16
//    lanes of a row hold it exactly as they hold a token of the window); the wave whose token it is
//    writes it to its slot.
//  * A full window goes to its page first: by the workgroup whose wave will attend to that page, before
//    anything else, with the encoder's own block quantizer (once in 128 steps of a sequence); it also
//    writes the new token to slot 0 then, behind its reads of the old window, which nobody else reads.
//  * The lengths are advanced by the reduce pass.  With a single split there is none: every workgroup
//    draws the cache's ticket as soon as it has the lengths, so that whoever draws the last one knows
//    that all have read them, and advances them at its end.
template <int BITS, int HP, int NGK, int NGV, bool ZPMIN, bool M32, bool STEP, int NW>
__global__ __launch_bounds__(64 * NW, NW == 8 ? 2 : STEP && step_one_per_cu(BITS, HP, NGK, NGV)
                                      ? 1 : oscar_decode_mfma_wgs_per_cu(BITS, HP, NGK, NGV, M32))
void oscar_decode_mfma_kernel(DecodeParams P, int gq) {
  constexpr int TPG = 8 / NGK;  // token tiles per key group
  constexpr int CPG = 8 / NGV;  // channel tiles per value group
  constexpr int TABW = D + 8;   // operand table row stride in halves
  // operand tiles unpacked one at a time (instead of in pairs) where the pair's second
  // register set would not fit
  constexpr bool ONE_TILE = (HP == 2) || (NGK == 4);

  // rows padded by 16 bytes: the 16-byte operand reads of lanes n = 0..7 hit 8 different banks
#if OSCAR_MFMA_STEP
  struct Tables {
    alignas(16) _Float16 A[NW][16][TABW], P[NW][16][TABW];
    alignas(16) float o[NW][OSCAR_MAX_GQA][D];
  };
  __shared__ union {   // (the flush is over before the tables are touched)
    Tables t;
    EncoderLds<__half, BITS, R / NGK, NW == 8 ? 4 : 8> enc;
  } s_u;
  auto& s_A = s_u.t.A;
  auto& s_P = s_u.t.P;
  auto& s_o = s_u.t.o;
#else
  __shared__ __align__(16) _Float16 s_A[NW][16][TABW];   // per wave: (Q_h Delta_k) hi/lo rows
  __shared__ __align__(16) _Float16 s_P[NW][16][TABW];   // per wave: (p Delta_v) hi/lo rows
  __shared__ __align__(16) float s_o[NW][OSCAR_MAX_GQA][D];  // wave results for the merge
#endif
  __shared__ float s_wm[NW][OSCAR_MAX_GQA], s_wl[NW][OSCAR_MAX_GQA];
  // two head slots: the rotated queries in operand order wait in LDS between pages instead of
  // registers (16 registers that the second slot's softmax state needs)
  __shared__ __align__(16) float4 s_qr[HP == 2 ? NW : 1][HP == 2 ? 2 : 1][2][HP == 2 ? 64 : 1];

  const int split = blockIdx.x, kvh = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63;
  // wave index as a scalar: page numbers and block-table lookups stay on the scalar unit
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, q4 = lane >> 4;
#ifdef OSCAR_DECODE_STAMPS
  const bool stamp_first = kvh == 0 && b == 0 && split < 4;
  const bool stamp_last = kvh == (int)gridDim.y - 1 && b == (int)gridDim.z - 1 && split < 4;
  const bool stamp_on = stamp_first || stamp_last;
  const int stamp_slot = (stamp_last ? 4 : 0) + (split & 3);
#endif
  OSCAR_STAMP(0);   // entry
  // highest priority from the start (it falls in the page loop, see there): the workgroup that
  // reached the CU second should not get its first loads out behind the first one's prologue
  if (OSCAR_DECODE_PRIORITY) __builtin_amdgcn_s_setprio(3);
  const int Hkv = P.c.cfg.n_kv_heads, Hq = P.c.cfg.n_q_heads;
  constexpr bool zp_min = ZPMIN;

  // Pages are dealt round-robin: wave w of split s owns pages 4*s + w + 4*S*k, in the eight-wave form
  // s + S*w + 8*S*k.  The page numbers (and so the block-table addresses) do not depend on the sequence
  // length, which lets the length, table, query and residual loads all start together.  (Eight waves
  // share four SIMDs: a last round of a few pages must not fall on waves of one workgroup.  Batch 1 x 16K,
  // 125 pages on 120 waves, whole step: 13.1 us with four waves, 13.4 with eight dealt like them, 12.3 so.)
  const int pstride = NW * P.num_splits;
  const int pg_first = NW == 8 ? split + P.num_splits * wave : 4 * split + wave;
  const int32_t* table = P.c.block_table + (size_t)b * P.c.max_pages_per_seq;
  // Block-table entries of this wave's pages live in a register, one per lane, 63 iterations and the
  // prefetch of the next one at a time: the page loop itself issues no dependent lookups.  Entries
  // past the sequence's last page are never used for an access.
  auto load_table = [&](int it0) -> int {
    const int idx = pg_first + pstride * (it0 + lane);
    return idx < P.c.max_pages_per_seq ? table[idx] : 0;
  };
  OSCAR_STAMP(1 + (P.num_splits & 0));   // kernel arguments have arrived
  int tab = load_table(0);
  // queries: DPP row q4 of every wave takes head q4 (and q4 + 4 in the second slot), 8
  // channels (channel group cg) per lane; absent heads read as zeros
  const int cg = channel_group_of_row_lane(n);
  Raw8rt qraw[HP];
  {
    IoRsrc qr_;   // the group's gq query vectors; heads past gq fall off its end and read zeros
    qr_.make(P.q, ((size_t)b * Hq + (size_t)kvh * gq) * D, gq * D, P.c.cfg.io_dtype, true);
#pragma unroll
    for (int s = 0; s < HP; ++s) qraw[s].load(qr_, (q4 + 4 * s) * D + 8 * cg);
  }

  const int seq_len = P.c.seq_lens[b];
  int r = P.c.res_lens[b];
  int n_pages = (seq_len - r) / R;
  [[maybe_unused]] bool step_ok = false, step_flush = false;
  [[maybe_unused]] int my_ticket = -1;
#if OSCAR_MFMA_STEP
  {
    const StepPlan plan(seq_len, r, P.c.max_pages_per_seq);
    step_ok = plan.ok;
    step_flush = plan.ok && plan.flush;
    if (!plan.ok && tid == 0 && split == 0 && kvh == 0 && P.c.dev_status) *P.c.dev_status = OSCAR_ERR_CAPACITY;
    if (step_flush && split == (NW == 8 ? plan.packed : plan.packed >> 2) % P.num_splits) {
      flush_window(s_u.enc, P, b, kvh, plan.packed, tid, cg);
      // the page's stores have reached memory before any wave of this workgroup reads it
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
    }
    if (step_ok) {
      r = step_flush ? 1 : r + 1;
      n_pages += step_flush ? 1 : 0;
    }
  }
#endif
  // Residual slice of this split: rs tokens per split (a multiple of 16), handed out from
  // the last split backwards; inside the workgroup, wave w takes tokens 4*NW*pass + 4*w + j.
  const int rs = 16 * ((((r + 15) >> 4) + P.num_splits - 1) / P.num_splits);
  const int t_lo = min(r, (P.num_splits - 1 - split) * rs);
  const int rcount = min(r, t_lo + rs) - t_lo;
  const bool wave_res = 4 * wave < rcount;

  // ---- first residual pass and first page: issued before anything is computed.  The residual
  // tokens go first: they need no block-table entry, they are few, and the plain-ALU attention
  // over them then runs while the page is still on its way.  Waves without residual tokens skip
  // their loads (a void load still takes its turn in the CU's address unit, and at kernel start
  // all eight waves of a CU queue there). ----
  constexpr int NORM_BYTES = M32 ? 4 : 2;
  const auto res_norms = __builtin_amdgcn_make_buffer_rsrc(
      static_cast<uint8_t*>(P.c.res_norm) + ((size_t)b * Hkv + kvh) * R * NORM_BYTES, 0, R * NORM_BYTES, 0x00020000);
  // slot of the wave's token i of pass p0
  auto res_slot = [&](int p0, int i) { return t_lo + p0 + 4 * wave + i; };
#if OSCAR_MFMA_STEP
  // the new token is the window's last; every wave of the workgroup that owns it has it in registers
  const bool has_new = step_ok && rcount > 0 && t_lo + rcount == r;
  // (its loads go first here, the work on it waits until everything has been asked for)
  ResTok<M32> tok_new;
  Raw8rt knew;
  if (has_new && wave_res) {
    IoRsrc kn, vn;
    const size_t e0 = ((size_t)b * Hkv + kvh) * D;
    kn.make(P.k_new, e0, D, P.c.cfg.io_dtype, true);
    vn.make(P.v_new, e0, D, P.c.cfg.io_dtype, true);
    knew.load(kn, 8 * cg);
    tok_new.v.load(vn, 8 * cg);
  }
#endif
  // The window's tokens go straight into LDS, into the wave's own operand tables, which the page loop is the
  // first to need: four passes of 16-bit values at a time (two of fp32), K_u in one table, V in the other, a
  // token a row of lanes and its channels as the lanes hold them.  A place past the slice is some other token
  // of the window, which the pass masks out.
  // Through registers two passes were on their way at a time, the values' type was asked for at every token, and
  // in a launch with one split, which walks the whole window in every workgroup, a pass of 32 tokens cost 1.0 us.
  // Now all of the first passes arrive together, the registers are free, there is one loop a type, and the new
  // token of a step is put where the others are instead of being chosen in their place: 0.7 us (attention alone,
  // 1 x 1K with 126 tokens in the window 12.25 -> 11.1 us, with none 7.8; 64 x 8K INT4 109.3 -> 105.8, 94.4; steps
  // of 1 x 1000 12.5 -> 11.8, of 16 ragged sequences of 4K 19.9 -> 19.0, of 64 x 8K INT4 106.0 -> 103.2).
  const bool wide = P.c.cfg.io_dtype == OSCAR_F32;
  const int depth = wide ? 2 : 4;
  const uint32_t k_stage = lds_byte(&s_A[wave][0][0]), v_stage = lds_byte(&s_P[wave][0][0]);
  const u32x4 k_win = lds_load_rsrc(static_cast<const uint8_t*>(P.c.res_k) + ((size_t)b * Hkv + kvh) * R * D * 2, R * D * 2);
  const uint32_t v_bytes = wide ? 4 : 2;
  const u32x4 v_win = lds_load_rsrc(static_cast<const uint8_t*>(P.c.res_v) + ((size_t)b * Hkv + kvh) * R * D * v_bytes,
                                    R * D * v_bytes);
  auto in_window = [&](int p) { return 4 * (NW * p + wave) < rcount; };   // wave-uniform, as p is
  auto stage = [&](int p) {
    const int at = p & (depth - 1), elem = (res_slot(4 * NW * p, q4) & (R - 1)) * D + 8 * cg;
    load_to_lds(k_win, k_stage + 1024 * at, elem * 2);
    load_to_lds(v_win, v_stage + (wide ? 2048 : 1024) * at, elem * (int)v_bytes);
    if (wide) load_to_lds(v_win, v_stage + 2048 * at + 1024, elem * 4 + 16);
  };
  // lane 4*p + i: the norm of token i of pass p, as stored.  Loads come back in order, so when this one is there
  // everything staged in front of it is.
  auto load_norms = [&]() {
    const int t = (t_lo + 4 * (NW * (lane >> 2) + wave) + (lane & 3)) & (R - 1);
    if constexpr (M32) return (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(res_norms, t * 4, 0, 0);
    else return (uint32_t)(unsigned short)__builtin_amdgcn_raw_buffer_load_b16(res_norms, t * 2, 0, 0);
  };
  uint32_t win_nrm = 0;
  if (wave_res) {
#pragma unroll
    for (int p = 0; p < 4; ++p)
      if (p < depth && in_window(p)) stage(p);
    win_nrm = load_norms();
  }
  __builtin_amdgcn_sched_barrier(0);
  PoolBases pools;
  pools.make(P, kvh);
  KeyRegs<BITS, NGK, M32> kr;
  ValRegs<BITS, NGV, M32> vr;
  PageRsrc first;
  first.make(pools, P, (uint32_t)__builtin_amdgcn_readlane(tab, 0), pg_first < n_pages);
  kr.load(first, lane);
  __builtin_amdgcn_sched_barrier(0);
#if OSCAR_MFMA_STEP
  // All waves have the lengths in registers (the loads above have waited for them) before the
  // workgroup draws its ticket; the answer is needed at the very end only, by when it has long come.
  // Drawn at the end, the tickets of a launch whose workgroups finish together queue up, 11 ns each.
  // (Drawn inside a branch, wave 0 waited for its answer, and for the whole first page asked for before it,
  // on the spot.  Device time of a step, 64 sequences of 500 tokens 20.5 -> 19.8 us, of 1000 22.8 -> 22.1,
  // 32 of 500 13.1 -> 12.4.)
  if (P.num_splits == 1) {
    asm volatile("" ::"s"(n_pages), "s"(r));
    __builtin_amdgcn_s_barrier();
  }
  my_ticket = draw_ticket(P.c.tickets, P.num_splits == 1, tid);
  __builtin_amdgcn_sched_barrier(0);
#endif
  OSCAR_STAMP(2);   // first page's key-side loads issued

  // Q_h = H(q)/sqrt(128) * scale*log2(e), every wave for itself (DPP butterflies inside the
  // row, no LDS, no workgroup barrier): qh[s][i] = channel 8*cg + i of head q4 + 4*s
  uint32_t sgn[4];
  butterfly_signs(cg, sgn);
  float qh[HP][8];
#pragma unroll
  for (int s = 0; s < HP; ++s) {
    qraw[s].widen(qh[s], P.c.cfg.io_dtype);
    if (P.c.cfg.rotation == OSCAR_ROTATION_ON) rotate8(qh[s], sgn);
#pragma unroll
    for (int i = 0; i < 8; ++i) qh[s][i] *= P.qk_scale_log2;
  }

  OSCAR_STAMP(3);   // queries rotated
  // ---- wave state: online softmax over this wave's pages, seeded by its residual tokens ----
  float m_run[HP], l_run[HP], bv[HP][NGV];
  float4v O[8];
#pragma unroll
  for (int s = 0; s < HP; ++s) {
    m_run[s] = -INFINITY;
    l_run[s] = 0.0f;
#pragma unroll
    for (int g = 0; g < NGV; ++g) bv[s][g] = 0.0f;
  }
#pragma unroll
  for (int ct = 0; ct < 8; ++ct) O[ct] = (float4v){0.0f, 0.0f, 0.0f, 0.0f};
  // accumulator scale: O holds out * 2^-(24 - xv_cur - offset); this start value makes it 1
  int xv_cur = 24 - slot_bitpos_min(BITS);
  // (M32) the output itself, see the value side of the page loop
  [[maybe_unused]] float om[HP][8];
#pragma unroll
  for (int s = 0; s < HP; ++s)
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) om[s][ct] = 0.0f;

  // ---- residual tokens: plain-ALU attention over fp16 K_u and raw V, wave-local.  Row q4
  // works for head q4 (+4) on all four tokens of the wave's pass, a lane on its 8 channels:
  // logits are reduced over the 16 lanes of the row, nothing crosses rows.  The result
  // becomes the starting state of the wave's accumulators, so it costs no barrier. ----
  if (wave_res) {
    float mw[HP], lw[HP], ow[HP][8];
#pragma unroll
    for (int s = 0; s < HP; ++s) {
      mw[s] = -INFINITY;
      lw[s] = 0.0f;
#pragma unroll
      for (int c = 0; c < 8; ++c) ow[s][c] = 0.0f;
    }
#if OSCAR_MFMA_STEP
    if (has_new) {
      float x[8], nf;
      knew.widen(x, P.c.cfg.io_dtype);
      tok_new.k = key_transform8<__half>(x, sgn, nf);
      tok_new.nrm = half_bits(nf);
      if (!step_flush && q4 == 0 && wave == (((r - 1 - t_lo) & (4 * NW - 1)) >> 2))
        store_new_token(P, ((size_t)b * Hkv + kvh) * R + r - 1, tok_new.k, tok_new.v, tok_new.nrm, cg);
    }
#endif
    // The passes, four of the wave's tokens each, from LDS; IO (a constant here) is the values' type.  Every
    // fused multiply-add is written out: left to the compiler, the step form and the attention alone
    // fused differently and their outputs differed in the last bit.
    auto run_window = [&](auto io_tag) __attribute__((always_inline)) {
    constexpr int IO = decltype(io_tag)::value;
    constexpr bool WIDE = IO == OSCAR_F32;
    constexpr int DEPTH = WIDE ? 2 : 4, V_PASS = WIDE ? 2048 : 1024;
    auto pass = [&](int p) __attribute__((always_inline)) {
#pragma clang fp contract(off)
      const int p0 = 4 * NW * p, at = p & (DEPTH - 1);
      u32x4 ks[4], va[4], vb[4];
      read_staged(k_stage + 1024 * at + 16 * n, ks);
      read_staged(v_stage + V_PASS * at + 16 * n, va);
      if constexpr (WIDE) read_staged(v_stage + V_PASS * at + 1024 + 16 * n, vb);
      // (a value that does not belong to the slice must not meet its probability of 0: an infinite one would
      // make NaN of it)
      if (p0 + 4 * wave + 4 > rcount) {
#pragma unroll
        for (int i = 1; i < 4; ++i) {
          const uint32_t held = p0 + 4 * wave + i < rcount ? ~0u : 0u;
          va[i] &= held;
          if constexpr (WIDE) vb[i] &= held;
        }
      }
      float sc[HP][4], vv[4][8];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool valid = p0 + 4 * wave + i < rcount;   // wave-uniform
        ResTok<M32> tok;
        tok.k = __builtin_bit_cast(uint4, ks[i]);
        tok.v.a = __builtin_bit_cast(uint4, va[i]);
        tok.v.b = WIDE ? __builtin_bit_cast(uint4, vb[i]) : tok.v.a;
        tok.nrm = __builtin_amdgcn_readlane(win_nrm, 4 * p + i);
        float kv[8];
        halves_to_f32(tok.k, kv);
        tok.v.widen(vv[i], IO);
        const float nrm = tok.norm();
#pragma unroll
        for (int s = 0; s < HP; ++s) {
          float acc = qh[s][0] * kv[0];
#pragma unroll
          for (int c = 1; c < 8; ++c) acc = fmaf(qh[s][c], kv[c], acc);
          sc[s][i] = valid ? nrm * row16_sum(acc) : -INFINITY;
        }
      }
#pragma unroll
      for (int s = 0; s < HP; ++s) {
        // the wave's first token of a pass is valid, so the maximum is finite
        const float m_new = fmaxf(fmaxf(mw[s], fmaxf(sc[s][0], sc[s][1])), fmaxf(sc[s][2], sc[s][3]));
        const float alpha = __builtin_amdgcn_exp2f(mw[s] - m_new);
        mw[s] = m_new;
#pragma unroll
        for (int c = 0; c < 8; ++c) ow[s][c] *= alpha;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float pw = __builtin_amdgcn_exp2f(sc[s][i] - m_new);
          lw[s] = i == 0 ? fmaf(lw[s], alpha, pw) : lw[s] + pw;
#pragma unroll
          for (int c = 0; c < 8; ++c) ow[s][c] = fmaf(pw, vv[i][c], ow[s][c]);
        }
      }
    };
    asm volatile("" : "+v"(win_nrm)::"memory");   // (the staged tokens are there)
    for (int p = 0;;) {
      const int end = p + DEPTH;
#if OSCAR_MFMA_STEP
      // the new token takes the place of what was read from its slot
      const int last = rcount - 1, pn = last / (4 * NW), i_new = last & 3;
      if (has_new && pn >= p && pn < end && wave == (last & (4 * NW - 1)) >> 2) {
        const int at = pn & (DEPTH - 1);
        if (q4 == 0) {
          uint8_t* kd = reinterpret_cast<uint8_t*>(&s_A[wave][0][0]) + 1024 * at + 256 * i_new + 16 * n;
          uint8_t* vd = reinterpret_cast<uint8_t*>(&s_P[wave][0][0]) + V_PASS * at + 256 * i_new + 16 * n;
          *reinterpret_cast<uint4*>(kd) = tok_new.k;
          *reinterpret_cast<uint4*>(vd) = tok_new.v.a;
          if constexpr (WIDE) *reinterpret_cast<uint4*>(vd + 1024) = tok_new.v.b;
        }
        if (lane == 4 * pn + i_new) win_nrm = tok_new.nrm;
        asm volatile("" ::: "memory");
      }
#endif
      for (; p < end && in_window(p); ++p) {
        pass(p);
        if (in_window(p + DEPTH)) stage(p + DEPTH);
      }
      if (!in_window(p)) break;
      uint32_t mark = load_norms();
      asm volatile("" : "+v"(mark)::"memory");
    }
    };
    if (wide) run_window(std::integral_constant<int, OSCAR_F32>());
    else if (P.c.cfg.io_dtype == OSCAR_BF16) run_window(std::integral_constant<int, OSCAR_BF16>());
    else run_window(std::integral_constant<int, OSCAR_F16>());
    // hand the result over in accumulator layout through the wave's own slice of s_o
    // (written again only by this wave: for the query hand-off below and at the very end)
#pragma unroll
    for (int s = 0; s < HP; ++s) {
      const int h = q4 + 4 * s;
      if (h < gq) {
        *reinterpret_cast<float4*>(&s_o[wave][h][8 * cg]) = make_float4(ow[s][0], ow[s][1], ow[s][2], ow[s][3]);
        *reinterpret_cast<float4*>(&s_o[wave][h][8 * cg + 4]) = make_float4(ow[s][4], ow[s][5], ow[s][6], ow[s][7]);
      }
    }
    wave_lds_fence();
#pragma unroll
    for (int s = 0; s < HP; ++s) {
      const int h = q4 + 4 * s;
      if (h < gq) {
        m_run[s] = mw[s];
        l_run[s] = (n == 0) ? lw[s] : 0.0f;   // l_run is summed over the 16 lanes at the end
#pragma unroll
        for (int ct = 0; ct < 8; ++ct) {
          const float x = s_o[wave][h][16 * ct + n];
          if constexpr (M32) om[s][ct] = x;
          else O[ct][2 * s] = x;
        }
      }
    }
    wave_lds_fence();
  }
  // this wave's operand tables start as zeros (rows of absent heads stay zero), behind the window's stay there
  for (int i = lane; i < 16 * TABW / 8; i += 64) {
    reinterpret_cast<uint4*>(&s_A[wave][0][0])[i] = make_uint4(0u, 0u, 0u, 0u);
    reinterpret_cast<uint4*>(&s_P[wave][0][0])[i] = make_uint4(0u, 0u, 0u, 0u);
  }
  // The first page's value side is asked for only now, behind the query rotation and the
  // residual window: all waves of the grid
  // ask for their first page at the same moment, and with the key side of every wave ahead of
  // every value side in the memory system's queues the first logits start earlier (about 1 %
  // on the small-batch workloads, nothing on the others).
  __builtin_amdgcn_sched_barrier(0);
  vr.load(first, lane);
  __builtin_amdgcn_sched_barrier(0);
  // rotated queries -> operand order, through the same wave-local slice
#pragma unroll
  for (int s = 0; s < HP; ++s) {
    const int h = q4 + 4 * s;
    if (h < gq) {
      *reinterpret_cast<float4*>(&s_o[wave][h][8 * cg]) = make_float4(qh[s][0], qh[s][1], qh[s][2], qh[s][3]);
      *reinterpret_cast<float4*>(&s_o[wave][h][8 * cg + 4]) = make_float4(qh[s][4], qh[s][5], qh[s][6], qh[s][7]);
    }
  }
  wave_lds_fence();

  // ---- per-lane constants ----
  // writer role for the key operand: positions 8n..8n+7 of heads q4 (+4)
  float qr[HP][8], qs[HP][8], ps[HP];
#if OSCAR_LIMBS_PACKED
  [[maybe_unused]] uint4 qsh[HP], qsl[HP];   // qs as fp16 limbs
#endif
#pragma unroll
  for (int s = 0; s < HP; ++s) {
    const int h = q4 + 4 * s;
    float mx = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int chan = 32 * (n >> 2) + slot_index(BITS, n & 3, i);
      qr[s][i] = (h < gq) ? s_o[wave][h][chan] : 0.0f;
      mx = fmaxf(mx, fabsf(qr[s][i]));
    }
    mx = row16_max(mx);
    int ex = 0;
    (void)frexpf(mx, &ex);           // mx < 2^ex
    if (mx == 0.0f) ex = 0;
    // |Q_h| * 2^(xh - bitpos) < 2^14 for every slot, and Delta_k <= 1
    const int xh = 14 + slot_bitpos_min(BITS) - ex;
#pragma unroll
    for (int i = 0; i < 8; ++i) qs[s][i] = ldexpf(qr[s][i], xh - slot_bitpos(BITS, n & 3, i));
    ps[s] = ldexpf(1.0f, 24 - xh);
#if OSCAR_LIMBS_PACKED
    if constexpr (!M32) split_to_halves(qs[s], qsh[s], qsl[s]);
#endif
    if constexpr (HP == 2) {
      s_qr[wave][s][0][lane] = make_float4(qr[s][0], qr[s][1], qr[s][2], qr[s][3]);
      s_qr[wave][s][1][lane] = make_float4(qr[s][4], qr[s][5], qr[s][6], qr[s][7]);
    }
  }
  // value side: this lane's tokens 16*T+n feed k-step n/4, element T
  float vsc0[8];
#pragma unroll
  for (int T = 0; T < 8; ++T)
    vsc0[T] = ldexpf(1.0f, slot_bitpos_min(BITS) - slot_bitpos(BITS, n >> 2, T));

  [[maybe_unused]] float vup[8];   // 1 / vsc0
#pragma unroll
  for (int T = 0; T < 8; ++T) vup[T] = ldexpf(1.0f, slot_bitpos(BITS, n >> 2, T) - slot_bitpos_min(BITS));

  Masks<BITS> masks;
  masks.init();
  OSCAR_STAMP(4);   // prologue done
  _Float16(*A_tab)[TABW] = s_A[wave];
  _Float16(*P_tab)[TABW] = s_P[wave];

  // Issue priority follows what is left to do.  Two workgroups share a CU, so every SIMD holds
  // one wave of each; between waves of equal priority the older one wins every issue slot it
  // can use, and the younger workgroup ran at 40 % of the older one's pace until that one was
  // done, then finished alone, without a partner to hide its stalls behind.  A wave therefore
  // lowers its priority as it gets through its pages (quarter by quarter): whichever wave of a
  // SIMD is behind is served first, and the two finish together.
  const int n_iter = pg_first < n_pages ? (n_pages - pg_first + pstride - 1) / pstride : 0;
  const int prio_step = max(1, (n_iter + 3) >> 2);
  int prio_next = prio_step, prio_level = 0;

  // Iterations come in chunks of 63: an iteration asks for the page of the next one, and the 64th entry
  // of the register is the first of the following chunk.  (A second register for that entry, loaded
  // behind the first page's loads and waited for in front of the loop, held the first logits back until
  // the whole page was there, value side included.)
  for (int it0 = 0; pg_first + pstride * it0 < n_pages; it0 += 63) {
  if (it0 > 0) {
    tab = load_table(it0);
    // touch the register here, so the wait for this load sits outside the page loop (inside it, it would
    // also wait for every prefetch in flight)
    asm volatile("" ::"v"(tab));
  }
  const int it_end = min(63, (n_pages - pg_first - pstride * it0 + pstride - 1) / pstride);
  for (int iti = 0; iti < it_end; ++iti) {
    const int pg = pg_first + pstride * (it0 + iti);
    OSCAR_STAMP(8 + min(it0 + iti, 15));   // top of page iteration 0..15
    if (OSCAR_DECODE_PRIORITY && it0 + iti == prio_next) {
      prio_next += prio_step;
      ++prio_level;
      if (prio_level == 1) __builtin_amdgcn_s_setprio(2);
      else if (prio_level == 2) __builtin_amdgcn_s_setprio(1);
      else __builtin_amdgcn_s_setprio(0);
    }
    const bool has_next = pg + pstride < n_pages;
    // entries past the wave's last page read as 0 (a valid page index) and the load is void
    const int phys = __builtin_amdgcn_readlane(tab, iti + 1);
    PageRsrc nx;   // the wave's next page
    nx.make(pools, P, (uint32_t)phys, has_next);

    // ---- q K^T ----
    float S[HP][8];
    {
      [[maybe_unused]] const uint32_t nt[4] = {kr.nr.a.x, kr.nr.a.y, kr.nr.a.z, kr.nr.a.w};
      [[maybe_unused]] float ntf[8];
      if constexpr (M32) kr.nr.floats(ntf);
#pragma unroll
      for (int g = 0; g < NGK; ++g) {
        // per channel, what one unit of Q_h takes off the logit
        float dz[8];
        zero_terms<zp_min>(kr.kd[g], kr.kz[g], dz);
        [[maybe_unused]] float kdf[8];
        if constexpr (M32) kr.kd[g].floats(kdf);
        float bias[HP];
#pragma unroll
        for (int s = 0; s < HP; ++s) {
          float bp = 0.0f;
          if constexpr (HP == 2) {
            const float4 qa = s_qr[wave][s][0][lane], qb = s_qr[wave][s][1][lane];
            const float qv[8] = {qa.x, qa.y, qa.z, qa.w, qb.x, qb.y, qb.z, qb.w};
#pragma unroll
            for (int i = 0; i < 8; ++i) bp = fmaf(qv[i], dz[i], bp);
          } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) bp = fmaf(qr[s][i], dz[i], bp);
          }
          bias[s] = row16_sum(bp);
          uint4 hi, lo;
          if constexpr (M32) {
            float t[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) t[i] = qs[s][i] * kdf[i];
            split_to_halves(t, hi, lo);
          }
#if OSCAR_LIMBS_PACKED
          else mul_limbs_packed(qsh[s], qsl[s], kr.kd[g].a, hi, lo);
#else
          else mul_split_hi_lo(qs[s], kr.kd[g].a, hi, lo);
#endif
          // (rows of heads past the group hold zeros either way: their queries are zero)
          const int h = q4 + 4 * s;
          *reinterpret_cast<uint4*>(&A_tab[row_hi(h)][8 * n]) = hi;
          *reinterpret_cast<uint4*>(&A_tab[row_hi(h) + 1][8 * n]) = lo;
        }
        kr.load_meta(nx, g, lane);
        wave_lds_fence();
        half8 areg[4];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
          areg[kk] = *reinterpret_cast<const half8*>(&A_tab[n][32 * q4 + 8 * kk]);
        wave_lds_fence();
        // logits of a tile pair: read one pair late, behind the next pair's matrix instructions,
        // so that nothing waits for an accumulator that is still in the matrix pipe
        auto logits = [&](int T, const float4v& a0, const float4v& a1) {
#pragma unroll
          for (int s = 0; s < HP; ++s) {
            // T is even: tokens T, T+1 are the two halves of norm word T/2
            const float l0 = fmaf(a0[2 * s] + a0[2 * s + 1], ps[s], -bias[s]);
            const float l1 = fmaf(a1[2 * s] + a1[2 * s + 1], ps[s], -bias[s]);
            if constexpr (M32) {
              S[s][T] = l0 * ntf[T];
              S[s][T + 1] = l1 * ntf[T + 1];
            } else {
              S[s][T] = mix_scale<0>(l0, nt[T >> 1]);
              S[s][T + 1] = mix_scale<1>(l1, nt[T >> 1]);
            }
          }
          keep_tuple(a0);
          keep_tuple(a1);
        };
        float4v prev0, prev1;
#pragma unroll
        for (int tt = 0; tt < TPG; tt += 2) {
          // two token tiles at a time: independent accumulators keep the MFMA pipe busy
          const int T = g * TPG + tt;
          float4v acc0 = (float4v){0.0f, 0.0f, 0.0f, 0.0f}, acc1 = acc0;
          if constexpr (!ONE_TILE) {
            u32x4 b0[4], b1[4];
            kr.kc[T >> 1].chunk(0).operands(b0, masks);
            kr.kc[T >> 1].chunk(1).operands(b1, masks);
            OSCAR_PREFETCH_FENCE();
            kr.load_codes(nx, T >> 1, lane);
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
              acc0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                  areg[kk], __builtin_bit_cast(half8, b0[kk]), acc0, 0, 0, 0);
              acc1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                  areg[kk], __builtin_bit_cast(half8, b1[kk]), acc1, 0, 0, 0);
            }
          } else {
            // one tile at a time: the second head slot needs the registers of the second
            // operand set (the other wave of the SIMD fills the matrix pipe instead)
            u32x4 b0[4];
            kr.kc[T >> 1].chunk(0).operands(b0, masks);
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
              acc0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                  areg[kk], __builtin_bit_cast(half8, b0[kk]), acc0, 0, 0, 0);
            asm volatile("" ::: "memory");
            kr.kc[T >> 1].chunk(1).operands(b0, masks);
            OSCAR_PREFETCH_FENCE();
            kr.load_codes(nx, T >> 1, lane);
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
              acc1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                  areg[kk], __builtin_bit_cast(half8, b0[kk]), acc1, 0, 0, 0);
          }
          if (tt > 0) logits(T - 2, prev0, prev1);
          prev0 = acc0;
          prev1 = acc1;
        }
        logits(g * TPG + TPG - 2, prev0, prev1);
      }
    }
    kr.load_norm(nx, lane);
    if (it0 + iti == 0) OSCAR_STAMP(5);   // first page's logits done

    // ---- online softmax (per head slot; the 16 lanes of a group share a head) ----
    float alpha[HP];
    bool rescale = false;
#pragma unroll
    for (int s = 0; s < HP; ++s) {
      float mx = S[s][0];
#pragma unroll
      for (int T = 1; T < 8; ++T) mx = fmaxf(mx, S[s][T]);
      const float m_new = fmaxf(m_run[s], row16_max_fast(mx));
      alpha[s] = __builtin_amdgcn_exp2f(m_run[s] - m_new);
      rescale |= (m_new != m_run[s]);
      m_run[s] = m_new;
      float sum = 0.0f;
#pragma unroll
      for (int T = 0; T < 8; ++T) {
        S[s][T] = __builtin_amdgcn_exp2f(S[s][T] - m_new);  // S now holds p
        sum += S[s][T];
      }
      l_run[s] = l_run[s] * alpha[s] + sum;
    }

    if constexpr (M32) {
      // ---- fp32 metadata: P V of this page on its own, then added to the output ----
      // The plain-ALU kernel forms Delta*(c - z) code by code in fp32; this one has to lose no more.
      // sum p*Delta*c and sum p*Delta*z are each many times their difference (c is near z for most
      // channels of a group that holds an outlier), so the page's sums start from zero accumulators
      // and both come from the same limbs on one grid (grid_limbs): the high limbs' sums are then
      // exact, in the matrix core as in the vector unit, and so is their difference.  Limbs rounded to
      // their own exponents lost the low bits of every small product beside a large one (a matrix
      // instruction aligns its products to the largest nominal exponent, for codes held as subnormals
      // up to 2^10 above their value): 3e-6 of sum p*Delta*z where the softmax is peaked.
      // The limbs of a product are off by 2^-24 of the grid's range, so the range is that of the
      // head's largest p*Delta of this page and value group: such an error is far below that token's
      // own step, whatever the other tokens, groups and heads hold.  (With one range for the page, set
      // by its largest step, a group or a softmax peak 2^12 below it was off by 1e-4 .. 1e-3, at 2^30
      // by 2e-2 and more, and an infinite step cleared the other groups.)
      // What the limbs multiply is c - zc with an integer zc among the codes; the rest of the
      // zero-point (a group whose values share a sign lies off zero by any number of steps, a float
      // zero-point between two) cancels against nothing and is weighted with the probabilities as
      // they are, in the vector unit.
      // (The own ranges and the split zero-point cost 1 .. 11 % of the time: attention alone, batch 4 x 8K,
      // INT2, G_k = 128, G_v = 32, 14.6 -> 15.7 us at GQA 4, 18.9 -> 20.8 at GQA 7.)
      constexpr float kz = 1.0f / (float)(1 << (24 - slot_bitpos_min(BITS)));   // limbs -> accumulator
      constexpr float qmax = (float)((1 << BITS) - 1);
      if (__any(rescale)) {
#pragma unroll
        for (int s = 0; s < HP; ++s)
#pragma unroll
          for (int ct = 0; ct < 8; ++ct) om[s][ct] *= alpha[s];
      }
#pragma unroll
      for (int g = 0; g < NGV; ++g) {
        float vdf[8], vzf[8], zcw[8], rest[8];   // value = Delta * (c - zc) + rest
        vr.vd[g].floats(vdf);
        vr.vz[g].floats(vzf);
#pragma unroll
        for (int T = 0; T < 8; ++T) {
          float zc;
          if constexpr (zp_min) {
            // (any integer will do, so the hardware's reciprocal does)
            zc = __builtin_amdgcn_fmed3f(rintf(-vzf[T] * __builtin_amdgcn_rcpf(vdf[T])), 0.0f, qmax);
            rest[T] = fmaf(vdf[T], zc, vzf[T]);
          } else {
            zc = __builtin_amdgcn_fmed3f(vzf[T], 0.0f, qmax);
            rest[T] = vdf[T] * (zc - vzf[T]);
          }
          zcw[T] = zc * vup[T];   // (the limbs carry the slots' weights, the zero-points take them back)
        }
        float zh[HP], zl[HP];
        int unscale_exp[HP];
#pragma unroll
        for (int s = 0; s < HP; ++s) {
          float t[8], gr[8], re[8];
          uint4 hi, lo;
          // (positive fp32 numbers order like their bit patterns; the exponent field E bounds the
          // largest product by 2^(E - 126))
          uint32_t tm = 0;
          float sh = 0.0f, sl = 0.0f, sx = 0.0f;
#pragma unroll
          for (int T = 0; T < 8; ++T) {
            t[T] = S[s][T] * vdf[T];
            tm = max(tm, __float_as_uint(t[T]));
            sx = fmaf(S[s][T], rest[T], sx);
          }
          const int xv = 139 - (int)(row16_max_u32(tm) >> 23);   // p * Delta_v * 2^xv < 2^13
          unscale_exp[s] = 24 - slot_bitpos_min(BITS) - xv;
#pragma unroll
          for (int T = 0; T < 8; ++T) t[T] = ldexpf(t[T], xv) * vsc0[T];
          grid_limbs(t, vsc0, gr, re, hi, lo);
          const int h = q4 + 4 * s;
          *reinterpret_cast<uint4*>(&P_tab[row_hi(h)][8 * n]) = hi;
          *reinterpret_cast<uint4*>(&P_tab[row_hi(h) + 1][8 * n]) = lo;
#pragma unroll
          for (int T = 0; T < 8; ++T) {
            sh = fmaf(gr[T], zcw[T], sh);
            sl = fmaf(re[T], zcw[T], sl);
          }
          zh[s] = row16_sum(sh) * kz;
          zl[s] = row16_sum(fmaf(sl, kz, -ldexpf(sx, -unscale_exp[s])));
        }
        vr.load_delta(nx, g, lane);
        wave_lds_fence();
        half8 preg[4];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
          preg[kk] = *reinterpret_cast<const half8*>(&P_tab[n][8 * (4 * kk + q4)]);
        wave_lds_fence();
        auto add_tile = [&](int ct, const float4v& a) {
#pragma unroll
          for (int s = 0; s < HP; ++s)
            om[s][ct] += ldexpf((a[2 * s] - zh[s]) + (a[2 * s + 1] - zl[s]), unscale_exp[s]);
          keep_tuple(a);
        };
        float4v prev = (float4v){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int cc = 0; cc < CPG; ++cc) {
          const int ct = g * CPG + cc;
          u32x4 b0[4];
          vr.vc[ct >> 1].chunk(ct & 1).operands(b0, masks);
          OSCAR_PREFETCH_FENCE();
          if (ct & 1) vr.load_codes(nx, ct >> 1, lane);
          float4v acc = (float4v){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int kk = 0; kk < 4; ++kk)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                preg[kk], __builtin_bit_cast(half8, b0[kk]), acc, 0, 0, 0);
          if (cc > 0) add_tile(ct - 1, prev);   // one tile late: its result has left the matrix pipe
          prev = acc;
        }
        add_tile(g * CPG + CPG - 1, prev);
      }
    } else {
      // ---- scale of the value operand for this page: Delta_v * 2^xv < 2^13 ----
      uint4 dm = vr.vd[0].a;
#pragma unroll
      for (int g = 1; g < NGV; ++g) dm = pk_max4(dm, vr.vd[g].a);
      // Step sizes are non-negative fp16 numbers: the largest has the largest bit pattern, and its
      // exponent field E bounds it by 2^(E - 14) (2^-14 for E = 0: zero or subnormal steps)
      const uint32_t dm2 = pk_max_u16(pk_max_u16(dm.x, dm.y), pk_max_u16(dm.z, dm.w));
      const uint32_t dbits = row16_max_u32(max(dm2 & 0xffffu, dm2 >> 16));  // the 16 lanes of a head group cover all 128 tokens
      const int xv = 27 - (int)(dbits >> 10);
      rescale |= (xv != xv_cur);
      if (__any(rescale)) {
        float f[HP];
#pragma unroll
        for (int s = 0; s < HP; ++s) f[s] = ldexpf(alpha[s], xv - xv_cur);
#pragma unroll
        for (int ct = 0; ct < 8; ++ct) {
#pragma unroll
          for (int s = 0; s < HP; ++s) {
            O[ct][2 * s] *= f[s];
            O[ct][2 * s + 1] *= f[s];
          }
        }
#pragma unroll
        for (int s = 0; s < HP; ++s)
#pragma unroll
          for (int g = 0; g < NGV; ++g) bv[s][g] *= alpha[s];
      }
      xv_cur = xv;

      // ---- P V, one value group at a time through the wave's LDS table ----
      [[maybe_unused]] const float pscale = ldexpf(1.0f, xv);
      float pc[HP][8];   // p * 2^(xv - slot offset): the value operand before Delta_v
#pragma unroll
      for (int s = 0; s < HP; ++s)
#pragma unroll
        for (int T = 0; T < 8; ++T)
          pc[s][T] = S[s][T] * (vsc0[T] * (OSCAR_LIMBS_PACKED ? 16384.0f : pscale));
#if OSCAR_LIMBS_PACKED
      // The probabilities are split as p * 2^14 (at most 2^14, whatever the page's step sizes
      // are); the rest of the page's power of two goes to the step sizes, whose largest then
      // sits in [2^-2, 2^-1): an exact scaling unless a step size is 2^12 times smaller than
      // the page's largest.
      uint4 pch[HP], pcl[HP];
#pragma unroll
      for (int s = 0; s < HP; ++s) split_to_halves(pc[s], pch[s], pcl[s]);
      const _Float16 ysc = (_Float16)ldexpf(1.0f, xv - 14);
      const half2v ysc2 = {ysc, ysc};
#endif
#pragma unroll
      for (int g = 0; g < NGV; ++g) {
        float dz[8];
        zero_terms<zp_min>(vr.vd[g], vr.vz[g], dz);
#if OSCAR_LIMBS_PACKED
        const uint4 yd = scale_halves(vr.vd[g].a, ysc2);
#endif
#pragma unroll
        for (int s = 0; s < HP; ++s) {
          float acc_b = 0.0f;
#pragma unroll
          for (int T = 0; T < 8; ++T) acc_b = fmaf(S[s][T], dz[T], acc_b);
          bv[s][g] += acc_b;
          uint4 hi, lo;
#if OSCAR_LIMBS_PACKED
          mul_limbs_packed(pch[s], pcl[s], yd, hi, lo);
#else
          mul_split_hi_lo(pc[s], vr.vd[g].a, hi, lo);
#endif
          // (heads past the group produce finite values in rows nobody reads back)
          const int h = q4 + 4 * s;
          *reinterpret_cast<uint4*>(&P_tab[row_hi(h)][8 * n]) = hi;
          *reinterpret_cast<uint4*>(&P_tab[row_hi(h) + 1][8 * n]) = lo;
        }
        vr.load_delta(nx, g, lane);
        wave_lds_fence();
        half8 preg[4];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
          preg[kk] = *reinterpret_cast<const half8*>(&P_tab[n][8 * (4 * kk + q4)]);
        wave_lds_fence();
#pragma unroll
        for (int cc = 0; cc < CPG; cc += 2) {
          const int ct = g * CPG + cc;
          if constexpr (!ONE_TILE) {
            u32x4 b0[4], b1[4];
            vr.vc[ct >> 1].chunk(0).operands(b0, masks);
            vr.vc[ct >> 1].chunk(1).operands(b1, masks);
            OSCAR_PREFETCH_FENCE();
            vr.load_codes(nx, ct >> 1, lane);
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
              O[ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                  preg[kk], __builtin_bit_cast(half8, b0[kk]), O[ct], 0, 0, 0);
              O[ct + 1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                  preg[kk], __builtin_bit_cast(half8, b1[kk]), O[ct + 1], 0, 0, 0);
            }
          } else {
            u32x4 b0[4];
            vr.vc[ct >> 1].chunk(0).operands(b0, masks);
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
              O[ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                  preg[kk], __builtin_bit_cast(half8, b0[kk]), O[ct], 0, 0, 0);
            asm volatile("" ::: "memory");
            vr.vc[ct >> 1].chunk(1).operands(b0, masks);
            OSCAR_PREFETCH_FENCE();
            vr.load_codes(nx, ct >> 1, lane);
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
              O[ct + 1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                  preg[kk], __builtin_bit_cast(half8, b0[kk]), O[ct + 1], 0, 0, 0);
          }
        }
      }
    }
    // The zero-points of the next page are fetched last, when every temporary of the
    // iteration is dead: fetched where they are consumed (inside the value groups), the
    // compiler parked the arriving registers elsewhere and moved half of each to its home
    // straight away, which made the wave wait for loads it had just issued.
#pragma unroll
    for (int g = 0; g < NGV; ++g) vr.load_zero(nx, g, lane);
  }
  }

#pragma unroll
  for (int ct = 0; ct < 8; ++ct) keep_tuple(O[ct]);
  OSCAR_STAMP(24);   // page loop done
  if (OSCAR_DECODE_PRIORITY) __builtin_amdgcn_s_setprio(0);
  // ---- wave results -> LDS ----
  {
    [[maybe_unused]] const float unscale = ldexpf(1.0f, 24 - xv_cur - slot_bitpos_min(BITS));
#pragma unroll
    for (int s = 0; s < HP; ++s) {
      const int h = q4 + 4 * s;
      const float l_tot = row16_sum(l_run[s]);
      float bvt[NGV];
#pragma unroll
      for (int g = 0; g < NGV; ++g) bvt[g] = row16_sum(bv[s][g]);
      if (h < gq) {
#pragma unroll
        for (int ct = 0; ct < 8; ++ct)
          s_o[wave][h][16 * ct + n] =
              M32 ? om[s][ct] : (O[ct][2 * s] + O[ct][2 * s + 1]) * unscale - bvt[ct / CPG];
        if (n == 0) {
          s_wm[wave][h] = m_run[s];
          s_wl[wave][h] = l_tot;
        }
      }
    }
  }

  // ---- merge the wave states and the residual state, write the split's record ----
  OSCAR_STAMP(25);   // wave results in LDS
  __syncthreads();
  OSCAR_STAMP(26);   // all waves there
  // a thread owns one channel of every second head (the head parity is wave-uniform, so no
  // lane idles); the reads of a head are independent and go out together
  const int ch = tid & (D - 1), hh = __builtin_amdgcn_readfirstlane(tid >> 7);
  // With a single split the record is the result: the host passes the output tensor and
  // launches no reduce pass.  acc / L below are the record's own numbers, divided as the
  // reduce pass divides them, so both routes give the same bits.
  const bool direct = P.out != nullptr;
#pragma unroll
  for (int k = 0; k < OSCAR_MAX_GQA / (NW / 2); ++k) {
    const int h = hh + NW / 2 * k;
    if (h < gq) {
      float m[NW], o[NW];
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        m[w] = s_wm[w][h];
        o[w] = s_o[w][h][ch];
      }
      float M = m[0];
#pragma unroll
      for (int w = 1; w < NW; ++w) M = fmaxf(M, m[w]);
      float acc = 0.0f;
      if (M != -INFINITY) {
#pragma unroll
        for (int w = 0; w < NW; ++w)
          if (m[w] != -INFINITY) acc += o[w] * __builtin_amdgcn_exp2f(m[w] - M);
      }
      const size_t unit = (size_t)b * Hq + (size_t)kvh * gq + h;
      if (direct) {
        float L = 0.0f;
        if (M != -INFINITY) {
#pragma unroll
          for (int w = 0; w < NW; ++w)
            if (m[w] != -INFINITY) L += s_wl[w][h] * __builtin_amdgcn_exp2f(m[w] - M);
        }
        const float res = L > 0.0f ? acc / L : 0.0f;
        const size_t oi = unit * D + ch;
        if (P.out_dtype == OSCAR_F32) reinterpret_cast<float*>(P.out)[oi] = res;
        else if (P.out_dtype == OSCAR_BF16) reinterpret_cast<__hip_bfloat16*>(P.out)[oi] = __float2bfloat16(res);
        else reinterpret_cast<__half*>(P.out)[oi] = __float2half_rn(res);
      } else {
        P.ws[(unit * P.num_splits + split) * WS_STRIDE + ch] = acc;
      }
    }
  }
  if (!direct && tid < gq) {
    const int h = tid;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, s_wm[w][h]);
    float L = 0.0f;
    if (M != -INFINITY) {
#pragma unroll
      for (int w = 0; w < NW; ++w)
        if (s_wm[w][h] != -INFINITY) L += s_wl[w][h] * __builtin_amdgcn_exp2f(s_wm[w][h] - M);
    }
    const size_t rec = ((size_t)b * Hq + (size_t)kvh * gq + h) * P.num_splits + split;
    P.ws[rec * WS_STRIDE + D] = M;
    P.ws[rec * WS_STRIDE + D + 1] = L;
  }
#if OSCAR_MFMA_STEP
  if (P.num_splits == 1 && wave == 0) {
    const int total = (int)(gridDim.x * gridDim.y * gridDim.z);
    if (ticket_answer(my_ticket) == total - 1) {
      for (int bb = lane; bb < P.c.batch; bb += 64)
        advance_lengths(P.c.seq_lens, P.c.res_lens, bb, P.c.max_pages_per_seq);
      if (lane == 0) P.c.tickets[0] = 0;
    }
  }
#endif
  OSCAR_STAMP(27);   // split record written
}

template <int BITS, int HP>
int launch_groups(const DecodeParams& P, int gq, dim3 grid, hipStream_t st, hipEvent_t e0,
                  hipEvent_t e1) {
  const int ngk = P.g.ngk, ngv = P.g.ngv;
  constexpr bool ZPM = OSCAR_MFMA_ZPMIN != 0, M32 = OSCAR_MFMA_META32 != 0, STEP = OSCAR_MFMA_STEP != 0;
  // (see eight_waves_built)
  const bool few = (BITS == 2 || P.num_splits == 1) &&
                   (unsigned long long)grid.x * grid.y * grid.z <= (unsigned long long)oscar_compute_units();
  // the event-carrying launch only when a timer asked for it: the plain launch is what a
  // stream capture records
#define OSCAR_MFMA_LAUNCH(NK, NV, NW)                                                      \
  do {                                                                                     \
    if (e0 || e1)                                                                          \
      hipExtLaunchKernelGGL((oscar_decode_mfma_kernel<BITS, HP, NK, NV, ZPM, M32, STEP, NW>), grid,   \
                            dim3(64 * NW), 0, st, e0, e1, 0, P, gq);                       \
    else                                                                                   \
      hipLaunchKernelGGL((oscar_decode_mfma_kernel<BITS, HP, NK, NV, ZPM, M32, STEP, NW>), grid,      \
                         dim3(64 * NW), 0, st, P, gq);                                     \
  } while (0)
#define OSCAR_MFMA_CASE(NK, NV)                                                            \
  if (ngk == NK && ngv == NV) {                                                            \
    if constexpr (eight_waves_built(BITS, HP, NK, NV, M32)) {                              \
      if (few) {                                                                           \
        OSCAR_MFMA_LAUNCH(NK, NV, 8);                                                      \
        return OSCAR_OK;                                                                   \
      }                                                                                    \
    }                                                                                      \
    OSCAR_MFMA_LAUNCH(NK, NV, 4);                                                          \
    return OSCAR_OK;                                                                       \
  }
  OSCAR_MFMA_CASE(1, 4)
  OSCAR_MFMA_CASE(4, 4)
  OSCAR_MFMA_CASE(1, 1)
  OSCAR_MFMA_CASE(2, 2)
  OSCAR_MFMA_CASE(1, 2)
  OSCAR_MFMA_CASE(2, 1)
  OSCAR_MFMA_CASE(2, 4)
  OSCAR_MFMA_CASE(4, 1)
  OSCAR_MFMA_CASE(4, 2)
#undef OSCAR_MFMA_CASE
#undef OSCAR_MFMA_LAUNCH
  return OSCAR_ERR_UNSUPPORTED;
}

// every variant of this translation unit's zero-point form
int launch_this_form(const DecodeParams& P, int gq, dim3 grid, hipStream_t st, hipEvent_t e0,
                     hipEvent_t e1) {
  if (P.g.bits == 2)
    return gq <= 4 ? launch_groups<2, 1>(P, gq, grid, st, e0, e1) : launch_groups<2, 2>(P, gq, grid, st, e0, e1);
  if (P.g.bits == 4)
    return gq <= 4 ? launch_groups<4, 1>(P, gq, grid, st, e0, e1) : launch_groups<4, 2>(P, gq, grid, st, e0, e1);
  return OSCAR_ERR_UNSUPPORTED;
}

}  // namespace

#if defined(OSCAR_DECODE_STAMPS) && !OSCAR_MFMA_ZPMIN && !OSCAR_MFMA_META32
// [8 workgroup slots][4 waves][32 stamps] of the last stamped launch (integer zero-point variants) of the
// attention alone, and of the decode step
#if OSCAR_MFMA_STEP
#define OSCAR_READ_STAMPS oscar_debug_read_step_stamps
#else
#define OSCAR_READ_STAMPS oscar_debug_read_stamps
#endif
extern "C" int OSCAR_READ_STAMPS(void* dst, size_t bytes) {
  if (!dst || bytes != sizeof(g_stamps)) return OSCAR_ERR_INVALID_ARG;
  return hipMemcpyFromSymbol(dst, HIP_SYMBOL(g_stamps), sizeof(g_stamps)) == hipSuccess ? OSCAR_OK : OSCAR_ERR_HIP;
}
#endif

// the other translation units' entries
#define OSCAR_MFMA_FORM(NAME) \
  int NAME(const void* params, int gq, dim3 grid, hipStream_t st, hipEvent_t e0, hipEvent_t e1)
#define OSCAR_MFMA_FORM_DEFINE(NAME)                                                             \
  OSCAR_MFMA_FORM(NAME) {                                                                        \
    return launch_this_form(*reinterpret_cast<const DecodeParams*>(params), gq, grid, st, e0, e1); \
  }
#if OSCAR_MFMA_STEP && OSCAR_MFMA_ZPMIN
OSCAR_MFMA_FORM_DEFINE(oscar_launch_decode_step_this_zpmin)
#elif OSCAR_MFMA_STEP
OSCAR_MFMA_FORM_DEFINE(oscar_launch_decode_step_this)
#elif OSCAR_MFMA_META32 && OSCAR_MFMA_ZPMIN
OSCAR_MFMA_FORM_DEFINE(oscar_launch_decode_mfma_meta32_zpmin)
#elif OSCAR_MFMA_META32
OSCAR_MFMA_FORM_DEFINE(oscar_launch_decode_mfma_meta32)
#elif OSCAR_MFMA_ZPMIN
OSCAR_MFMA_FORM_DEFINE(oscar_launch_decode_mfma_zpmin)
#else
OSCAR_MFMA_FORM(oscar_launch_decode_mfma_zpmin);
OSCAR_MFMA_FORM(oscar_launch_decode_mfma_meta32);
OSCAR_MFMA_FORM(oscar_launch_decode_mfma_meta32_zpmin);
OSCAR_MFMA_FORM(oscar_launch_decode_step_this);
OSCAR_MFMA_FORM(oscar_launch_decode_step_this_zpmin);

// Test / profiling switch of oscar_debug_force_generic_decode: the only process-wide state of
// the library besides the cached device properties, one relaxed atomic flag read per launch.
static std::atomic<int> g_force_generic{0};

extern "C" int oscar_debug_force_generic_decode(int32_t on) {
  return g_force_generic.exchange(on ? 1 : 0, std::memory_order_relaxed);
}

// (see step_form_pays)
static constexpr bool one_split_step_pays(int bits, int hp, int ngk) { return !(bits == 2 && hp == 2 && ngk == 4); }

bool oscar_decode_one_split_of_eight_waves(int bits, int hp, int ngk, int ngv) {
  return eight_waves_built(bits, hp, ngk, ngv, false) && one_split_step_pays(bits, hp, ngk);
}

// Whether the matrix-core kernel is built for a configuration: group sizes 32, 64 or 128 on either
// side, keys scaled into [-1, 1], page pools below 2 GiB each.
static bool mfma_takes(const DecodeParams& P) {
  // the key operand's fixed exponent assumes Delta_k <= 1, which holds when |K_u| <= 1 (L2 or
  // maximum scaling); the un-scaled and mean-absolute-value ablations go to the generic kernel
  if (P.c.cfg.scale_mode != OSCAR_SCALE_L2 && P.c.cfg.scale_mode != OSCAR_SCALE_MAX) return false;
  if (g_force_generic.load(std::memory_order_relaxed)) return false;
  // a page is addressed as a 32-bit scalar offset into its pool
  const unsigned long long units = (unsigned long long)P.c.num_pages * (unsigned long long)P.c.cfg.n_kv_heads;
  int biggest = P.g.k_codes_bytes > P.g.v_meta_bytes ? P.g.k_codes_bytes : P.g.v_meta_bytes;
  if (P.g.k_meta_bytes > biggest) biggest = P.g.k_meta_bytes;
  return units * (unsigned long long)biggest <= 0x7FFFFFFFull;
}

// Launches the matrix-core partial pass; OSCAR_ERR_UNSUPPORTED tells the caller to use the generic
// kernel.
int oscar_launch_decode_mfma(const void* params, int gq, dim3 grid, hipStream_t st,
                             hipEvent_t e0, hipEvent_t e1) {
  const DecodeParams& P = *reinterpret_cast<const DecodeParams*>(params);
  if (!mfma_takes(P)) return OSCAR_ERR_UNSUPPORTED;
  const bool zpm = P.c.cfg.zp_mode == OSCAR_ZP_MIN;
  if (P.c.cfg.meta_dtype == OSCAR_F32)
    return zpm ? oscar_launch_decode_mfma_meta32_zpmin(params, gq, grid, st, e0, e1)
               : oscar_launch_decode_mfma_meta32(params, gq, grid, st, e0, e1);
  if (zpm) return oscar_launch_decode_mfma_zpmin(params, gq, grid, st, e0, e1);
  return launch_this_form(P, gq, grid, st, e0, e1);
}

// Whether a step takes the append inside the attention kernel or as two calls.  Inside is faster in most variants
// (1.01 .. 1.32 times, device time of 128 steps with one flush a sequence, batch 1 .. 64, 0.5K .. 32K tokens).  The
// others ran out of registers while the residual window went through them, and the lines lie where that build
// put them:
//  * five run at one workgroup a CU.  A grid of at most a workgroup a CU: 0.98 .. 1.19 times (batch 1 x
//    32K, 31 splits, 4-bit, G_k = 32, G_v = 64: 15.6 us against 18.0); a larger one: 0.80 .. 1.01.
//  * 2-bit, more than four query heads per kv head, G_k = 32 and G_v above 32, at two a CU: 1.02 .. 1.19 with
//    several splits, 0.95 .. 1.00 with one.
// Of the present kernels the inside form is the faster one beyond both lines (whole step in us, two calls as the
// rule has it / inside, the five at two workgroups a CU): 2-bit, G_k = 32, G_v = 64, 28 heads on 4, one split,
// 1 x 1000 17.0 / 15.5, 44 x 4000 31.7 / 28.2, 128 x 1000 31.1 / 26.0; G_k = G_v = 32, 128 x 1000 32.2 / 27.5; 4-bit,
// G_k = 32, G_v = 64, 32 on 8, 8 x 8000 with 8 splits 23.2 / 20.1, 64 x 4000 62.2 / 57.3; G_k = G_v = 128, 28 on 4,
// 128 x 1000 30.9 / 25.6.
static bool step_form_pays(const DecodeParams& P, int gq, dim3 grid) {
  const int hp = gq <= 4 ? 1 : 2;
  if (step_one_per_cu(P.g.bits, hp, P.g.ngk, P.g.ngv))
    return (unsigned long long)grid.x * grid.y * grid.z <= (unsigned long long)oscar_compute_units();
  return P.num_splits > 1 || one_split_step_pays(P.g.bits, hp, P.g.ngk);
}

// The same launch for a whole decode step (fp16 metadata); OSCAR_ERR_UNSUPPORTED: append and attention
// as two calls.
int oscar_launch_decode_step_mfma(const void* params, int gq, dim3 grid, hipStream_t st,
                                  hipEvent_t e0, hipEvent_t e1) {
  const DecodeParams& P = *reinterpret_cast<const DecodeParams*>(params);
  if (!mfma_takes(P) || P.c.cfg.meta_dtype != OSCAR_F16 || !step_form_pays(P, gq, grid))
    return OSCAR_ERR_UNSUPPORTED;
  return P.c.cfg.zp_mode == OSCAR_ZP_MIN ? oscar_launch_decode_step_this_zpmin(params, gq, grid, st, e0, e1)
                                         : oscar_launch_decode_step_this(params, gq, grid, st, e0, e1);
}

#endif
