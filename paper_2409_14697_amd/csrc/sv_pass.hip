// In-cache tile pass: the block-by-block all-in-cache execution of QueenV2
// (Sec. II-B "In-cache Operations", Sec. III-B) on gfx950 LDS.
//
// One block owns one tile of 2^m amplitudes: the indices that agree with the
// tile base on every non-local bit.  The tile is gathered from HBM with the
// PDEP-like deposit of its local index into the pass's local bit positions
// (Sec. III-B), so the low pinned positions give contiguous runs.  The pass's
// register stages then run in LDS: a stage gives each lane a group of 32
// (complex64) or 16 (complex128) amplitudes (5 or 4 local bits held in
// registers) and applies, as straight-line code with the bit positions
// fixed at compile time,
//   - the tensor product of one 2x2 per register bit (a layer of
//     single-qubit gates: the tensor product booster of Sec. III-A), in the
//     cheapest of four forms that holds all of them;
//   - a diagonal: one factor per register index, times per-lane factors for
//     the gates that involve bits outside the registers (a fused run of
//     phase gates, Sec. III-A, is a fixed-point phase function of the index
//     bits; its tile part is summed once per tile and stage);
//   - a permutation of the register index (X, CNOT, SWAP) at no cost: the
//     stage's LDS store writes each amplitude to its permuted address.
// The tile is written back with local bit j at physical position wpos[j],
// which fuses qubit reordering (Sec. II-B) into the store.
//
// LDS rows are 128 bytes; the element index is XOR-swizzled (low bits folded
// with every higher group of bits) so that power-of-two strides between the
// lanes of a wave fall into distinct banks.
#include <stddef.h>

#include "sv_device.h"
#include "sv_kernels.h"
#include "sv_tile_kernels.h"

namespace sv {
namespace {

constexpr int kBlock = 256;

// Register bits of a stage: 32 complex64 or 16 complex128 amplitudes per lane.
template <typename R>
struct Regs {
  static constexpr int RB = sizeof(R) == 4 ? 5 : 4;
  static constexpr int NR = 1 << RB;
};

// LDS index of local amplitude x.  Global memory moves 16-byte elements (LB
// amplitude bits inside one: 1 for complex64, 0 for complex128); the three
// element bits above them (one 128-byte row of LDS) are XORed with every
// higher group of three element bits, so that power-of-two strides between
// the lanes of a wave spread over the banks.  The map is linear over GF(2)
// and its own inverse, and keeps the amplitudes of one element together.
template <int LB>
__device__ __forceinline__ uint32_t swz(uint32_t x) {
  uint32_t y = x >> (LB + 3), h = 0;
#pragma unroll
  for (int k = 0; k < 5; ++k) h ^= y >> (3 * k);
  return x ^ ((h & 7u) << LB);
}

template <typename R>
struct dev_elem;
template <>
struct dev_elem<double> {
  typedef dbl2 E;
};
template <>
struct dev_elem<float> {
  typedef flt2 E;
};

// Program memory (pass descriptors, stages, items, matrices, batch items) is
// read-only while a pass kernel runs.  Reading it through the constant
// address space lets uniform reads go through scalar loads even where the
// compiler cannot prove that the state's stores do not alias it (the batched
// kernel takes the state and program pointers from one descriptor array).
template <typename T>
using cptr = const __attribute__((address_space(4))) T*;
// The state lives in global memory; saying so keeps its loads and stores
// global (not flat) after its pointer passed through scalar registers.
template <typename T>
using gptr = __attribute__((address_space(1))) T*;
template <typename T>
__device__ __forceinline__ gptr<T> as_global(T* p) {
  return (gptr<T>)p;
}
template <typename T>
__device__ __forceinline__ T ldg(gptr<const T> p) {
  return __builtin_nontemporal_load(p);
}
template <typename T>
__device__ __forceinline__ void stg(gptr<T> p, T v) {
  __builtin_nontemporal_store(v, p);
}

template <typename T>
__device__ __forceinline__ cptr<T> as_const(const T* p) {
  return (cptr<T>)p;
}
// A value that is the same in every lane, moved to scalar registers.
__device__ __forceinline__ uint64_t uniform64(uint64_t x) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(x >> 32));
  return ((uint64_t)hi << 32) | lo;
}
template <typename P>
__device__ __forceinline__ P uniform_ptr(P p) {
  return (P)uniform64((uint64_t)p);
}

template <typename R>
__device__ __forceinline__ cplx<R> cget(cptr<cplx<R>> M, uint32_t i) {
  return cplx<R>{M[i].re, M[i].im};
}
// Copy a program struct out of constant memory (dword by dword: the
// implicit copy constructor cannot read another address space).
template <typename T>
__device__ __forceinline__ T cload(cptr<T> p) {
  static_assert(sizeof(T) % 4 == 0, "program structs are dword multiples");
  T out;
  const __attribute__((address_space(4))) uint32_t* src = (const __attribute__((address_space(4))) uint32_t*)p;
  uint32_t* dst = reinterpret_cast<uint32_t*>(&out);
#pragma unroll
  for (unsigned i = 0; i < sizeof(T) / 4; ++i) dst[i] = src[i];
  return out;
}

// The head of a stage descriptor in scalar registers (one burst of loads; the
// store map's columns and the earlier layers are read where they are needed).
struct StageHead {
  uint32_t w[offsetof(PassStageDev, colimg) / 4];
};
static_assert(offsetof(PassStageDev, q) == 0, "q leads the head");
struct Stage {
  StageHead h;
  cptr<PassStageDev> p;
#define SV_HEAD(NAME) \
  __device__ __forceinline__ uint32_t NAME() const { return h.w[offsetof(PassStageDev, NAME) / 4]; }
  SV_HEAD(form) SV_HEAD(flags) SV_HEAD(slots) SV_HEAD(u2) SV_HEAD(dr) SV_HEAD(item_first) SV_HEAD(item_count)
  SV_HEAD(px_first) SV_HEAD(px_count) SV_HEAD(mat_base) SV_HEAD(rows) SV_HEAD(row_count) SV_HEAD(pconst)
  SV_HEAD(slot_mask) SV_HEAD(nsub) SV_HEAD(mx)
#undef SV_HEAD
  __device__ __forceinline__ uint32_t q(int b) const { return h.w[b]; }
  __device__ __forceinline__ uint32_t qsort(int b) const { return h.w[offsetof(PassStageDev, qsort) / 4 + b]; }
};
__device__ __forceinline__ Stage load_stage(cptr<PassStageDev> p) { return {cload((cptr<StageHead>)p), p}; }

// ---- the 2x2 part: one gate per register bit, in the stage's form ----------
// Each applies the 2x2 at M[0..3] to every pair of register amplitudes that
// differ in bit B (Eq. 2 on the register bits).

// General complex 2x2: 8 multiply-adds per amplitude.
template <int B, typename R>
__device__ __forceinline__ void op_u1(cplx<R>* v, cptr<cplx<R>> M) {
  constexpr int NR = Regs<R>::NR;
  const cplx<R> m0 = cget(M, 0), m1 = cget(M, 1), m2 = cget(M, 2), m3 = cget(M, 3);
#pragma unroll
  for (int r = 0; r < NR; ++r)
    if (!((r >> B) & 1)) {
      const cplx<R> a0 = v[r], a1 = v[r | (1 << B)];
      v[r] = cfma(cmul(m0, a0), m1, a1);
      v[r | (1 << B)] = cfma(cmul(m2, a0), m3, a1);
    }
}

// Real 2x2 (H, RY): 4 per amplitude.
template <int B, typename R>
__device__ __forceinline__ void op_ur(cplx<R>* v, cptr<cplx<R>> M) {
  constexpr int NR = Regs<R>::NR;
  const R m0 = cget(M, 0).re, m1 = cget(M, 1).re, m2 = cget(M, 2).re, m3 = cget(M, 3).re;
#pragma unroll
  for (int r = 0; r < NR; ++r)
    if (!((r >> B) & 1)) {
      const cplx<R> a0 = v[r], a1 = v[r | (1 << B)];
      v[r] = cplx<R>{fma(m1, a1.re, m0 * a0.re), fma(m1, a1.im, m0 * a0.im)};
      v[r | (1 << B)] = cplx<R>{fma(m3, a1.re, m2 * a0.re), fma(m3, a1.im, m2 * a0.im)};
    }
}

// Real diagonal, imaginary off-diagonal (RX, Y): (x + i y) * (i s) = -s y + i s x.
template <int B, typename R>
__device__ __forceinline__ void op_ui(cplx<R>* v, cptr<cplx<R>> M) {
  constexpr int NR = Regs<R>::NR;
  const R m0 = cget(M, 0).re, s1 = cget(M, 1).im, s2 = cget(M, 2).im, m3 = cget(M, 3).re;
#pragma unroll
  for (int r = 0; r < NR; ++r)
    if (!((r >> B) & 1)) {
      const cplx<R> a0 = v[r], a1 = v[r | (1 << B)];
      v[r] = cplx<R>{fma(-s1, a1.im, m0 * a0.re), fma(s1, a1.re, m0 * a0.im)};
      v[r | (1 << B)] = cplx<R>{fma(-s2, a0.im, m3 * a1.re), fma(s2, a0.re, m3 * a1.im)};
    }
}

// Real diagonal, complex off-diagonal (a layer mixing the two kinds above): 6.
template <int B, typename R>
__device__ __forceinline__ void op_rc(cplx<R>* v, cptr<cplx<R>> M) {
  constexpr int NR = Regs<R>::NR;
  const R m0 = cget(M, 0).re, m3 = cget(M, 3).re;
  const cplx<R> m1 = cget(M, 1), m2 = cget(M, 2);
#pragma unroll
  for (int r = 0; r < NR; ++r)
    if (!((r >> B) & 1)) {
      const cplx<R> a0 = v[r], a1 = v[r | (1 << B)];
      cplx<R> o0 = cmul(m1, a1), o1 = cmul(m2, a0);
      o0.re = fma(m0, a0.re, o0.re);
      o0.im = fma(m0, a0.im, o0.im);
      o1.re = fma(m3, a1.re, o1.re);
      o1.im = fma(m3, a1.im, o1.im);
      v[r] = o0;
      v[r | (1 << B)] = o1;
    }
}

// Dense 4x4 on register bits (1 = most significant bit of its index, 0).
template <typename R>
__device__ __forceinline__ void op_u2(cplx<R>* v, cptr<cplx<R>> M) {
  constexpr int NR = Regs<R>::NR;
#pragma unroll
  for (int r = 0; r < NR; r += 4) {
    const cplx<R> x0 = v[r], x1 = v[r | 1], x2 = v[r | 2], x3 = v[r | 3];
#pragma unroll
    for (int o = 0; o < 4; ++o) {
      cplx<R> y = cmul(cget(M, 4 * o), x0);
      y = cfma(y, cget(M, 4 * o + 1), x1);
      y = cfma(y, cget(M, 4 * o + 2), x2);
      y = cfma(y, cget(M, 4 * o + 3), x3);
      v[r | o] = y;
    }
  }
}

// The tensor product of one 2x2 per register bit (4 entries per bit, bit 0
// first): bit B in its own form (three bits of `forms` each); bits without a
// gate are skipped.
template <int B, typename R>
__device__ __forceinline__ void slot(cplx<R>* v, cptr<cplx<R>> M, uint32_t forms) {
  const uint32_t f = pass_form_of(forms, B);
  if (f == PFORM_NONE) return;
  if (f == PFORM_UR) op_ur<B>(v, M + 4 * B);
  else if (f == PFORM_UI) op_ui<B>(v, M + 4 * B);
  else if (f == PFORM_RC) op_rc<B>(v, M + 4 * B);
  else op_u1<B>(v, M + 4 * B);
}
template <typename R>
__device__ __forceinline__ void layer(cplx<R>* v, cptr<cplx<R>> M, uint32_t forms) {
  slot<0>(v, M, forms);
  slot<1>(v, M, forms);
  slot<2>(v, M, forms);
  slot<3>(v, M, forms);
  if constexpr (Regs<R>::RB > 4) slot<4>(v, M, forms);
}

// s_waitcnt with only the vector-memory counter (gfx9 encoding: expcnt and
// lgkmcnt at their no-wait values).
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// ---- FP32 products on the bf16 matrix cores --------------------------------
// The FP32 matrix instructions run at 1/16 of the bf16 rate (64 against 1024
// flops per cycle and SIMD).  An FP32 value is exactly the sum of three bf16
// values, h + m + l (the top 8 bits, the next 8 rounded to nearest, the
// rest), while the rest stays within bf16's range (see below), and products of
// bf16 values are exact in the FP32 accumulator.  h is truncated, so m reaches
// 2^-7 and l 2^-16 of an amplitude; a matrix entry's parts are all rounded and
// reach 2^-8 and 2^-17.  Of the nine part products of u x the six that reach
// 2^-17 |u x| or more are summed (smallest first); the dropped ones reach 2^-24
// |u x| (two of them) and 2^-33, 2^-23 together: two roundings of an FP32
// product at most, an eighth of 2^-24 on average (numeric model, 4e6 pairs).
// Error against FP64 for Haar 32 x 32 blocks on Gaussian columns: 5.1e-8
// relative, against 1.55e-7 for the three real FP32 products of Gauss's
// complex multiplication (measured; the accumulator rounds once per sixteen
// products instead of once per two, and Yi = P3 - P1 - P2 cancels).  Four
// real products are formed (P1 = Ur Xr, P2 = Ui Xi, Yi = Ur Xi + Ui Xr).
// An infinite or NaN amplitude leaves its whole column not finite (zero times
// infinity is not a number), as FP32 products with the 32 x 32 matrix do.  The
// layers of a tile stage mix an amplitude only with the members that their
// gates reach, so a wave with such an amplitude runs them one by one.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Range.  bf16 ends 16 binades above the last bit of the smallest FP32 values,
// so amplitudes are split as 2^16 x: exact below 2^112; beyond, the parts are
// not numbers and the results show it.  A tile stage scales its own
// amplitudes and has fragments of 2^-16 U; in a matrix pass the first stage
// scales them, the last one's fragments scale back and the others' are of U.
// These hold matrix entries from kMxSmallEntry up with all their bits; a stage
// with smaller nonzero entries is marked (kFragSmallEntries): a tile stage then
// runs on the VALU, a matrix stage has fragments 2^32 times as large and scales
// its results back, which must stay finite.  Measured: 64 VALU instructions more
// per wave and scaling stage, QFT N = 28 6.76 -> 6.83 ms (6.78 since its lane
// factors skip products with 1); brickwork N = 30 stays at 136 ms (138 with a
// scaling in every stage of a pass).
constexpr float kMxScale = 0x1p16f, kMxUnscale = 0x1p-16f;
constexpr float kMxSmallScale = 0x1p32f, kMxSmallUnscale = 0x1p-32f;
constexpr double kMxSmallEntry = 0x1p-94;

// The parts of (x, y), x in the low halves.  (v_dot2_f32_bf16 would form a
// residual without unpacking, 7 instructions per pair against 11, but it does
// not run beside a matrix instruction: 27 ns per MFMA with four of them
// interleaved against 17 ns with any of the instructions used here.)
__device__ __forceinline__ void split_bf16(float x, float y, uint32_t* h, uint32_t* m, uint32_t* l) {
  const uint32_t xb = __builtin_bit_cast(uint32_t, x), yb = __builtin_bit_cast(uint32_t, y);
  *h = __builtin_amdgcn_perm(yb, xb, 0x07060302u);  // truncated: a finite value stays finite
  x -= __builtin_bit_cast(float, xb & 0xffff0000u);
  y -= __builtin_bit_cast(float, yb & 0xffff0000u);
  const uint32_t mm = __builtin_bit_cast(uint32_t, __builtin_convertvector(flt2{x, y}, bf16x2));
  x -= __builtin_bit_cast(float, mm << 16);
  y -= __builtin_bit_cast(float, mm & 0xffff0000u);
  *m = mm;
  *l = __builtin_bit_cast(uint32_t, __builtin_convertvector(flt2{x, y}, bf16x2));
}

typedef float f32x16 __attribute__((ext_vector_type(16)));
__device__ __forceinline__ f32x16 mma_bf16(u32x4 a, u32x4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                 0);
}

// Matrix fragments of a stage: one 16-byte entry (eight columns of a row) per
// lane for part p, component c (0 real, 1 imaginary) and k-step ks.
// v_mfma_f32_32x32x16_bf16: lane l holds A[l % 32][8 (l / 32) + j] and
// B[8 (l / 32) + j][l % 32], j = 0..7 (two per register); accumulator
// register r of lane l is C[8 (r / 4) + 4 (l / 32) + r % 4][l % 32].
constexpr uint32_t frag_at(int p, int c, int ks) { return (uint32_t)(((p * 2 + c) * 2 + ks) * 64); }
static_assert(frag_at(3, 0, 0) * 16 == kStageFragBytes, "fragment size");

// One k-step of a column block: the operand fragments of its 32 columns
// (members 16 ks + 8 (l / 32) + j, which a lane holds in x[j]).
struct MxOperand {
  u32x4 re[3], im[3];  // part
};
template <bool SCALE>
__device__ __forceinline__ MxOperand mx_split(const flt2* x) {
  const float s = SCALE ? kMxScale : 1.f;
  MxOperand b;
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const flt2 x0 = x[2 * d], x1 = x[2 * d + 1];
    uint32_t p[3];
    split_bf16(s * x0.x, s * x1.x, &p[0], &p[1], &p[2]);
#pragma unroll
    for (int k = 0; k < 3; ++k) b.re[k][d] = p[k];
    split_bf16(s * x0.y, s * x1.y, &p[0], &p[1], &p[2]);
#pragma unroll
    for (int k = 0; k < 3; ++k) b.im[k][d] = p[k];
  }
  return b;
}
struct MxProducts {
  f32x16 rr = {}, ii = {}, im = {};  // Ur Xr, Ui Xi, Ur Xi + Ui Xr
};
// The part products of one k-step for NB column blocks (each A fragment is
// read once for all of them).
template <int NB>
__device__ __forceinline__ void mx_products(const MxOperand* const* b, gptr<const u32x4> fr, int ks, MxProducts* const* p) {
  constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
  for (int t = 0; t < 6; ++t) {
    const u32x4 ar = fr[frag_at(pa[t], 0, 0) + 64 * ks], ai = fr[frag_at(pa[t], 1, 0) + 64 * ks];
#pragma unroll
    for (int c = 0; c < NB; ++c) {
      p[c]->rr = mma_bf16(ar, b[c]->re[pb[t]], p[c]->rr);
      p[c]->im = mma_bf16(ar, b[c]->im[pb[t]], p[c]->im);
      p[c]->ii = mma_bf16(ai, b[c]->im[pb[t]], p[c]->ii);
      p[c]->im = mma_bf16(ai, b[c]->re[pb[t]], p[c]->im);
    }
  }
}

// Exchange the upper half of the wave's lanes of a with the lower half of b.
__device__ __forceinline__ void swap_halves(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}
__device__ __forceinline__ void swap_halves(float& a, float& b) {
  uint32_t x = __builtin_bit_cast(uint32_t, a), y = __builtin_bit_cast(uint32_t, b);
  swap_halves(x, y);
  a = __builtin_bit_cast(float, x);
  b = __builtin_bit_cast(float, y);
}

// The fragments of a stage (its `mx` entry).
__device__ __forceinline__ gptr<const u32x4> mx_frags(const void* frags, uint32_t mx) {
  return as_global(reinterpret_cast<const u32x4*>(frags)) + (size_t)(mx & ~kFragSmallEntries) * (kStageFragBytes / 16);
}
// Results x, y of fragments with small entries, scaled back; returns the largest
// magnitude (not a number if one of them is not).
__device__ __forceinline__ float mx_unscale(float largest, float& x, float& y) {
  largest = __builtin_elementwise_maximum(__builtin_elementwise_maximum(largest, __builtin_fabsf(x)), __builtin_fabsf(y));
  x *= kMxSmallUnscale;
  y *= kMxSmallUnscale;
  return largest;
}

// v <- U v for the 32 register amplitudes of every lane (all 64 lanes run
// it); false, with v undefined, if one of the wave's amplitudes is not finite
// (the zeros of U would spread it over its whole column).  A lane holds one
// column; the instruction wants 32 columns, each
// spread over two lanes: exchanging the halves of the wave turns the 64
// columns into two column blocks and the results back into columns, with
// one lane exchange per pair of registers and no LDS traffic.
__device__ __forceinline__ bool mx_apply(cplx<float>* v, const void* frags, uint32_t mx) {
  const gptr<const u32x4> fr = mx_frags(frags, mx) + (threadIdx.x & 63u);
  f32x16 p1[2], p2[2], p3[2];
#pragma unroll
  for (int cb = 0; cb < 2; ++cb) p1[cb] = p2[cb] = p3[cb] = f32x16{};
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    u32x4 br[2][3], bi[2][3];  // column block, part
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
      for (int h = 0; h < 2; ++h) {  // members 16 ks + 8 h + 2 d, + 1
        const cplx<float> x0 = v[16 * ks + 8 * h + 2 * d], x1 = v[16 * ks + 8 * h + 2 * d + 1];
        uint32_t p[3];
        split_bf16(kMxScale * x0.re, kMxScale * x1.re, &p[0], &p[1], &p[2]);
#pragma unroll
        for (int k = 0; k < 3; ++k) br[h][k][d] = p[k];
        split_bf16(kMxScale * x0.im, kMxScale * x1.im, &p[0], &p[1], &p[2]);
#pragma unroll
        for (int k = 0; k < 3; ++k) bi[h][k][d] = p[k];
      }
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        uint32_t a = br[0][k][d], b = br[1][k][d];
        swap_halves(a, b);
        br[0][k][d] = a;
        br[1][k][d] = b;
        a = bi[0][k][d];
        b = bi[1][k][d];
        swap_halves(a, b);
        bi[0][k][d] = a;
        bi[1][k][d] = b;
      }
    constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
    for (int t = 0; t < 6; ++t) {
      const u32x4 ar = fr[frag_at(pa[t], 0, ks)], ai = fr[frag_at(pa[t], 1, ks)];
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) {
        p1[cb] = mma_bf16(ar, br[cb][pb[t]], p1[cb]);
        p3[cb] = mma_bf16(ar, bi[cb][pb[t]], p3[cb]);
        p2[cb] = mma_bf16(ai, bi[cb][pb[t]], p2[cb]);
        p3[cb] = mma_bf16(ai, br[cb][pb[t]], p3[cb]);
      }
    }
    if (ks == 0) {  // the next k-step's splitting runs beside this one's products
#pragma unroll
      for (int q = 0; q < 48; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = 8 * (r / 4) + r % 4;
    float a = p1[0][r] - p2[0][r], b = p1[1][r] - p2[1][r];
    swap_halves(a, b);
    v[row].re = a;
    v[row + 4].re = b;
    a = p3[0][r];
    b = p3[1][r];
    swap_halves(a, b);
    v[row].im = a;
    v[row + 4].im = b;
  }
  // every row takes in every part of every member, and the residual of an
  // infinity is not a number: one result of the column tells
  return __builtin_amdgcn_ballot_w64(v[0].im != v[0].im) == 0;
}

// The three bf16 parts of an FP64 matrix entry, in the low halves.
__device__ __forceinline__ uint32_t bf16_bits(float x) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(flt2{x, 0.f}, bf16x2)) & 0xffffu;
}
__device__ __forceinline__ void split_entry(double x, uint32_t* p) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    p[k] = bf16_bits((float)x);
    x -= (double)__builtin_bit_cast(float, p[k] << 16);
  }
}

// Build the matrix fragments of the listed stages, one block per stage: the
// register part (4x4, layers, register factors) applied to the columns of
// the identity in FP64, or the matrix of a matrix-pass stage (the entries of
// either are FP32 numbers of the pool).  Marks the stages with small entries.
// Runs once per upload of a program; a few microseconds, latency-bound.
__global__ __launch_bounds__(kBlock) void k_stage_frags(PassStageDev* __restrict__ stages,
                                                        const uint32_t* __restrict__ list,
                                                        const cplx<float>* __restrict__ mats, uint32_t* __restrict__ frags) {
  constexpr int D = 32, NG = kBlock / D;
  __shared__ cplx<double> U[D][D + 1];
  const uint32_t e = list[blockIdx.x];
  const cptr<PassStageDev> sp = as_const(stages) + (e & kFragStage);
  const PassStageDev S = cload(sp);
  const uint32_t c = threadIdx.x % D, g = threadIdx.x / D;
  auto entry = [&](uint32_t i) { return cplx<double>{(double)mats[i].re, (double)mats[i].im}; };
  if (e & kFragMatrixStage) {
    for (uint32_t r = g; r < (uint32_t)D; r += NG) U[r][c] = entry(S.u2 + r * D + c);
  } else {
    for (uint32_t r = g; r < (uint32_t)D; r += NG) U[r][c] = cplx<double>{r == c ? 1.0 : 0.0, 0.0};
    __syncthreads();
    if (S.flags & PSF_U2) {
      static_assert(NG * 4 == D, "one quad of rows per thread");
      cplx<double> x[4], y[4];
      for (int i = 0; i < 4; ++i) x[i] = U[4 * g + i][c];
      for (int o = 0; o < 4; ++o) {
        y[o] = cmul(entry(S.u2 + 4 * o), x[0]);
        for (int i = 1; i < 4; ++i) y[o] = cfma(y[o], entry(S.u2 + 4 * o + i), x[i]);
      }
      for (int o = 0; o < 4; ++o) U[4 * g + o][c] = y[o];
      __syncthreads();
    }
    for (uint32_t li = 0; li <= S.nsub; ++li) {
      const bool last = li == S.nsub;
      const cptr<PassSubDev> subs = (cptr<PassSubDev>)((cptr<uint32_t>)sp + offsetof(PassStageDev, sub) / 4);
      const PassSubDev L = last ? PassSubDev{S.form, S.slot_mask, S.slots, (S.flags & PSF_DR) ? S.dr : kPassNoTable}
                                : cload(subs + li);
      for (int b = 0; b < 5; ++b) {
        if (pass_form_of(L.form, b) == PFORM_NONE) continue;
        const cplx<double> m0 = entry(L.slots + 4 * b), m1 = entry(L.slots + 4 * b + 1), m2 = entry(L.slots + 4 * b + 2),
                           m3 = entry(L.slots + 4 * b + 3);
        for (uint32_t p = g; p < (uint32_t)D / 2; p += NG) {
          const uint32_t r0 = ((p >> b) << (b + 1)) | (p & ((1u << b) - 1u)), r1 = r0 | (1u << b);
          const cplx<double> x0 = U[r0][c], x1 = U[r1][c];
          U[r0][c] = cfma(cmul(m0, x0), m1, x1);
          U[r1][c] = cfma(cmul(m2, x0), m3, x1);
        }
        __syncthreads();
      }
      if (L.dr != kPassNoTable) {
        for (uint32_t r = g; r < (uint32_t)D; r += NG) U[r][c] = cmul(entry(L.dr + r), U[r][c]);
        __syncthreads();
      }
    }
  }
  __syncthreads();
  bool small = false;  // nonzero entries below kMxSmallEntry
  for (uint32_t r = g; r < (uint32_t)D; r += NG)
    for (const double x : {U[r][c].re, U[r][c].im}) small = small || (x != 0.0 && fabs(x) < kMxSmallEntry);
  small = __syncthreads_or(small);
  if (small && threadIdx.x == 0) stages[e & kFragStage].mx = S.mx | kFragSmallEntries;
  const bool unscales = !(e & kFragMatrixStage) || (e & kFragLastStage);
  const double scale = (unscales ? (double)kMxUnscale : 1.0) * (small ? (double)kMxSmallScale : 1.0);
  uint32_t* out = frags + (size_t)blockIdx.x * (kStageFragBytes / 4);
  for (uint32_t f = threadIdx.x; f < 512; f += kBlock) {  // k-step, lane, register of the fragment
    const uint32_t ks = f / 256, l = (f / 4) % 64, d = f % 4;
    const cplx<double> a = U[l % 32][16 * ks + 8 * (l / 32) + 2 * d], b = U[l % 32][16 * ks + 8 * (l / 32) + 2 * d + 1];
    uint32_t x[3], y[3];
    split_entry(scale * a.re, x);
    split_entry(scale * b.re, y);
    for (int p = 0; p < 3; ++p) out[(frag_at(p, 0, 0) + ks * 64 + l) * 4 + d] = x[p] | (y[p] << 16);
    split_entry(scale * a.im, x);
    split_entry(scale * b.im, y);
    for (int p = 0; p < 3; ++p) out[(frag_at(p, 1, 0) + ks * 64 + l) * 4 + d] = x[p] | (y[p] << 16);
  }
}

// Angle words of the phase ladder: fixed-point turns, summed modulo one turn.
template <typename R>
struct lp_word;
template <>
struct lp_word<float> {
  typedef uint32_t W;
  typedef int32_t S;
  static __device__ __forceinline__ cplx<float> phase(W t) {
    float s, c;
    sincospif((float)(S)t * 0x1p-31f, &s, &c);  // angle 2 pi t / 2^32, as (-1, 1] half turns
    return cplx<float>{c, s};
  }
};
template <>
struct lp_word<double> {
  typedef uint64_t W;
  typedef int64_t S;
  static __device__ __forceinline__ cplx<double> phase(W t) {
    double s, c;
    sincospi((double)(S)t * 0x1p-63, &s, &c);
    return cplx<double>{c, s};
  }
};

// Sum of the local words (ladder layout) of the lane's set local bits.
template <typename R>
__device__ __forceinline__ typename lp_word<R>::W lp_local(cptr<typename lp_word<R>::W> words, uint32_t lsel) {
  typedef typename lp_word<R>::W W;
  // words in chunks of 8 (one scalar load each; the loop stays rolled so
  // that only one chunk is live in scalar registers)
  constexpr int CH = 8;
  static_assert(kPassLPLocalBits % CH == 0, "local words come in whole chunks");
  W t = 0;
#pragma unroll 1
  for (int c = 0; c < kPassLPLocalBits / CH; ++c, lsel >>= CH) {
#pragma unroll
    for (int b = 0; b < CH; ++b) {
      const W w = words[CH * c + b];
      t += ((lsel >> b) & 1) ? w : W(0);
    }
  }
  return t;
}

// Tile rows of a fixed-point item (entries of the stage's row table).
__device__ __forceinline__ uint32_t item_rows(const PassItemDev& it) {
  if (it.type == PIT_LP) return 1u;
  if (it.type == PIT_QG) return 1u + __builtin_popcount(it.a) + __builtin_popcountll(it.tt);
  return 0u;
}

// PIT_LP: the phase of the lane's amplitudes whose register bit `a` is 1:
// the constant word and the words of the lane's set local group bits (xg
// has zeros at the register positions) -- the lane's part, the same for
// every tile -- plus the row's tile sum (ts[0], the same in every lane).
template <typename R>
__device__ __forceinline__ typename lp_word<R>::W lp_lane_part(const PassItemDev& it, cptr<cplx<R>> M, uint32_t xg) {
  typedef typename lp_word<R>::W W;
  const cptr<W> words = (cptr<W>)M;
  return words[kPassLPConst] + lp_local<R>(words, xg & it.lmask);
}

// PIT_QG: row 0 and the constant, then the rows of the local targets set in
// the lane, then the tile-target rows (their tile sums are zero unless the
// target bit is set).  The lane's part is the constant and the local words
// of row 0 and of the set local targets' rows; the tile part is the tile
// sums of row 0, of those rows and of the tile-target rows.
template <typename R>
__device__ __forceinline__ typename lp_word<R>::W qg_lane_part(const PassItemDev& it, cptr<cplx<R>> M, uint32_t xg) {
  typedef typename lp_word<R>::W W;
  cptr<W> words = (cptr<W>)M;
  const uint32_t lsel = xg & it.lmask;
  W t = words[kPassLPConst] + lp_local<R>(words, lsel);
#pragma unroll 1
  for (uint32_t lt = it.a; lt; lt &= lt - 1u) {
    words += kPassLPWords;
    const W h = lp_local<R>(words, lsel);
    t += ((xg >> __builtin_ctz(lt)) & 1u) ? h : W(0);
  }
  return t;
}
template <typename R>
__device__ __forceinline__ typename lp_word<R>::W qg_tile_part(const PassItemDev& it, uint32_t xg,
                                                                const typename lp_word<R>::W* ts) {
  typedef typename lp_word<R>::W W;
  W t = ts[0];
  uint32_t k = 1;
#pragma unroll 1
  for (uint32_t lt = it.a; lt; lt &= lt - 1u, ++k) t += ((xg >> __builtin_ctz(lt)) & 1u) ? ts[k] : W(0);
  const uint32_t end = item_rows(it);
#pragma unroll 1
  for (; k < end; ++k) t += ts[k];
  return t;
}

// Fixed-point phase items whose lane parts a block computes once, before its
// tiles (k_pass): pre[k][t] holds the lane part of the pass's k-th such item
// for thread t.  Later items compute theirs per tile.
template <typename R>
struct pre_cap {
  static constexpr int N = sizeof(R) == 4 ? 14 : 6;
};

// Tile sums of the stage's fixed-point rows into ts[] (all threads; ends
// with a barrier).  Each thread sums whole rows: its 34 tile words are
// independent loads, so they are in flight together.
template <typename R>
__device__ __forceinline__ void stage_rows(const Stage& S, cptr<cplx<R>> mats, uint64_t base,
                                           typename lp_word<R>::W* ts) {
  typedef typename lp_word<R>::W W;
  const cptr<cplx<R>> sm = mats + S.mat_base();
  const cptr<uint32_t> rt = (cptr<uint32_t>)(sm + S.rows());
  const uint32_t rows = S.row_count();
  for (uint32_t j = threadIdx.x; j < rows; j += kBlock) {
    const uint32_t word = rt[4 * j], pred = rt[4 * j + 1];
    const uint64_t sel = base & (rt[4 * j + 2] | ((uint64_t)rt[4 * j + 3] << 32));
    const cptr<W> w = (cptr<W>)sm + word;
    W acc = 0;
#pragma unroll
    for (int i = 0; i < kPassLPTileBits; ++i) acc += ((sel >> i) & 1) ? w[i] : W(0);
    ts[j] = (pred == kPassRowAlways || ((base >> pred) & 1)) ? acc : W(0);
  }
  lds_sync();
}

// Value of selector code c for the lane: local bit c of its group index, or
// tile physical bit c - 64 of the tile base.
__device__ __forceinline__ uint32_t sel_bit(uint32_t c, uint32_t xg, uint64_t base) {
  return c < kPassTileSel ? (xg >> c) & 1u : (uint32_t)(base >> (c - kPassTileSel)) & 1u;
}
__device__ __forceinline__ uint32_t item_var(uint32_t sel, uint32_t xg, uint64_t base) {
  const uint32_t a = sel & 0xffu, b = (sel >> 8) & 0xffu;
  uint32_t var = a == kPassNoSel ? 0u : sel_bit(a, xg, base);
  if (b != kPassNoSel) var = (var << 1) | sel_bit(b, xg, base);
  return var;
}

// Entry `var` of a table of n <= 4 entries, loaded uniformly (scalar loads)
// and selected per lane.
template <typename R>
__device__ __forceinline__ cplx<R> pick(cptr<cplx<R>> T, uint32_t var, int n) {
  cplx<R> x = cget(T, 0);
  if (n > 1) {
    const cplx<R> y = cget(T, 1);
    x.re = (var & 1u) ? y.re : x.re;
    x.im = (var & 1u) ? y.im : x.im;
  }
  if (n > 2) {
    const cplx<R> z = cget(T, 2), w = cget(T, 3);
    const R zr = (var & 1u) ? w.re : z.re, zi = (var & 1u) ? w.im : z.im;
    x.re = (var & 2u) ? zr : x.re;
    x.im = (var & 2u) ? zi : x.im;
  }
  return x;
}

// The diagonal part with lane items (folded: without the register factors):
// per lane a factor G on all amplitudes
// and, per register bit a, factors f0[a] / f1[a] on the amplitudes whose bit
// a is 0 / 1; amplitude r is multiplied by G * prod_a f_{r_a}[a] * dr[r].
template <typename R, bool LP>
__device__ __forceinline__ void lane_diag(const Stage& S, cptr<PassItemDev> items, cptr<cplx<R>> mats,
                                          uint32_t xg, uint64_t base, const typename lp_word<R>::W* ts,
                                          const typename lp_word<R>::W* pre, uint32_t npre, uint32_t* kfix,
                                          bool folded, cplx<R>* v) {
  typedef typename lp_word<R>::W W;
  constexpr int RB = Regs<R>::RB, NR = Regs<R>::NR, HALF = NR / 2;
  const cplx<R> one = {R(1), R(0)};
  cplx<R> G = one, f0[RB], f1[RB];
#pragma unroll
  for (int b = 0; b < RB; ++b) f0[b] = f1[b] = one;
  uint32_t row = 0;  // the item's first row in ts
  const cptr<PassItemDev> ip = items + S.item_first();
  const uint32_t n_items = S.item_count();
  for (uint32_t i = 0; i < n_items; ++i) {
    const PassItemDev it = cload(ip + i);
    const cptr<cplx<R>> T = mats + it.mat;
    if (it.type == PIT_DG) {
      const uint32_t sb = (it.sel >> 8) & 0xffu;
      G = cmul(G, pick<R>(T, item_var(it.sel, xg, base), sb == kPassNoSel ? 2 : 4));
    } else if (it.type == PIT_D1) {
      const uint32_t var = item_var(it.sel, xg, base);
      const cplx<R> e0 = pick<R>(T, var << 1, 4), e1 = pick<R>(T, (var << 1) | 1u, 4);
#pragma unroll
      for (int b = 0; b < RB; ++b)
        if (it.a == (uint32_t)b) {
          f0[b] = cmul(f0[b], e0);
          f1[b] = cmul(f1[b], e1);
        }
    } else if (LP && it.type == PIT_LP) {
      const W lane = *kfix < npre ? pre[*kfix * kBlock + threadIdx.x] : lp_lane_part<R>(it, T, xg);
      ++*kfix;
      const cplx<R> p = lp_word<R>::phase(lane + ts[row]);
#pragma unroll
      for (int b = 0; b < RB; ++b)
        if (it.a == (uint32_t)b) f1[b] = cmul(f1[b], p);
      row += 1;
    } else if (LP && it.type == PIT_QG) {
      const W lane = *kfix < npre ? pre[*kfix * kBlock + threadIdx.x] : qg_lane_part<R>(it, T, xg);
      ++*kfix;
      G = cmul(G, lp_word<R>::phase(lane + qg_tile_part<R>(it, xg, ts + row)));
      row += item_rows(it);
    }
  }
  // factors of the register index over the bits below the top one, by doubling
  cplx<R> H[HALF];
  H[0] = G;
  if (S.flags() & PSF_F0) {
#pragma unroll
    for (int a = 0; a < RB - 1; ++a)
#pragma unroll
      for (int k = 0; k < (1 << a); ++k) {
        H[k | (1 << a)] = cmul(H[k], f1[a]);
        H[k] = cmul(H[k], f0[a]);
      }
  } else {
#pragma unroll
    for (int a = 0; a < RB - 1; ++a)
#pragma unroll
      for (int k = 0; k < (1 << a); ++k) H[k | (1 << a)] = cmul(H[k], f1[a]);
  }
  if (folded) {  // the register factors are part of the stage's matrix
#pragma unroll
    for (int r = 0; r < HALF; ++r) v[r + HALF] = cmul(cmul(H[r], f1[RB - 1]), v[r + HALF]);
    if (S.flags() & PSF_F0) {  // (else f0 is 1: 16 products that the stage's scaling costs)
#pragma unroll
      for (int r = 0; r < HALF; ++r) H[r] = cmul(H[r], f0[RB - 1]);
    }
#pragma unroll
    for (int r = 0; r < HALF; ++r) v[r] = cmul(H[r], v[r]);
    return;
  }
  const cptr<cplx<R>> D = mats + S.dr();
#pragma unroll
  for (int r = 0; r < HALF; ++r) {
    const cplx<R> lo = cmul(cmul(H[r], f0[RB - 1]), cget(D, r));
    const cplx<R> hi = cmul(cmul(H[r], f1[RB - 1]), cget(D, r + HALF));
    v[r] = cmul(lo, v[r]);
    v[r + HALF] = cmul(hi, v[r + HALF]);
  }
}

// Global memory is moved in 16-byte elements: one complex128 amplitude, or a
// pair of complex64 amplitudes whose local bit 0 (always physical bit 0: the
// low bits are pinned) lies inside the element.
template <typename R>
struct gelem;
template <>
struct gelem<double> {
  typedef dbl2 G;
  static constexpr int LB = 0;  // local bits inside one element
};
template <>
struct gelem<float> {
  typedef flt4 G;
  static constexpr int LB = 1;
};

// Everything a lane needs to move one tile: the pass, the state and the
// tile's base index.
template <typename R>
struct TileRef {
  typename dev_elem<R>::E* psi;
  cptr<PassDescDev> P;
  cptr<PassStageDev> stages;
  cptr<PassItemDev> items;
  cptr<cplx<R>> mats;
  const void* frags;  // matrix fragments of the program's stages (complex64)
  uint64_t base;
};

template <typename R>
__device__ __forceinline__ TileRef<R> tile_ref(typename dev_elem<R>::E* psi, int n, cptr<PassDescDev> P,
                                               cptr<PassStageDev> stages, cptr<PassItemDev> items,
                                               cptr<cplx<R>> mats, const void* frags, uint64_t tile_id) {
  TileRef<R> r;
  r.psi = uniform_ptr(psi);
  r.P = uniform_ptr(P);
  r.stages = uniform_ptr(stages);
  r.items = uniform_ptr(items);
  r.mats = uniform_ptr(mats);
  r.frags = uniform_ptr(frags);
  r.base = uniform64(deposit(tile_id, ((1ull << n) - 1ull) & ~r.P->lmask));
  return r;
}

constexpr int kBatch = 16;  // 16-byte elements per lane: 64 KiB tiles

// Thread geometry of a block of NT threads moving a 64 KiB tile (4096
// 16-byte elements): TB lane bits, BATCH elements per lane (UB bits).
template <int NT>
struct TileThreads {
  static_assert(NT == 256 || NT == 512, "256 or 512 threads");
  static constexpr int TB = NT == 512 ? 9 : 8;
  static constexpr int BATCH = 4096 / NT;
  static constexpr int UB = 12 - TB;
};

// Lane geometry of a tile: LDS element slot e = t + NT u (u < per) of lane t.
struct LaneGeo {
  uint32_t per;
  bool on;
  bool full;  // a 64 KiB tile: every lane moves BATCH elements
};

template <int LB, int NT = kBlock>
__device__ __forceinline__ LaneGeo lane_geo(uint32_t m) {
  const uint32_t elems = (1u << m) >> LB;
  return {elems >= (uint32_t)NT ? elems / NT : 1u, threadIdx.x < elems, elems == 4096u};
}

// Physical offset of element slot bit i when the load fills slot e with tile
// element swz(e) (amplitude index swz(e) << LB): the swizzle is linear, so
// the address of a slot is the XOR of the offsets of its set bits.  pos =
// local bit positions (lpos for the load).
template <int LB>
__device__ __forceinline__ uint64_t slot_offset(cptr<uint32_t> pos, uint32_t m, uint32_t i) {
  if (LB + i >= m) return 0ull;
  uint64_t o = 1ull << pos[LB + i];
  if (i >= 3) o ^= 1ull << pos[LB + (i - 3) % 3];
  return o;
}

// Offsets of the slot bits a lane owns (bits 0..TB-1 of its slot index).
template <int LB, int NT = kBlock>
__device__ __forceinline__ uint64_t lane_slot_bits(cptr<uint32_t> pos, uint32_t m) {
  uint64_t r = 0;
  for (uint32_t j = 0; j < (uint32_t)TileThreads<NT>::TB; ++j)
    if ((threadIdx.x >> j) & 1u) r ^= slot_offset<LB>(pos, m, j);
  return r;
}

// Issue the tile's loads straight into LDS (global_load_lds_dwordx4): slot e
// of the tile receives tile element swz(e), so the tile lands in LDS in its
// swizzled layout without passing through registers.  Each instruction of a
// wave writes 1 KiB of consecutive slots; its 64 lanes read whole 128-byte
// lines (the swizzle permutes elements within a line).  No wait.
template <typename R>
__device__ __forceinline__ void tile_load_lds(const TileRef<R>& T, typename dev_elem<R>::E* tile) {
  typedef typename gelem<R>::G G;
  constexpr int LB = gelem<R>::LB;
  const cptr<PassDescDev> P = T.P;
  const uint32_t m = P->m;
  const LaneGeo lg = lane_geo<LB>(m);
  const gptr<const G> gpsi = as_global(reinterpret_cast<const G*>(T.psi));
  const uint64_t a0 = T.base | lane_slot_bits<LB>(P->lpos, m);
  uint64_t hb[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) hb[b] = slot_offset<LB>(P->lpos, m, 8 + b);
  // the wave's first slot of instruction u: uniform (the LDS destination of
  // the instruction is wave-uniform; lanes land at consecutive 16 bytes)
  const uint32_t wslot = (threadIdx.x & ~63u);
  __attribute__((address_space(3))) G* lds = (__attribute__((address_space(3))) G*)tile;
  auto move = [&](uint32_t u) {
    uint64_t ad = a0;
#pragma unroll
    for (int b = 0; b < 4; ++b)
      if ((u >> b) & 1) ad ^= hb[b];
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(gpsi + (ad >> LB)),
                                     (__attribute__((address_space(3))) void*)(lds + wslot + u * kBlock), 16, 0, 0);
  };
  if (lg.full) {
#pragma unroll
    for (int u = 0; u < kBatch; ++u) move(u);
  } else if (lg.on) {
#pragma unroll 1
    for (uint32_t u = 0; u < lg.per; ++u) move(u);
  }
}

// The pass's register stages on the tile in LDS (ends with a barrier).
// The lane's group index in a stage: thread t's group with zeros inserted at
// the register bits (ascending positions qsort).
template <int RB>
__device__ __forceinline__ uint32_t group_bits(uint32_t gi, const Stage& S) {
  uint32_t xg = gi;
#pragma unroll
  for (int b = 0; b < RB; ++b) {
    const uint32_t q = S.qsort(b);
    xg = ((xg >> q) << (q + 1)) | (xg & ((1u << q) - 1u));
  }
  return xg;
}

// Lane parts of the pass's first fixed-point phase items (at most cap) into
// pre[k * kBlock + t]; returns how many.  Valid when every thread owns at
// most one group per stage (tiles of at most kBlock groups), as in k_pass.
template <typename R>
__device__ __forceinline__ uint32_t pre_fill(cptr<PassDescDev> P, cptr<PassStageDev> stages, cptr<PassItemDev> items,
                                             cptr<cplx<R>> mats, typename lp_word<R>::W* pre, uint32_t cap) {
  constexpr int RB = Regs<R>::RB;
  const uint32_t groups = (1u << P->m) >> RB, t = threadIdx.x;
  uint32_t k = 0;
  for (uint32_t si = 0; si < P->stage_count && k < cap; ++si) {
    const Stage S = load_stage(stages + (P->stage_first + si));
    if (!(S.flags() & PSF_LANE)) continue;
    const uint32_t xg = group_bits<RB>(t, S), n_items = S.item_count(), first = S.item_first();
    for (uint32_t i = 0; i < n_items && k < cap; ++i) {
      const PassItemDev it = cload(items + (first + i));
      if (it.type != PIT_LP && it.type != PIT_QG) continue;
      if (t < groups)
        pre[k * kBlock + t] = it.type == PIT_LP ? lp_lane_part<R>(it, mats + it.mat, xg)
                                                : qg_lane_part<R>(it, mats + it.mat, xg);
      ++k;
    }
  }
  return k;
}

// Offsets of one stage of a matrix pass: a lane's columns and members in the
// swizzled tile.
struct MxGeo {
  uint32_t sb[5];      // member bits
  uint32_t in0, out0;  // the lane's first column block: operand and result rows
  uint32_t next;       // from a wave's first column block to its second
};
// Rows a lane reads (member 16 (i / 8) + 8 (l / 32) + i % 8) and writes
// (member 8 (r / 4) + 4 (l / 32) + r % 4), lane part left out.
__device__ __forceinline__ uint32_t mx_in(const MxGeo& g, int i) {
  return ((i & 1) ? g.sb[0] : 0u) ^ ((i & 2) ? g.sb[1] : 0u) ^ ((i & 4) ? g.sb[2] : 0u) ^ ((i & 8) ? g.sb[4] : 0u);
}
__device__ __forceinline__ uint32_t mx_out(const MxGeo& g, int r) {
  return ((r & 1) ? g.sb[0] : 0u) ^ ((r & 2) ? g.sb[1] : 0u) ^ ((r & 4) ? g.sb[3] : 0u) ^ ((r & 8) ? g.sb[4] : 0u);
}
// PAIRS: member bit 0 is local bit 0, members 2 i and 2 i + 1 share a 16-byte
// slot (else local bit 0 is a lane bit: both ways the accesses spread over
// all banks).
template <bool PAIRS>
__device__ __forceinline__ void mx_read(const MxGeo& g, const flt2* tile, uint32_t at, flt2* x) {
#pragma unroll
  for (int i = 0; i < 16; i += 2) {
    if constexpr (PAIRS) {
      const flt4 v = *reinterpret_cast<const flt4*>(tile + (at ^ mx_in(g, i)));
      x[i] = flt2{v.x, v.y};
      x[i + 1] = flt2{v.z, v.w};
    } else {
      x[i] = tile[at ^ mx_in(g, i)];
      x[i + 1] = tile[at ^ mx_in(g, i + 1)];
    }
  }
}
template <bool PAIRS>
__device__ __forceinline__ void mx_write(const MxGeo& g, const MxProducts& p, uint32_t at, flt2* tile) {
#pragma unroll
  for (int r = 0; r < 16; r += 2) {
    const flt2 y0 = {p.rr[r] - p.ii[r], p.im[r]}, y1 = {p.rr[r + 1] - p.ii[r + 1], p.im[r + 1]};
    if constexpr (PAIRS) {
      *reinterpret_cast<flt4*>(tile + (at ^ mx_out(g, r))) = flt4{y0.x, y0.y, y1.x, y1.y};
    } else {
      tile[at ^ mx_out(g, r)] = y0;
      tile[at ^ mx_out(g, r + 1)] = y1;
    }
  }
}

// The results of fragments with small entries of a column block, scaled back;
// returns whether one is not finite.
__device__ __forceinline__ bool mx_unscale_block(const MxGeo& g, uint32_t at, flt2* tile) {
  float largest = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    flt2 y = tile[at ^ mx_out(g, r)];
    float re = y.x, im = y.y;
    largest = mx_unscale(largest, re, im);
    tile[at ^ mx_out(g, r)] = flt2{re, im};
  }
  return !(largest < __builtin_inff());
}

// The stage in FP32 on a column block, one product after the other, in place.
__device__ __forceinline__ void mx_stage_fp32(const MxGeo& g, cptr<cplx<float>> U, uint32_t out, flt2* tile) {
  const uint32_t half = (threadIdx.x >> 5) & 1u;
  const uint32_t col = out ^ (half ? g.sb[2] : 0u);
  const gptr<const flt2> u = as_global(reinterpret_cast<const flt2*>((uint64_t)U)) + 4 * 32 * half;
  flt2 y[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) y[r] = flt2{0.f, 0.f};
#pragma unroll 1
  for (uint32_t k = 0; k < 32; ++k) {
    uint32_t at = col;
#pragma unroll
    for (int b = 0; b < 5; ++b) at ^= ((k >> b) & 1u) ? g.sb[b] : 0u;
    const flt2 x = tile[at];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const flt2 a = u[(8 * (r / 4) + r % 4) * 32 + k];
      y[r].x = __builtin_fmaf(-a.y, x.y, __builtin_fmaf(a.x, x.x, y[r].x));
      y[r].y = __builtin_fmaf(a.y, x.x, __builtin_fmaf(a.x, x.y, y[r].y));
    }
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) tile[out ^ mx_out(g, r)] = y[r];
}

// One stage on a wave's two column blocks.  A matrix instruction (32 cycles)
// leaves room for six VALU instructions of the two waves of a SIMD (measured),
// so the second k-step is split beside the first one's products.  Both blocks
// share each A fragment: reading them once per block instead costs more than
// finishing one block early gains (N = 28, 6 stages: 2.31 against 2.20 ms).
// Returns whether the lane's columns hold what the split cannot (of the last
// stage: it shows by then).
template <bool PAIRS, bool FIRST>
__device__ __forceinline__ bool mx_stage_two(const MxGeo& g, gptr<const u32x4> fr, flt2* tile) {
  flt2 x0[16], x1[16];
  mx_read<PAIRS>(g, tile, g.in0, x0);
  mx_read<PAIRS>(g, tile, g.in0 ^ g.next, x1);
  MxProducts p0, p1;
  const MxOperand b0 = mx_split<FIRST>(x0), b1 = mx_split<FIRST>(x1);
  const MxOperand* const b[2] = {&b0, &b1};
  MxProducts* const p[2] = {&p0, &p1};
  __builtin_amdgcn_sched_barrier(0);
  mx_products<2>(b, fr, 0, p);
  const MxOperand c0 = mx_split<FIRST>(x0 + 8), c1 = mx_split<FIRST>(x1 + 8);
#pragma unroll
  for (int i = 0; i < 48; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
    __builtin_amdgcn_sched_group_barrier(0x002, FIRST ? 5 : 4, 0);  // VALU
  }
  __builtin_amdgcn_sched_barrier(0);
  const MxOperand* const c[2] = {&c0, &c1};
  mx_products<2>(c, fr, 1, p);
  __builtin_amdgcn_sched_barrier(0);
  mx_write<PAIRS>(g, p0, g.out0, tile);
  mx_write<PAIRS>(g, p1, g.out0 ^ g.next, tile);
  __builtin_amdgcn_sched_barrier(0);  // (the second block's products need not end before the first is written)
  return p0.im[0] != p0.im[0] || p1.im[0] != p1.im[0];  // as in mx_apply, one result of a column tells
}
template <bool PAIRS, bool FIRST>
__device__ __forceinline__ bool mx_stage_one(const MxGeo& g, gptr<const u32x4> fr, flt2* tile) {
  flt2 x[16];
  mx_read<PAIRS>(g, tile, g.in0, x);
  MxProducts p0;
  MxProducts* const p[1] = {&p0};
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const MxOperand b0 = mx_split<FIRST>(x + 8 * ks);
    const MxOperand* const b[1] = {&b0};
    mx_products<1>(b, fr, ks, p);
  }
  mx_write<PAIRS>(g, p0, g.out0, tile);
  return p0.im[0] != p0.im[0];
}

template <bool PAIRS, bool FIRST>
__device__ __forceinline__ bool mx_stage(bool two, const MxGeo& g, gptr<const u32x4> fr, flt2* tile) {
  return two ? mx_stage_two<PAIRS, FIRST>(g, fr, tile) : mx_stage_one<PAIRS, FIRST>(g, fr, tile);
}

// Offsets of stage S for wave w of a tile of 2^m amplitudes.  Column bit j of a
// stage is local bit colimg[j]: lane bits first, then wave bits.
__device__ __forceinline__ MxGeo mx_geo(cptr<PassStageDev> S, uint32_t m, uint32_t w) {
  constexpr int LB = 1;
  const uint32_t l = threadIdx.x & 63u;
  MxGeo g;
#pragma unroll
  for (int b = 0; b < 5; ++b) g.sb[b] = swz<LB>(1u << S->q[b]);
  uint32_t col = 0;  // the lane's column bits
#pragma unroll
  for (int j = 0; j < 5; ++j) col ^= ((l >> j) & 1u) ? swz<LB>(1u << S->colimg[j]) : 0u;
  uint32_t wc[3];  // column block bits
#pragma unroll
  for (int j = 0; j < 3; ++j) wc[j] = 5u + j < m - 5u ? swz<LB>(1u << S->colimg[5 + j]) : 0u;
  col ^= ((w & 1u) ? wc[0] : 0u) ^ ((w & 2u) ? wc[1] : 0u);
  g.in0 = col ^ (l >= 32u ? g.sb[3] : 0u);
  g.out0 = col ^ (l >= 32u ? g.sb[2] : 0u);
  g.next = wc[2];
  return g;
}

// The stages of a complex64 matrix pass.  Wave w owns the column blocks w and
// w + 4 and overwrites them in place, so stages without kMatrixStageSync
// (which keep every element with its wave) need no barrier.  A tile with
// values that the split cannot hold (amplitudes from 2^112 or not finite,
// matrix entries that are not finite, overflow beside small entries) leaves
// results that are not numbers: some lane of the last stage sees one and writes
// the tile's number `id` (nonzero, of its own) to *redo; the caller then runs
// matrix_stages_fp32.
__device__ __forceinline__ void matrix_stages(const TileRef<float>& T, flt2* tile, uint32_t id, uint32_t* redo) {
  constexpr int NW = kBlock / 64;
  const cptr<PassDescDev> P = T.P;
  const uint32_t m = P->m, ns = P->stage_count;
  const uint32_t l = threadIdx.x & 63u;
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t cblocks = 1u << (m - 10u);
  bool bad = false;
  for (uint32_t si = 0; si < ns; ++si) {
    const cptr<PassStageDev> S = T.stages + (P->stage_first + si);
    if (si > 0) {
      if (S->flags & kMatrixStageSync) {
        lds_sync();
      } else {  // the stage reads only what this wave wrote
        wait_lgkm0();
        asm volatile("" ::: "memory");
      }
    }
    const uint32_t mx = S->mx;
    const gptr<const u32x4> fr = mx_frags(T.frags, mx) + l;
    const bool first = si == 0;
    const MxGeo g = mx_geo(S, m, w);
    const bool pairs = S->q[0] == 0;
    const bool two = cblocks == 2 * NW;  // (else a small tile: one column block per wave)
    if (first) bad = pairs ? mx_stage<true, true>(two, g, fr, tile) : mx_stage<false, true>(two, g, fr, tile);
    else bad = pairs ? mx_stage<true, false>(two, g, fr, tile) : mx_stage<false, false>(two, g, fr, tile);
    if (__builtin_expect((mx & kFragSmallEntries) != 0, 0)) {
      wait_lgkm0();  // (the wave's own results)
#pragma unroll 1
      for (uint32_t cb = w; cb < cblocks; cb += NW) bad |= mx_unscale_block(g, g.out0 ^ (cb != w ? g.next : 0u), tile);
    }
  }
  if (bad) *redo = id;
  lds_sync();
}
// The tile once more, from memory and in FP32 (no lane reads the tile any more).
__device__ __forceinline__ void matrix_stages_fp32(const TileRef<float>& T, flt2* tile) {
  constexpr int NW = kBlock / 64;
  const cptr<PassDescDev> P = T.P;
  const uint32_t m = P->m, ns = P->stage_count;
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t cblocks = 1u << (m - 10u);
  tile_load_lds<float>(T, tile);
  wait_vm<0>();
  for (uint32_t si = 0; si < ns; ++si) {
    lds_sync();
    const cptr<PassStageDev> S = T.stages + (P->stage_first + si);
    const MxGeo g = mx_geo(S, m, w);
#pragma unroll 1
    for (uint32_t cb = w; cb < cblocks; cb += NW) mx_stage_fp32(g, T.mats + S->u2, g.out0 ^ (cb != w ? g.next : 0u), tile);
  }
  lds_sync();
}

// Kernel variants (each carries only the code its passes need).  LP: the
// pass holds fixed-point phase items.  MX_NONE: the register parts of its
// stages run on the VALU; MX_TILE: on the matrix cores (and on the VALU in
// waves whose amplitudes the split cannot hold); MX_ONLY: a matrix pass, whose
// stages are matrices and nothing else; MX_MIXED: MX_NONE or MX_TILE, as the
// tile's pass says.
enum { MX_NONE = 0, MX_TILE = 1, MX_ONLY = 2, MX_MIXED = 3 };

template <typename R, bool LP, int MX>
__device__ __forceinline__ void tile_stages(const TileRef<R>& T, typename dev_elem<R>::E* tile,
                                            const typename lp_word<R>::W* pre, uint32_t npre) {
  typedef typename dev_elem<R>::E E;
  constexpr int LB = gelem<R>::LB;
  const cptr<PassDescDev> P = T.P;
  const cptr<PassStageDev> stages = T.stages;
  const cptr<PassItemDev> items = T.items;
  const cptr<cplx<R>> mats = T.mats;
  const uint64_t base = T.base;
  const uint32_t size = 1u << P->m;
  const uint32_t t = threadIdx.x;
  constexpr int RB = Regs<R>::RB, NR = Regs<R>::NR;
  typedef typename lp_word<R>::W W;
  __shared__ W tsum[LP ? kPassStageRowsMax : 1];  // tile sums of the stage's fixed-point rows
  uint32_t kfix = 0;  // fixed-point phase items of the pass so far
  for (uint32_t si = 0; si < P->stage_count; ++si) {
    const Stage S = load_stage(stages + (P->stage_first + si));
    const uint32_t flags = S.flags();
    if constexpr (LP) {
      if (S.row_count()) stage_rows<R>(S, mats, base, tsum);
    }
    const uint32_t groups = size >> RB;
    // swz is linear over XOR and xg shares no bit with a register offset, so
    // swz(xg | off) = swz(xg) ^ (XOR of swz(bit) over the offset's bits): only
    // the swizzled register bits are kept, not one offset per register
    uint32_t sbit[RB], cbit[RB];
#pragma unroll
    for (int b = 0; b < RB; ++b) sbit[b] = swz<LB>(1u << S.q(b));
    // the store writes local index x to M x ^ c: register bit j of an
    // amplitude moves its address by the swizzled image of column q[j]
#pragma unroll
    for (int j = 0; j < RB; ++j) {
      uint32_t img = 1u << S.q(j);
      if (flags & PSF_PERM) img = S.p->colimg[S.q(j)];
      cbit[j] = __builtin_amdgcn_readfirstlane(swz<LB>(img));
    }
    // the constant of the map for this tile (the terms selected by tile bits)
    uint32_t cmap = S.pconst();
    for (uint32_t k = 0; k < S.px_count(); ++k) {
      const PassItemDev it = cload(items + (S.px_first() + k));
      if (sel_bit(it.sel & 0xffu, 0u, base)) cmap ^= it.a;
    }
    const bool xperm = (flags & PSF_XPERM) != 0;
    // fixed-point items of this stage (every group of the stage walks them)
    uint32_t nfix = 0;
    if constexpr (LP) {
      if (flags & PSF_LANE)
        for (uint32_t i = 0; i < S.item_count(); ++i) {
          const uint32_t ty = items[S.item_first() + i].type;
          nfix += ty == PIT_LP || ty == PIT_QG;
        }
    }
    // a tile holds at most kBlock groups: one per thread
    const bool own = t < groups;
    {
      // lanes without a group read group 0 (and store nothing)
      const uint32_t xg = own ? group_bits<RB>(t, S) : 0u;
      const uint32_t sx = swz<LB>(xg);
      cplx<R> v[NR];
      auto gather = [&](uint32_t at) {
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          uint32_t o = at;
#pragma unroll
          for (int b = 0; b < RB; ++b)
            if ((r >> b) & 1) o ^= sbit[b];
          const E e = tile[o];
          v[r] = cplx<R>{e.x, e.y};
        }
      };
      gather(sx);
      // the register part on the VALU: the 4x4, the earlier layers (2x2s, then
      // register factors), then the last one; one copy of the layer code
      // serves all layers
      auto register_part = [&](const Stage& F) {
        if (F.flags() & PSF_U2) op_u2<R>(v, mats + F.u2());
        const cptr<PassSubDev> subs = (cptr<PassSubDev>)((cptr<uint32_t>)F.p + offsetof(PassStageDev, sub) / 4);
        for (uint32_t li = 0; li <= F.nsub(); ++li) {
          const bool last = li == F.nsub();
          const PassSubDev L = last ? PassSubDev{F.form(), F.slot_mask(), F.slots(), kPassNoTable} : cload(subs + li);
          if (L.form) layer<R>(v, mats + L.slots, L.form);
          if (L.dr != kPassNoTable) {
            const cptr<cplx<R>> D = mats + L.dr;
#pragma unroll
            for (int r = 0; r < NR; ++r) v[r] = cmul(cget(D, r), v[r]);
          }
        }
      };
      bool folded = false;  // the register factors are part of the stage's matrix
      if constexpr (MX == MX_NONE) {
        register_part(S);
      } else if (S.mx() != kPassNoTable) {
        if (!(S.mx() & kFragSmallEntries)) folded = mx_apply(v, T.frags, S.mx());
        if (__builtin_expect(!folded, 0)) {
          // the tile still holds the wave's amplitudes (opaque copies: what
          // this rare branch needs does not occupy registers before it)
          uint32_t at = sx;
          asm volatile("" : "+v"(at));
          gather(at);
          cptr<PassStageDev> sp = S.p;
          asm volatile("" : "+s"(sp));
          register_part(load_stage(sp));
        }
      }
      if (flags & PSF_LANE) {
        uint32_t kf = kfix;
        lane_diag<R, LP>(S, items, mats, xg, base, tsum, pre, npre, &kf, folded, v);
      } else if (!folded && (flags & PSF_DR)) {
        const cptr<cplx<R>> D = mats + S.dr();
#pragma unroll
        for (int r = 0; r < NR; ++r) v[r] = cmul(cget(D, r), v[r]);
      }
      // address of the group's register index 0 after the map: M xg ^ c
      uint32_t so = sx;
      if (flags & PSF_PERM) {
        uint32_t y = cmap;
#pragma unroll
        for (int l = 0; l < kPassLocalMax; ++l)
          if ((xg >> l) & 1u) y ^= S.p->colimg[l];
        so = swz<LB>(y);
      }
      // a map that moves amplitudes between groups writes after every
      // group has been read
      if (xperm) lds_sync();
      // The store recomputes the offsets from opaque copies of the inputs, so
      // the compiler cannot keep NR offsets live across the stage's work.
      asm volatile("" : "+v"(so));
#pragma unroll
      for (int b = 0; b < RB; ++b) asm volatile("" : "+s"(cbit[b]));
      if (own) {
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          E e;
          e.x = v[r].re;
          e.y = v[r].im;
          uint32_t o = so;
#pragma unroll
          for (int b = 0; b < RB; ++b)
            if ((r >> b) & 1) o ^= cbit[b];
          tile[o] = e;
        }
      }
    }
    kfix += nfix;
    lds_sync();
  }
}

// The write-back: local bit j goes to physical position wpos[j], a
// permutation of the positions the tile was loaded from.  When the lowest
// element bits keep their positions lanes walk the tile in load order
// (element x = t + 256 u); otherwise they walk the destination addresses in
// the load's order (the same coalesced runs and 16-byte elements whatever the
// permutation) and gather each element from LDS: the element's k-th address
// bit holds local bit winv[k].
//
// LDS index (swizzled) of the tile's element u of this lane and, complex64,
// of the element's second amplitude.
template <typename R>
struct GatherMap {
  uint32_t xl, xo[4], xp;
  bool lane_order;
};
template <typename R>
__device__ __forceinline__ GatherMap<R> gather_map(cptr<PassDescDev> P) {
  constexpr int LB = gelem<R>::LB;
  const uint32_t m = P->m;
  // an opaque copy of the thread index: the addresses are recomputed per
  // tile instead of being kept live (or spilled) across the whole loop
  uint32_t tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  GatherMap<R> g;
  g.lane_order = (P->flags & kPassStoreLaneOrder) != 0;
  if (g.lane_order) {
    g.xl = swz<LB>(tid << LB);
#pragma unroll
    for (int b = 0; b < 4; ++b) g.xo[b] = swz<LB>(kBlock << (LB + b));
    g.xp = 1;
    return g;
  }
  uint32_t xl = 0;
#pragma unroll
  for (uint32_t jb = 0; jb < 8; ++jb) {
    const uint32_t w = LB + jb < m ? 1u << P->winv[LB + jb] : 0u;
    xl |= ((tid >> jb) & 1u) ? w : 0u;
  }
  g.xl = swz<LB>(xl);
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const uint32_t k = LB + 8 + b;
    g.xo[b] = k < m ? swz<LB>(1u << P->winv[k]) : 0u;
  }
  g.xp = LB ? swz<LB>(1u << P->winv[0]) : 0u;
  return g;
}
template <typename R>
__device__ __forceinline__ typename gelem<R>::G gather_one(const GatherMap<R>& g, const typename dev_elem<R>::E* tile,
                                                           uint32_t u) {
  typedef typename dev_elem<R>::E E;
  typedef typename gelem<R>::G G;
  uint32_t x = g.xl;
#pragma unroll
  for (int b = 0; b < 4; ++b)
    if ((u >> b) & 1) x ^= g.xo[b];
  if constexpr (gelem<R>::LB == 1) {
    // in load order both amplitudes of the element sit in one 16-byte slot
    if (g.lane_order) return *reinterpret_cast<const G*>(tile + x);
    const E e0 = tile[x], e1 = tile[x ^ g.xp];
    return G{e0.x, e0.y, e1.x, e1.y};
  } else {
    return tile[x];
  }
}

// Addresses of the lane's stores: in load order the wpos positions of the
// element's bits, in destination order the lpos positions.
template <typename R>
struct PutMap {
  uint64_t a0, hb[4];
};
template <typename R>
__device__ __forceinline__ PutMap<R> put_map(const TileRef<R>& T) {
  constexpr int LB = gelem<R>::LB;
  const cptr<PassDescDev> P = T.P;
  const uint32_t m = P->m;
  const cptr<uint32_t> pos = (P->flags & kPassStoreLaneOrder) ? P->wpos : P->lpos;
  uint32_t tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  PutMap<R> p;
  p.a0 = T.base;
#pragma unroll
  for (uint32_t j = 0; j < 8; ++j) {
    const uint64_t w = LB + j < m ? 1ull << pos[LB + j] : 0ull;
    p.a0 |= ((tid >> j) & 1u) ? w : 0ull;
  }
#pragma unroll
  for (int b = 0; b < 4; ++b) p.hb[b] = LB + 8 + b < (int)m ? 1ull << pos[LB + 8 + b] : 0ull;
  return p;
}
template <typename R>
__device__ __forceinline__ void put_one(const TileRef<R>& T, const PutMap<R>& p, uint32_t u, typename gelem<R>::G v) {
  typedef typename gelem<R>::G G;
  const gptr<G> gpsi = as_global(reinterpret_cast<G*>(T.psi));
  uint64_t ad = p.a0;
#pragma unroll
  for (int b = 0; b < 4; ++b)
    if ((u >> b) & 1) ad |= p.hb[b];
  stg<G>(gpsi + (ad >> gelem<R>::LB), v);
}

// Moves of a full tile (64 KiB: 16 elements per lane) are straight-line code,
// those of a smaller tile a loop, and lanes without a group read group 0
// instead of skipping their LDS reads: with a predicate per element every
// read was a branch of its own, its result merged with an older register, and
// the gathered elements were live (or spilled) through the whole loop.  With
// the stage heads read in one burst and the store map's columns only where
// there is a map: N = 26 passes of three QAOA levels 7.48 -> 6.37 ms
// (complex128) and 4.05 -> 3.55 ms (complex64), ten layered levels 12.4 ->
// 11.0 and 6.79 -> 5.96 ms; registers 248 -> 184 (complex128 with phase items).
//
// Persistent loop over tiles.  Per tile: the tile's loads land in LDS, the
// stages run, the result is read back into registers, and after a barrier
// the next tile's loads are issued before this tile's stores, so that the
// wait for a tile's data never waits for the previous tile's stores (the
// vector-memory counter retires in issue order).  The two blocks a CU holds
// overlap one block's memory phase with the other's stages.
template <typename R, bool LP, int MX, typename Src>
__device__ __forceinline__ void tile_loop(uint64_t total, const Src& src, typename dev_elem<R>::E* tile,
                                          const typename lp_word<R>::W* pre, uint32_t npre) {
  typedef typename gelem<R>::G G;
  uint64_t g = xcd_block();
  if (g >= total) return;
  tile_load_lds<R>(src(g), tile);
  bool full_prev = false;  // the previous tile's kBatch stores per lane follow the loads
  __shared__ uint32_t redo;  // the tile that a matrix pass computes again
  if (MX == MX_ONLY && threadIdx.x == 0) redo = 0;
  while (true) {
    const uint64_t ng = g + gridDim.x;
    const TileRef<R> cur = src(g);
    // this tile's loads are older than the previous tile's stores: when that
    // tile issued kBatch stores per lane, waiting until at most kBatch
    // operations remain waits for exactly the loads
    if (full_prev) wait_vm<kBatch>();
    else wait_vm<0>();
    lds_barrier();
    [[maybe_unused]] const uint32_t id = (uint32_t)g + 1u;
    if constexpr (MX == MX_ONLY) matrix_stages(cur, tile, id, &redo);
    // (code of its own for either: a pass rounds as it does in a launch alone)
    else if constexpr (MX != MX_MIXED) tile_stages<R, LP, MX>(cur, tile, pre, npre);
    else if (cur.P->flags & kPassMatrixStages) tile_stages<R, LP, MX_TILE>(cur, tile, pre, npre);
    else tile_stages<R, LP, MX_NONE>(cur, tile, pre, npre);
    const LaneGeo lg = lane_geo<gelem<R>::LB>(cur.P->m);
    full_prev = lg.full;
    if (lg.full) {
      G out[kBatch];
      const GatherMap<R> gm = gather_map<R>(cur.P);
      // (two arms, so that the order is a constant in each)
      if (gm.lane_order) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) out[u] = gather_one<R>(gm, tile, u);
      } else {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) out[u] = gather_one<R>(gm, tile, u);
      }
      if constexpr (MX == MX_ONLY) {  // (read beside the tile: the wait is the gather's)
        if (__builtin_expect(__builtin_amdgcn_readfirstlane(redo) == id, 0)) {
          lds_sync();
          matrix_stages_fp32(cur, tile);
#pragma unroll
          for (int u = 0; u < kBatch; ++u) out[u] = gather_one<R>(gm, tile, u);
        }
      }
      wait_lgkm0();  // this lane's LDS reads are done
      lds_barrier();
      if (ng < total) tile_load_lds<R>(src(ng), tile);
      asm volatile("" ::: "memory");  // the loads stay ahead of the stores
      const PutMap<R> pm = put_map<R>(cur);
#pragma unroll
      for (int u = 0; u < kBatch; ++u) put_one<R>(cur, pm, u, out[u]);
    } else {  // a small tile: element by element
      if constexpr (MX == MX_ONLY)
        if (__builtin_expect(__builtin_amdgcn_readfirstlane(redo) == id, 0)) {
          lds_sync();
          matrix_stages_fp32(cur, tile);
        }
      const GatherMap<R> gm = gather_map<R>(cur.P);
      const PutMap<R> pm = put_map<R>(cur);
      if (lg.on) {
#pragma unroll 1
        for (uint32_t u = 0; u < lg.per; ++u) put_one<R>(cur, pm, u, gather_one<R>(gm, tile, u));
      }
      wait_lgkm0();
      lds_barrier();
      if (ng < total) tile_load_lds<R>(src(ng), tile);
    }
    if (ng >= total) break;
    g = ng;
  }
}

template <typename R>
struct SingleSrc {
  typename dev_elem<R>::E* psi;
  int n;
  cptr<PassDescDev> P;
  cptr<PassStageDev> stages;
  cptr<PassItemDev> items;
  cptr<cplx<R>> mats;
  const void* frags;
  __device__ __forceinline__ TileRef<R> operator()(uint64_t g) const {
    return tile_ref<R>(psi, n, P, stages, items, mats, frags, g);
  }
};

template <typename R, bool LP, int MX>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_pass(
    typename dev_elem<R>::E* __restrict__ psi, int n, const PassDescDev* __restrict__ passes, int pi,
    const PassStageDev* __restrict__ stages, const PassItemDev* __restrict__ items,
    const cplx<R>* __restrict__ mats, const void* __restrict__ frags) {
  typedef typename dev_elem<R>::E E;
  extern __shared__ __align__(16) unsigned char smem[];
  E* tile = reinterpret_cast<E*>(smem);
  const cptr<PassDescDev> P = as_const(passes + pi);
  const SingleSrc<R> src{psi, n, P, as_const(stages), as_const(items), as_const(mats), frags};
  typedef typename lp_word<R>::W W;
  // lane parts of the fixed-point phase items, computed once for all tiles
  __shared__ W pre[LP ? pre_cap<R>::N * kBlock : 1];
  uint32_t npre = 0;
  if constexpr (LP) {
    npre = pre_fill<R>(P, as_const(stages), as_const(items), as_const(mats), pre, pre_cap<R>::N);
    wait_lgkm0();  // the table is complete before the first tile's barrier
  }
  tile_loop<R, LP, MX>(1ull << (n - P->m), src, tile, pre, npre);
}

// Many states in one launch: work item i runs pass `pass` of its own program
// over its own tiles; global tile g belongs to the item whose [tile_begin,
// tile_begin + tiles) range holds g.  No item reads another's state, so each
// result is independent of the batch it ran in.
template <typename R>
struct BatchSrc {
  cptr<BatchItemDev> items;
  int count;
  __device__ __forceinline__ TileRef<R> operator()(uint64_t g) const {
    int lo = 0, hi = count - 1;  // last item with tile_begin <= g
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (items[mid].tile_begin <= g) lo = mid;
      else hi = mid - 1;
    }
    lo = __builtin_amdgcn_readfirstlane(lo);  // the same in every lane
    const cptr<BatchItemDev> it = items + lo;  // fields read one by one: scalar loads
    return tile_ref<R>((typename dev_elem<R>::E*)it->psi, it->n, as_const(it->passes + it->pass),
                       as_const(it->stages), as_const(it->items), as_const((const cplx<R>*)it->mats),
                       it->frags, g - it->tile_begin);
  }
};

template <typename R, bool LP, int MX>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_pass_batch(const BatchItemDev* __restrict__ items, int count,
                                                       uint64_t total_tiles) {
  typedef typename dev_elem<R>::E E;
  extern __shared__ __align__(16) unsigned char smem[];
  E* tile = reinterpret_cast<E*>(smem);
  const BatchSrc<R> src{as_const(items), count};
  tile_loop<R, LP, MX>(total_tiles, src, tile, nullptr, 0);
}

struct PassRun {
  void* psi;
  int n, m;
  const PassDescDev* passes;
  int pass;
  const PassStageDev* stages;
  const PassItemDev* items;
  const void *mats, *frags;
  hipStream_t s;
};

template <typename R, bool LP, int MX>
hipError_t run(const PassRun& r) {
  typedef typename dev_elem<R>::E E;
  const size_t lds = ((size_t)1 << r.m) * sizeof(E);
  static KernelLaunchCache cache;
  uint64_t resident = 0;
  hipError_t e = prepare_launch(cache, (const void*)k_pass<R, LP, MX>, kBlock, lds, &resident);
  if (e != hipSuccess) return e;
  const uint64_t tiles = 1ull << (r.n - r.m);
  const uint64_t blocks = tiles < resident ? tiles : resident;
  hipLaunchKernelGGL((k_pass<R, LP, MX>), dim3((unsigned)blocks), dim3(kBlock), lds, r.s, (E*)r.psi, r.n, r.passes,
                     r.pass, r.stages, r.items, (const cplx<R>*)r.mats, r.frags);
  return hipGetLastError();
}

template <typename R, bool LP, int MX>
hipError_t run_batch(const BatchItemDev* items, int count, uint64_t total_tiles, int max_m, hipStream_t s) {
  typedef typename dev_elem<R>::E E;
  const size_t lds = ((size_t)1 << max_m) * sizeof(E);
  static KernelLaunchCache cache;
  uint64_t resident = 0;
  hipError_t e = prepare_launch(cache, (const void*)k_pass_batch<R, LP, MX>, kBlock, lds, &resident);
  if (e != hipSuccess) return e;
  if (total_tiles == 0) return hipSuccess;
  const uint64_t blocks = total_tiles < resident ? total_tiles : resident;
  hipLaunchKernelGGL((k_pass_batch<R, LP, MX>), dim3((unsigned)blocks), dim3(kBlock), lds, s, items, count, total_tiles);
  return hipGetLastError();
}

// ---------------------------------------------------------------- matrix passes
// A complex128 matrix pass (complex64 ones run as tile passes whose stages
// are matrices) runs dense fused ops (general gate fusion, Sec. II-B) inside
// the tiles of one pass (in-cache operation, Sec. II-B / III-B), on the
// matrix cores.  Stage s views the tile as a 2^K x 2^(m-K) matrix X: rows
// ("members") are the K local bits of the stage (member bit b = local bit
// q[b]), columns the other local bits in the stage's column order (lane
// bits, wave bits, the rest).  It computes Y = U X with three real FP64
// products (Gauss's complex multiplication):
//   P1 = Ur Xr,  P2 = Ui Xi,  P3 = (Ur + Ui)(Xr + Xi),  Yr = P1 - P2,
//   Yi = P3 - P1 - P2.
// Every wave owns whole column blocks (those whose wave bits spell its
// index), so a stage reads and overwrites its columns in place; a barrier
// separates two stages only when their wave bits differ.  A-operand
// fragments and address tables of all stages sit in LDS beside the tile
// (filled once per block).  The next tile's loads go to registers while the
// stages run and are written to LDS once the current tile has been read
// back; a tile's stores go out after the next tile's first stage.  A block
// (eight waves, two per SIMD) is the only one on its CU.
typedef double mx_f64x4 __attribute__((ext_vector_type(4)));

// v_mfma_f64_16x16x4f64: lane l holds A[l % 16][l / 16] and B[l / 16][l % 16];
// accumulator register r of lane l is C[l / 16 + 4 r][l % 16]
struct mx_shape {
  static constexpr int BM = 16, BN = 16, BK = 4, NACC = 4;
  typedef mx_f64x4 acc_t;
  static __device__ __forceinline__ acc_t mma(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};

template <int K>
struct mx_plan {
  static constexpr int D = 1 << K;
  static constexpr int RBK = D / mx_shape::BM;  // row blocks
  static constexpr int KS = D / mx_shape::BK;   // k-steps
  static constexpr int AF = RBK * KS * 64;      // A-fragment entries of one stage
  static_assert(RBK >= 1, "a stage fills at least one row block");
  static_assert(AF == D * D, "one A-fragment entry per matrix entry (matrix_pass_max_stages)");
};

// Swizzled LDS offset of a member: the XOR of the offsets of its set bits
// (swz is linear, and members and columns occupy disjoint local bits).
template <int K>
__device__ __forceinline__ uint32_t mx_member(uint32_t mem, const uint32_t* sm) {
  uint32_t o = 0;
#pragma unroll
  for (int b = 0; b < K; ++b)
    if ((mem >> b) & 1u) o ^= sm[b];
  return o;
}

// Threads of a matrix-pass block: eight waves, two per SIMD, so that one
// wave's LDS and vector work overlaps the other's matrix-core products.
constexpr int kMxThreads = 512;

// Per-stage address table of a matrix pass (uint32 words, byte offsets into
// the tile; every offset is an XOR of swizzled bit offsets, so offsets of
// disjoint bit sets combine by XOR), filled once per block:
//   [kMxBoff + ks]           member BK ks (operand reads, uniform part)
//   [kMxOoff + rb NACC + r]  member BM rb + 4 r (results, uniform part)
//   [kMxCol + cb]            column BN cb
//   [kMxLane + 2 l (+ 1)]    lane l: column l % BN with member l / BN, for
//                            the operands (for the results: the same offset,
//                            read into a register of its own, as one register
//                            for both made every fragment read a wait: three
//                            stages at N = 28 3.38 against 3.32 ms)
constexpr int kMxBoff = 0, kMxOoff = 16, kMxCol = 48, kMxLane = 64, kMxTab = 192;
static_assert(kMxTab * 4 == kMatrixStageTable, "table size shared with the planner");

// Fill the tables of stages 0..ns-1, one entry of one stage per thread and
// step (the stages' reads are in flight together).
template <int K>
__device__ __forceinline__ void mx_tables(const PassStageDev* __restrict__ st, uint32_t ns, uint32_t m, uint32_t* tab) {
  typedef mx_shape MS;
  typedef mx_plan<K> MP;
  constexpr uint32_t EB = sizeof(dbl2);
  constexpr int LBN = 4;     // lane bits of a column block
  constexpr int NC = 12 - K;  // column bits, at most
  const uint32_t nc = m - K;
  const uint32_t cblocks = (1u << nc) / MS::BN;
  for (uint32_t e = threadIdx.x; e < ns * (uint32_t)kMxTab; e += kMxThreads) {
    const PassStageDev* S = st + e / kMxTab;
    const uint32_t t = e % kMxTab;
    uint32_t sm[K], sc[NC];  // swizzled offsets of the member and column bits
#pragma unroll
    for (int b = 0; b < K; ++b) sm[b] = swz<0>(1u << S->q[b]) * EB;
#pragma unroll
    for (int j = 0; j < NC; ++j) sc[j] = (uint32_t)j < nc ? swz<0>(1u << S->colimg[j]) * EB : 0u;
    uint32_t mem = 0, col = 0;
    bool used = true;
    if (t < (uint32_t)kMxOoff) {
      used = t < (uint32_t)MP::KS;
      mem = MS::BK * (t - kMxBoff);
    } else if (t < (uint32_t)kMxCol) {
      const uint32_t i = t - kMxOoff;
      used = i < (uint32_t)(MP::RBK * MS::NACC);
      mem = MS::BM * (i / MS::NACC) + 4 * (i % MS::NACC);
    } else if (t < (uint32_t)kMxLane) {
      used = t - kMxCol < cblocks;
      col = (t - kMxCol) << LBN;
    } else {
      const uint32_t l = (t - kMxLane) / 2;
      col = l % MS::BN;
      mem = (l / MS::BN) % 4u;
    }
    uint32_t v = mx_member<K>(mem, sm);
#pragma unroll
    for (int j = 0; j < NC; ++j) v ^= ((col >> j) & 1u) ? sc[j] : 0u;
    tab[e] = used ? v : 0u;
  }
}

// One stage on the tile in LDS (no barrier inside).  tab: the stage's
// address table; am: its A fragments, entry (rb KS + ks) 64 + l =
// U[BM rb + l % BM][BK ks + l / BM].  Each wave owns whole column blocks.
template <int K>
__device__ __forceinline__ void mx_stage(dbl2* tile, const uint32_t* tab, const cplx<double>* am, uint32_t m) {
  typedef mx_shape MS;
  typedef mx_plan<K> MP;
  unsigned char* tb = reinterpret_cast<unsigned char*>(tile);
  const uint32_t l = threadIdx.x & 63u;
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t cblocks = (1u << (m - K)) / MS::BN;
  const uint32_t lb = tab[kMxLane + 2 * l], lo = tab[kMxLane + 2 * l + 1];
  // the result offsets are read with the operands' and held in registers:
  // read next to their stores, each would cost a wait on the LDS queue
  constexpr int NO = MP::RBK * MS::NACC;
  uint32_t oo[NO];
#pragma unroll
  for (int j = 0; j < NO; ++j) oo[j] = tab[kMxOoff + j];
#pragma unroll
  for (int j = 0; j < NO; ++j) asm volatile("" : "+v"(oo[j]));
  for (uint32_t cb = w; cb < cblocks; cb += kMxThreads / 64) {
    const uint32_t cu = tab[kMxCol + cb];
    const uint32_t bb = lb ^ cu, bo = lo ^ cu;
    MS::acc_t p1[MP::RBK], p2[MP::RBK], p3[MP::RBK];
#pragma unroll
    for (int rb = 0; rb < MP::RBK; ++rb) p1[rb] = p2[rb] = p3[rb] = MS::acc_t{};
#pragma unroll
    for (int ks = 0; ks < MP::KS; ++ks) {
      const dbl2 x = *reinterpret_cast<const dbl2*>(tb + (bb ^ tab[kMxBoff + ks]));
      const double xs = x.x + x.y;
#pragma unroll
      for (int rb = 0; rb < MP::RBK; ++rb) {
        const cplx<double> a = am[(rb * MP::KS + ks) * 64 + l];
        p1[rb] = MS::mma(a.re, x.x, p1[rb]);
        p2[rb] = MS::mma(a.im, x.y, p2[rb]);
        p3[rb] = MS::mma(a.re + a.im, xs, p3[rb]);
      }
    }
    // reads ahead of the products: the first k-steps' operands and fragments,
    // then one read beside every three products (N = 28, K = 5, two and five
    // stages: 2.48 -> 2.41 and 5.09 -> 5.01 ms with the result offsets in
    // registers of their own)
    __builtin_amdgcn_sched_group_barrier(0x100, MP::KS + 6, 0);  // LDS reads
#pragma unroll
    for (int i = 0; i < MP::KS * MP::RBK; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);  // MFMA
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    // this wave has read every member of its columns: overwrite them
#pragma unroll
    for (int rb = 0; rb < MP::RBK; ++rb)
#pragma unroll
      for (int r = 0; r < MS::NACC; ++r) {
        dbl2 y;
        y.x = p1[rb][r] - p2[rb][r];
        y.y = p3[rb][r] - p1[rb][r] - p2[rb][r];
        *reinterpret_cast<dbl2*>(tb + (bo ^ oo[rb * MS::NACC + r])) = y;
      }
  }
}

// Global addresses of a lane's tile elements: register u of lane t is
// element slot e = t + NT u, which holds tile element swz(e) (the layout
// tile_load_lds produces).  The same for every tile of a pass but the base.
template <int NT>
struct MoveGeo {
  uint64_t lane;
  uint64_t hb[TileThreads<NT>::UB];
  LaneGeo lg;
};

template <typename R, int NT>
__device__ __forceinline__ MoveGeo<NT> move_geo(cptr<PassDescDev> P) {
  constexpr int LB = gelem<R>::LB;
  typedef TileThreads<NT> TT;
  MoveGeo<NT> g;
  const uint32_t m = P->m;
  g.lane = lane_slot_bits<LB, NT>(P->lpos, m);
#pragma unroll
  for (int b = 0; b < TT::UB; ++b) g.hb[b] = slot_offset<LB>(P->lpos, m, TT::TB + b);
  g.lg = lane_geo<LB, NT>(m);
  return g;
}

// Move the tile's elements between HBM and registers.  STORE: write them
// back to the addresses they were loaded from (a pass whose write positions
// are its load positions).
template <typename R, int NT, bool STORE>
__device__ __forceinline__ void tile_move(const TileRef<R>& T, const MoveGeo<NT>& mg, typename gelem<R>::G* v) {
  typedef typename gelem<R>::G G;
  typedef TileThreads<NT> TT;
  constexpr int LB = gelem<R>::LB;
  const gptr<G> gpsi = as_global(reinterpret_cast<G*>(T.psi));
  const uint64_t a0 = T.base | mg.lane;
  // Loads are not predicated: a lane without element u reads the tile's
  // first element instead, so that no load result merges with an older value
  // (which would wait for the load right away).
#pragma unroll
  for (int u = 0; u < TT::BATCH; ++u) {
    uint64_t ad = a0;
#pragma unroll
    for (int b = 0; b < TT::UB; ++b)
      if ((u >> b) & 1) ad ^= mg.hb[b];
    const bool ok = (uint32_t)u < mg.lg.per && mg.lg.on;
    if constexpr (STORE) {
      if (ok) stg<G>(gpsi + (ad >> LB), v[u]);
    } else {
      v[u] = ldg<G>((gptr<const G>)(gpsi + ((ok ? ad : T.base) >> LB)));
    }
  }
}

// The tile's element slots to or from registers (register u of lane t = slot t + NT u).
template <typename R, int NT, bool TO_LDS>
__device__ __forceinline__ void tile_slots(typename gelem<R>::G* v, typename dev_elem<R>::E* tile, const LaneGeo& lg) {
  typedef typename gelem<R>::G G;
  G* slots = reinterpret_cast<G*>(tile);
#pragma unroll
  for (int u = 0; u < TileThreads<NT>::BATCH; ++u)
    if ((uint32_t)u < lg.per && lg.on) {
      if constexpr (TO_LDS) slots[threadIdx.x + u * NT] = v[u];
      else v[u] = slots[threadIdx.x + u * NT];
    }
}

template <int K>
__global__ __launch_bounds__(kMxThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_mpass(
    dbl2* __restrict__ psi, int n, const PassDescDev* __restrict__ passes, int pi,
    const PassStageDev* __restrict__ stages, const cplx<double>* __restrict__ mats) {
  typedef double R;
  typedef gelem<R>::G G;
  typedef mx_shape MS;
  typedef mx_plan<K> MP;
  extern __shared__ __align__(16) unsigned char smem[];
  const cptr<PassDescDev> P = as_const(passes + pi);
  const uint32_t m = P->m, ns = P->stage_count;
  dbl2* tile = reinterpret_cast<dbl2*>(smem);
  cplx<R>* am = reinterpret_cast<cplx<R>*>(tile + (1u << m));
  uint32_t* tab = reinterpret_cast<uint32_t*>(am + ns * MP::AF);
  const cptr<PassStageDev> st = as_const(stages) + P->stage_first;
  constexpr int NT = kMxThreads, BATCH = TileThreads<NT>::BATCH;
  for (uint32_t s = 0; s < ns; ++s) {
    const uint32_t at = ((cptr<uint32_t>)(st + s))[offsetof(PassStageDev, u2) / 4];
#pragma unroll
    for (int j = 0; j < (MP::AF + NT - 1) / NT; ++j) {
      const uint32_t f = threadIdx.x + j * NT, l = f % 64, ks = (f / 64) % MP::KS, rb = f / (64 * MP::KS);
      const uint32_t row = MS::BM * rb + l % MS::BM, col = MS::BK * ks + l / MS::BM;
      if (f < (uint32_t)MP::AF) am[s * MP::AF + f] = mats[at + row * MP::D + col];
    }
  }
  mx_tables<K>(stages + P->stage_first, ns, m, tab);
  const SingleSrc<R> src{psi, n, P, as_const(stages), as_const((const PassItemDev*)nullptr), as_const(mats), nullptr};
  const MoveGeo<NT> mg = move_geo<R, NT>(P);
  const uint64_t total = 1ull << (n - m);
  uint64_t g = xcd_block();
  // Per tile: the next tile's loads go out first, the previous tile's
  // stores after the first stage, so neither burst waits behind the other in
  // the memory queue while the stages could run.
  G nx[BATCH], out[BATCH];
  if (g < total) tile_move<R, NT, false>(src(g), mg, nx);
  __syncthreads();  // the A fragments and tables are in LDS
  if (g >= total) return;
  tile_slots<R, NT, true>(nx, tile, mg.lg);
  uint64_t prev = total;  // tile whose results wait in `out` (none yet)
  while (true) {
    const uint64_t ng = g + gridDim.x;
    lds_sync();  // the tile is in LDS
    if (ng < total) tile_move<R, NT, false>(src(ng), mg, nx);
    for (uint32_t s = 0; s < ns; ++s) {
      if (s > 0) {
        const uint32_t fl = ((cptr<uint32_t>)(st + s))[offsetof(PassStageDev, flags) / 4];
        if (fl & kMatrixStageSync) {
          lds_sync();
        } else {
          // the stage reads only what this wave wrote: its own LDS writes
          // are done, no other wave is waited for
          wait_lgkm0();
          asm volatile("" ::: "memory");
        }
      }
      mx_stage<K>(tile, tab + s * kMxTab, am + s * MP::AF, m);
      if (s == 0 && prev < total) tile_move<R, NT, true>(src(prev), mg, out);
    }
    lds_sync();  // every wave's results are in LDS
    if (ns == 0 && prev < total) tile_move<R, NT, true>(src(prev), mg, out);  // (a pass has stages)
    tile_slots<R, NT, false>(out, tile, mg.lg);
    lds_sync();  // every lane has read the tile
    prev = g;
    if (ng >= total) break;
    tile_slots<R, NT, true>(nx, tile, mg.lg);
    g = ng;
  }
  tile_move<R, NT, true>(src(prev), mg, out);
}

template <int K>
hipError_t run_mpass(void* psi, int n, int m, const PassDescDev* passes, int pass, int n_stages,
                     const PassStageDev* stages, const void* mats, hipStream_t s) {
  const size_t lds = ((size_t)1 << m) * sizeof(dbl2) +
                     (size_t)n_stages * (mx_plan<K>::AF * sizeof(cplx<double>) + kMxTab * sizeof(uint32_t));
  if (lds > (size_t)kMatrixPassLds) return hipErrorInvalidValue;
  static KernelLaunchCache cache;
  uint64_t resident = 0;
  hipError_t e = prepare_launch(cache, (const void*)k_mpass<K>, kMxThreads, lds, &resident);
  if (e != hipSuccess) return e;
  const uint64_t tiles = 1ull << (n - m);
  const uint64_t blocks = tiles < resident ? tiles : resident;
  hipLaunchKernelGGL((k_mpass<K>), dim3((unsigned)blocks), dim3(kMxThreads), lds, s, (dbl2*)psi, n, passes, pass,
                     stages, (const cplx<double>*)mats);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_matrix_pass(int k, void* psi, int n, int m, const PassDescDev* passes, int pass, int n_stages,
                              const PassStageDev* stages, const void* mats, hipStream_t s) {
  if (k == 4) return run_mpass<4>(psi, n, m, passes, pass, n_stages, stages, mats, s);
  if (k == 5) return run_mpass<5>(psi, n, m, passes, pass, n_stages, stages, mats, s);
  return hipErrorInvalidValue;
}

hipError_t launch_stage_frags(PassStageDev* stages, const uint32_t* list, int count, const void* pool,
                              void* frags, hipStream_t s) {
  hipLaunchKernelGGL(k_stage_frags, dim3((unsigned)count), dim3(kBlock), 0, s, stages, list, (const cplx<float>*)pool,
                     (uint32_t*)frags);
  return hipGetLastError();
}

hipError_t launch_pass(sv_dtype dt, void* psi, int n, int m, const PassDescDev* passes, int pass,
                       const PassStageDev* stages, const PassItemDev* items, const void* mats, const void* frags,
                       bool ladders, PassMatrix mx, hipStream_t s) {
  const PassRun r{psi, n, m, passes, pass, stages, items, mats, frags, s};
  if (dt == SV_C128) return ladders ? run<double, true, MX_NONE>(r) : run<double, false, MX_NONE>(r);
  if (mx == kPassMatrixOnly) return run<float, false, MX_ONLY>(r);
  if (mx == kPassMatrixTile) return ladders ? run<float, true, MX_TILE>(r) : run<float, false, MX_TILE>(r);
  return ladders ? run<float, true, MX_NONE>(r) : run<float, false, MX_NONE>(r);
}

hipError_t launch_pass_batch(sv_dtype dt, const BatchItemDev* items, int count, uint64_t total_tiles, int max_m,
                             bool ladders, PassMatrix mx, hipStream_t s) {
  if (dt == SV_C128)
    return ladders ? run_batch<double, true, MX_NONE>(items, count, total_tiles, max_m, s)
                   : run_batch<double, false, MX_NONE>(items, count, total_tiles, max_m, s);
  if (mx == kPassMatrixOnly) return run_batch<float, false, MX_ONLY>(items, count, total_tiles, max_m, s);
  if (mx == kPassMatrixTile)
    return ladders ? run_batch<float, true, MX_TILE>(items, count, total_tiles, max_m, s)
                   : run_batch<float, false, MX_TILE>(items, count, total_tiles, max_m, s);
  if (mx == kPassMatrixMixed)
    return ladders ? run_batch<float, true, MX_MIXED>(items, count, total_tiles, max_m, s)
                   : run_batch<float, false, MX_MIXED>(items, count, total_tiles, max_m, s);
  return ladders ? run_batch<float, true, MX_NONE>(items, count, total_tiles, max_m, s)
                 : run_batch<float, false, MX_NONE>(items, count, total_tiles, max_m, s);
}

}  // namespace sv
