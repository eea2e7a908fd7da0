// fp32 products on the bf16 matrix cores: the operands in three bf16 parts.
//
// An fp32 value is the sum of three bf16 values, x = h + m + l (h = x rounded to
// bf16, m = x - h rounded, l the rest: 8 + 8 + 8 significant bits).  It is exact from
// 2^-110 up; below, l runs out of bf16's subnormals (which the matrix cores
// honour) and x is off by up to 2^-134: 2^-24 of it at 2^-110, 2^-14 at 2^-120.  A product
// is formed from the six partial products h h', h m', m h', h l', m m', l h', each
// exact in the fp32 accumulator's input; the dropped ones (m l', l m', l l')
// are below 2^-26 of it, less than the rounding of one fp32 addition.  The
// fp32 instruction v_mfma_f32_16x16x4 does 32 multiply-adds a cycle, the bf16
// one (16x16x32) 512 by six products = 85, at a quarter fewer roundings of the
// accumulator; on this part the fp32 instruction also excludes vector work,
// the bf16 one does not.
//
// Operand A (rows of X, fp32 in memory) is loaded straight into the lanes
// that multiply it and split there: no LDS for X.  Operand B (W, or the
// residuals) is split once into fragments in lane order (sg_frag), which a
// block copies to LDS a slice of 32 K at a time; its NW waves, stacked along
// M, share them.  Lane l = 16 g + c of v_mfma_f32_16x16x32_bf16 holds A row
// c, K 8 g .. 8 g + 7; B column c, the same K; accumulator element r is row
// 4 g + r, column c (the fp32 instruction's too).
//
// Infinities and values that round to infinity in bf16 have no such parts
// (inf - inf), and sums of very small products may be made of operands below
// 2^-110.  An accumulator that is not finite, or below 2^-90, is formed again with
// the fp32 instruction (sg_redo), so those inputs give what fp32 arithmetic
// gives.  A larger sum is off by at most K 2^-134 times the other operand's
// largest value for such operands: less than fp32's own rounding while that
// product is below 2^20.  (The packed operand of a sum formed again is its
// parts': the softmax's residuals are scaled so that these are exact; dA of the
// MLP is held to 2^-134.)
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "dbw_buffer.h"

namespace dbw {

// (native vectors: arrays of HIP's uint4 do not stay in registers)
typedef uint32_t sg_u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t sg_u32x2 __attribute__((ext_vector_type(2)));
typedef float sg_f32x4 __attribute__((ext_vector_type(4)));
typedef float sg_f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 sg_bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 sg_bf16x8 __attribute__((ext_vector_type(8)));

constexpr int SG_K = 32;   // K of one slice

// Fragments (1 KiB: 64 lanes x 8 bf16) of a K x N operand: three parts (h, m,
// l) for each slice of 32 K and tile of 16 columns.
__host__ __device__ inline int64_t sg_frag(int64_t kb, int64_t tiles, int64_t nt, int part) {
  return (kb * tiles + nt) * 3 + part;
}
inline int64_t sg_frag_bytes(int64_t kblocks, int64_t tiles) { return kblocks * tiles * 3 * 1024; }

__device__ __forceinline__ uint32_t sg_pk(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(sg_f32x2{a, b}, sg_bf16x2));
}
__device__ __forceinline__ float sg_lo(uint32_t v) { return __builtin_bit_cast(float, v << 16); }
__device__ __forceinline__ float sg_hi(uint32_t v) { return __builtin_bit_cast(float, v & 0xffff0000u); }

// The parts of two values, packed.
struct SgPair {
  uint32_t h, m, l;
};
__device__ __forceinline__ SgPair sg_split2(float a, float b) {
  SgPair p;
  p.h = sg_pk(a, b);
  const float ra = a - sg_lo(p.h), rb = b - sg_hi(p.h);
  p.m = sg_pk(ra, rb);
  p.l = sg_pk(ra - sg_lo(p.m), rb - sg_hi(p.m));
  return p;
}
// The same where a part of an infinity or a NaN must not be a NaN of its own:
// the sum of the stored parts is the value in every case.
__device__ __forceinline__ SgPair sg_split2_any(float a, float b) {
  SgPair p;
  uint32_t h = sg_pk(a, b);
  // a finite value that rounds to infinity keeps its truncation instead
  if (!(fabsf(sg_lo(h)) <= 3.4e38f) && a == a) h = (h & 0xffff0000u) | (__builtin_bit_cast(uint32_t, a) >> 16);
  if (!(fabsf(sg_hi(h)) <= 3.4e38f) && b == b) h = (h & 0xffffu) | (__builtin_bit_cast(uint32_t, b) & 0xffff0000u);
  float ra = a - sg_lo(h), rb = b - sg_hi(h);
  ra = ra == ra ? ra : 0.f;
  rb = rb == rb ? rb : 0.f;
  p.h = h;
  p.m = sg_pk(ra, rb);
  p.l = sg_pk(ra - sg_lo(p.m), rb - sg_hi(p.m));
  return p;
}

__device__ __forceinline__ sg_bf16x8 sg_op(const sg_u32x4& v) { return __builtin_bit_cast(sg_bf16x8, v); }

// One operand fragment of a lane: eight K of one row (or column).
struct SgParts {
  sg_u32x4 h, m, l;
};
__device__ __forceinline__ SgParts sg_split8(const float (&x)[8]) {
  SgParts p;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const SgPair v = sg_split2(x[2 * q], x[2 * q + 1]);
    p.h[q] = v.h;
    p.m[q] = v.m;
    p.l[q] = v.l;
  }
  return p;
}

__device__ __forceinline__ sg_f32x4 sg_mfma(const sg_u32x4& a, const sg_u32x4& b, sg_f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(sg_op(a), sg_op(b), c, 0, 0, 0);
}

// acc[mt] += A[mt] B for one column tile.  APART: the five small products are
// summed by themselves (their roundings are some 2^-8 of the accumulator's) and
// added with the large one, so an accumulator is rounded twice a slice of 32 K
// instead of six times.  Gradient error against 64 bits, together / apart / fp32
// instruction: MLP 32 x 64 x 784-512-10 1.7e-7 / 0.8e-7 / 1.4e-7, MLP 16 x 256 x
// 3072-1024-10 5.7e-7 / 2.9e-7 / 6.1e-7, softmax 20 x 300 x 1200 x 60 2.5e-7 /
// 1.3e-7 / 3.1e-7, 256 x 512 x 3072 x 100 3.2e-7 / 1.7e-7 / 4.1e-7.  It takes
// registers and 6 - 10% of the time of a kernel that is bound by its products,
// so the wide tiles of the softmax keep one sum.
template <bool APART, int MT>
__device__ __forceinline__ void sg_products(const SgParts (&a)[MT], const sg_u32x4& bh, const sg_u32x4& bm,
                                            const sg_u32x4& bl, sg_f32x4 (&acc)[MT]) {
  sg_f32x4 small[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) small[t] = APART ? sg_f32x4{0.f, 0.f, 0.f, 0.f} : acc[t];
#pragma unroll
  for (int p = 0; p < 5; ++p)
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const sg_u32x4& x = p == 0 ? a[t].l : p == 2 || p == 3 ? a[t].m : a[t].h;
      const sg_u32x4& y = p == 1 ? bl : p == 2 || p == 4 ? bm : bh;
      small[t] = sg_mfma(x, y, small[t]);
    }
#pragma unroll
  for (int t = 0; t < MT; ++t) acc[t] = sg_mfma(a[t].h, bh, APART ? acc[t] : small[t]);
  if constexpr (APART) {
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[t] += small[t];
  }
}

// Two slices' B fragments; padded to whole rounds of the block's NW waves.
template <int NT, int NW>
struct SgLds {
  static constexpr int NB = (NT * 3 + NW - 1) / NW;   // fragments a wave copies
  sg_u32x4 B[2][NB * NW][64];
};

template <int MT, int NT>
__device__ __forceinline__ void sg_zero(sg_f32x4 (&acc)[NT][MT]) {
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = sg_f32x4{0.f, 0.f, 0.f, 0.f};
}

// Block barrier after this wave's LDS work; global loads stay in flight.
__device__ __forceinline__ void sg_barrier() {
  __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
  asm volatile("s_barrier" ::: "memory");
}

// The slice loop over K slices kb0 .. kb1 - 1.  load(kb, x, dead) fetches this
// wave's A values of a slice (MT tiles x 8), frag(kb) is the address of the
// slice's first B fragment (NT * 3 of them, consecutive), prep(kb, x) runs just
// before a slice's values are split.  PD slices are on their way in registers
// (PD = 2 where a block's matrix work per slice is shorter than a memory
// latency; 4 gained nothing more, nor did two teams of waves that split K); a
// slice's B fragments are loaded before its A values, so that storing them to
// LDS does not wait for the A values.  Loads past the last slice are out of
// range (dead), so that the number in flight is the same at every step and they
// cost no memory access, and the last slice neither stages nor waits (fetching
// it again, as before: step of 4 x 32 x 784 x 10 23.7 -> 20.6 us, MLP 32 x 64 x 784-512-10
// 53.4 -> 51.8, softmax 64 x 38 x 164 x 580 45.5 -> 42.7).  Bodies of their own for
// the last slices take up to 60 registers more, for the accumulators' ways
// through them: 71 x 155 x 760 x 380 109 -> 117 us.
template <bool APART, int MT, int NT, int NW, int PD, class Load, class Prep, class Frag>
__device__ __forceinline__ void sg_loop(SgLds<NT, NW>& L, int kb0, int kb1, Load&& load, Prep&& prep, Frag&& frag,
                                        sg_f32x4 (&acc)[NT][MT]) {
  static_assert(PD == 1 || PD == 2, "register slots");
  constexpr int NB = SgLds<NT, NW>::NB;
  // the largest logits blocks (16 row tiles) have many slices: there the last
  // one's extra cost is nothing, and the steps towards saving it 5% (256 x 512 x
  // 3072 x 100: 214 / 224 us)
  constexpr bool LONG = MT == 2 && NW == 8;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  sg_u32x4 rb[PD][NB];
  float x[PD][MT][8];
  auto fetch = [&](int kb, sg_u32x4 (&r)[NB], float (&v)[MT][8]) {
    const bool live = kb < kb1;
    kb = min(kb, kb1 - 1);
    if constexpr (LONG) {
      const sg_u32x4* src = frag(kb);
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        const int f = wv + NW * q;
        r[q] = src[(NT * 3 % NW == 0 ? f : min(f, NT * 3 - 1)) * 64 + lane];
      }
      load(kb, v, 0u);
      return;
    }
    // (dead slices by the vector offset: the resource's size, from which the
    // bounds check takes the scalar offset, stays larger than that)
    const uint32_t dead = live ? 0u : kOutOfRange;
    const __amdgpu_buffer_rsrc_t src = make_rsrc(frag(kb), NT * 3 * 1024u);
    const uint32_t off = static_cast<uint32_t>((wv * 64 + lane) * 16) | dead;
#pragma unroll
    for (int q = 0; q < NB; ++q)   // (fragments past the slice's NT * 3 read as 0)
      r[q] = __builtin_bit_cast(sg_u32x4, __builtin_amdgcn_raw_buffer_load_b128(src, off, q * NW * 1024, 0));
    load(kb, v, dead);
  };
  auto stage = [&](int buf, const sg_u32x4 (&r)[NB]) {
#pragma unroll
    for (int q = 0; q < NB; ++q) L.B[buf][wv + NW * q][lane] = r[q];
  };
  if (kb0 >= kb1) return;
#pragma unroll
  for (int p = 0; p < PD; ++p) fetch(kb0 + p, rb[p], x[p]);
  stage(0, rb[0]);
  sg_barrier();
  // slice kb: LDS buffer u (its B), register slot u % PD (its A); the slot is
  // refilled with slice kb + PD once its A values are split (its B fragments
  // were staged a slice ago).  more: another slice follows (at the end of an
  // odd count known beforehand: LAST)
  auto slice = [&](int kb, auto uc, auto last, bool more) {
    constexpr int u = decltype(uc)::value, slot = u % PD, next = (u + 1) % PD;
    constexpr bool LAST = decltype(last)::value;
    SgParts a[MT];
    prep(kb, x[slot]);
#pragma unroll
    for (int t = 0; t < MT; ++t) a[t] = sg_split8(x[slot][t]);
    if constexpr (LONG || !LAST) fetch(kb + PD, rb[slot], x[slot]);
    __builtin_amdgcn_sched_barrier(0);   // the loads go out before the products
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
      sg_products<APART, MT>(a, L.B[u][3 * nt][lane], L.B[u][3 * nt + 1][lane], L.B[u][3 * nt + 2][lane], acc[nt]);
    // a column tile's fragments are read while the previous tile's products run
    __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      if (nt + 1 < NT) __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 6 * MT, 0);
    }
    __builtin_amdgcn_sched_barrier(0);   // and are waited for after them
    if (LONG || (!LAST && more)) {
      stage(u ^ 1, rb[next]);
      sg_barrier();
    }
  };
  // (whole pairs in the loop: a way round the second slice would make the
  // compiler wait for every load at the loop's head)
  int kb = kb0;
  for (; kb + 1 < kb1; kb += 2) {
    slice(kb, std::integral_constant<int, 0>{}, std::false_type{}, true);
    slice(kb + 1, std::integral_constant<int, 1>{}, std::false_type{}, kb + 2 < kb1);
  }
  if (kb < kb1) slice(kb, std::integral_constant<int, 0>{}, std::true_type{}, false);
}

// The loop for products with few tiles: the block's NW waves work on the same
// MT x NT tiles and share the K slices (wave w takes kb0 + w, kb0 + w + NW, ..),
// each reading its B fragments from the L2 itself, with no barrier; the waves'
// sums meet in LDS and wave 0 adds them in wave order (it alone goes on with
// the result).  A slice costs a memory latency either way; here a wave waits
// for one in NW of them.
// B comes as fragments (SgFrags) or straight from a row-major K x N matrix
// (SgMatrix: each lane loads and splits its own eight values; no packing
// launch before, worth it while a block has few column tiles).
template <int NT>
struct SgFrags {
  const sg_u32x4* first;   // slice 0
  int64_t stride;          // pieces per slice
  using Raw = sg_u32x4[NT * 3];
  __device__ __forceinline__ void load(int kb, Raw& b) const {
    const sg_u32x4* src = first + kb * stride;
#pragma unroll
    for (int f = 0; f < NT * 3; ++f) b[f] = src[f * 64 + (threadIdx.x & 63)];
  }
  __device__ __forceinline__ void parts(const Raw& b, int nt, sg_u32x4 (&p)[3]) const {
#pragma unroll
    for (int q = 0; q < 3; ++q) p[q] = b[3 * nt + q];
  }
};
template <int NT>
struct SgMatrix {
  __amdgpu_buffer_rsrc_t rs;   // exactly the K x N floats: rows past K read as 0
  int N;
  uint32_t off[NT];            // the lane's column, K 8 g (kOutOfRange past N)
  using Raw = float[NT][8];
  __device__ __forceinline__ SgMatrix(__amdgpu_buffer_rsrc_t r, int n, int n0) : rs(r), N(n) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int c = n0 + 16 * nt + (lane & 15);
      off[nt] = c < n ? static_cast<uint32_t>((8 * (lane >> 4) * n + c) * 4) : kOutOfRange;
    }
  }
  __device__ __forceinline__ void load(int kb, Raw& b) const {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int e = 0; e < 8; ++e) b[nt][e] = buf_f32(rs, off[nt] + static_cast<uint32_t>((kb * SG_K + e) * N * 4));
  }
  __device__ __forceinline__ void parts(const Raw& b, int nt, sg_u32x4 (&p)[3]) const {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const SgPair v = sg_split2(b[nt][2 * q], b[nt][2 * q + 1]);
      p[0][q] = v.h;
      p[1][q] = v.m;
      p[2][q] = v.l;
    }
  }
};
template <int MT, int NT, int NW>
struct SgRed {
  sg_f32x4 v[NW - 1][NT * MT][64];
};
template <bool APART, int MT, int NT, int NW, class Load, class Prep, class Bsrc>
__device__ __forceinline__ void sg_loop_k(SgRed<MT, NT, NW>& R, int kb0, int kb1, Load&& load, Prep&& prep,
                                          const Bsrc& bsrc, sg_f32x4 (&acc)[NT][MT]) {
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float x[MT][8];
  typename Bsrc::Raw b;
  int kb = kb0 + wv;
  if (kb < kb1) {
    bsrc.load(kb, b);
    load(kb, x);
  }
  for (; kb < kb1; kb += NW) {
    SgParts a[MT];
    sg_u32x4 bp[NT][3];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) bsrc.parts(b, nt, bp[nt]);
    prep(kb, x);
#pragma unroll
    for (int t = 0; t < MT; ++t) a[t] = sg_split8(x[t]);
    if (kb + NW < kb1) {
      bsrc.load(kb + NW, b);
      load(kb + NW, x);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) sg_products<APART, MT>(a, bp[nt][0], bp[nt][1], bp[nt][2], acc[nt]);
  }
  if (wv > 0) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        R.v[wv - 1][nt * MT + mt][lane] = acc[nt][mt];
        acc[nt][mt] = sg_f32x4{0.f, 0.f, 0.f, 0.f};
      }
  }
  __syncthreads();
  if (wv == 0) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int w = 0; w < NW - 1; ++w) acc[nt][mt] += R.v[w][nt * MT + mt][lane];
  }
}

// A values of rows of X: lane (g, c) takes K 32 kb + 8 g .. + 7 of the row at
// byte offset roff[t] + 32 g (kOutOfRange: no row, zeros), in two 16-byte loads
// that need 4-byte alignment only.  In the last, partial slice a lane whose
// eight values would pass the row's end loads the row's last eight and
// shifts them down, zeros behind (no branch around the loads: the waits for
// them stay partial).  K < 8 (TINY): value by value.
template <int MT, bool TINY>
struct SgRows {
  __amdgpu_buffer_rsrc_t xs;
  int K, tail;            // tail: the partial slice (or none: the slice count)
  uint32_t roff[MT];
  int shift;
  __device__ __forceinline__ SgRows(__amdgpu_buffer_rsrc_t r, int k) : xs(r), K(k), tail(k / SG_K) {
    const int k0 = tail * SG_K + 8 * ((threadIdx.x & 63) >> 4);
    shift = TINY ? 0 : max(0, k0 - (K - 8));
  }
  __device__ __forceinline__ int slices() const { return (K + SG_K - 1) / SG_K; }
  __device__ __forceinline__ void operator()(int kb, float (&x)[MT][8], uint32_t dead = 0) const {
    if constexpr (TINY) {
      const int kg = 8 * ((threadIdx.x & 63) >> 4);
#pragma unroll
      for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int e = 0; e < 8; ++e) x[t][e] = buf_f32(xs, (kg + e < K ? roff[t] + 4 * e : kOutOfRange) | dead);
    } else {
      // (the tail's offset goes to the vector operand, which alone must not be
      // negative for the bounds check: the first row's would be)
      const uint32_t at = kb == tail ? static_cast<uint32_t>(kb * SG_K - shift) * 4 : 0u;
      const uint32_t so = kb == tail ? 0u : static_cast<uint32_t>(kb * SG_K * 4);
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        const uint32_t off = (roff[t] + at) | dead;
        const float4 u = buf_f32x4_s(xs, off, so);
        const float4 v = buf_f32x4_s(xs, off + 16, so);
        x[t][0] = u.x; x[t][1] = u.y; x[t][2] = u.z; x[t][3] = u.w;
        x[t][4] = v.x; x[t][5] = v.y; x[t][6] = v.z; x[t][7] = v.w;
      }
    }
  }
  __device__ __forceinline__ void prep(int kb, float (&x)[MT][8]) const {
    if (TINY || kb != tail) return;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
#pragma unroll
      for (int q = 4; q >= 1; q >>= 1)
#pragma unroll
        for (int e = 0; e < 8; ++e) x[t][e] = shift & q ? (e + q < 8 ? x[t][e + q] : 0.f) : x[t][e];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[t][e] = shift >= 8 ? 0.f : x[t][e];
    }
  }
};

// A values of X^T: lane (g, c) takes MT features from f (one per tile) of rows
// 32 kb + 8 g .. + 7, whose byte offsets stand in LDS (kOutOfRange: no row).
// Every lane loads MT features inside the row, from byte offset foff: near the
// row's end from `shift` features before f (sg_feature); `edge` is
// wave-uniform and says whether any lane of the wave has a shift.
template <int MT>
__device__ __forceinline__ void sg_feature(int f, int d, uint32_t& foff, int& shift) {
  const int at = f < d ? min(f, d - MT) : 0;   // past d: any feature, its results are not stored
  shift = f < d ? f - at : 0;
  foff = static_cast<uint32_t>(at * 4);
}
template <int MT>
__device__ __forceinline__ void sg_load_cols(__amdgpu_buffer_rsrc_t xs, const uint32_t* srow, uint32_t foff, float (&x)[MT][8],
                                             uint32_t dead = 0) {
  static_assert(MT == 1 || MT == 2 || MT == 4, "features per lane");
  const sg_u32x4 o[2] = {*reinterpret_cast<const sg_u32x4*>(srow), *reinterpret_cast<const sg_u32x4*>(srow + 4)};
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const uint32_t off = (o[e >> 2][e & 3] + foff) | dead;
    if constexpr (MT == 1) {
      x[0][e] = buf_f32(xs, off);
    } else if constexpr (MT == 2) {
      const float2 v = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(xs, off, 0, 0));
      x[0][e] = v.x;
      x[1][e] = v.y;
    } else {
      const float4 v = buf_f32x4(xs, off);
      x[0][e] = v.x;
      x[1][e] = v.y;
      x[2][e] = v.z;
      x[3][e] = v.w;
    }
  }
}
// The loaded values at their places, just before they are used.
template <int MT>
__device__ __forceinline__ void sg_shift(int shift, bool edge, float (&x)[MT][8]) {
  if (MT > 1 && edge) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int q = 1; t + q < MT; ++q) x[t][e] = shift == q ? x[t + q][e] : x[t][e];
  }
}

// A sum that its parts may not hold: not finite, or not zero and below 2^-90.
__device__ __forceinline__ bool sg_doubtful(float v) {
  const uint32_t u = __builtin_bit_cast(uint32_t, v) & 0x7fffffffu;   // [2^-90, infinity) is [0x12800000, 0x7f800000)
  return u - 0x12800000u >= 0x7f800000u - 0x12800000u && u != 0;
}

// Doubtful accumulators are formed again with the fp32 matrix instruction, a
// tile at a time: ea(mt, k) is A of the lane's row c of tile mt at K index k, eb(nt, k)
// B of the lane's column c of column tile nt (k < K; 0 where there is no row or
// column).  2.5 instructions per accumulator when none is doubtful.  (A
// scalar dot product in each lane took 30 - 170 times the whole launch where a NaN
// has reached the parameters: 32 x 128 x 2048 x 1000 41 ms, now 3.3 (0.39 on fp32
// products throughout); 24 x 200 x 1000 x 37 1.9, now 0.16 (0.13).)
template <int MT, int NT, class Ea, class Eb>
__device__ __forceinline__ void sg_redo(sg_f32x4 (&acc)[NT][MT], int K, Ea&& ea, Eb&& eb) {
  float s = 0.f;             // NaN if one is not finite
  uint32_t least = ~0u;      // the least 2 |bits| - 1 (zeros: the largest value)
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s = fmaf(acc[nt][mt][r], 0.f, s);
        least = min(least, (__builtin_bit_cast(uint32_t, acc[nt][mt][r]) << 1) - 1u);
      }
  if (__builtin_amdgcn_ballot_w64(s != s || least < 2u * 0x12800000u - 1u) == 0) return;
  const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      bool bad = false;
#pragma unroll
      for (int r = 0; r < 4; ++r) bad |= sg_doubtful(acc[nt][mt][r]);
      if (__builtin_amdgcn_ballot_w64(bad) == 0) continue;
      sg_f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
      for (int k0 = 0; k0 < K; k0 += 16) {
        float x[4], y[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          // (loads of the last k past K, whose values are dropped: no branches)
          const int k = k0 + 4 * q + g, kc = min(k, K - 1);
          x[q] = ea(mt, kc);
          y[q] = eb(nt, kc);
          x[q] = k < K ? x[q] : 0.f;
          y[q] = k < K ? y[q] : 0.f;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) z = __builtin_amdgcn_mfma_f32_16x16x4f32(x[q], y[q], z, 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[nt][mt][r] = sg_doubtful(acc[nt][mt][r]) ? z[r] : acc[nt][mt][r];
    }
}

// Element (k, n) of a packed operand, put together again.
__device__ __forceinline__ float sg_unpack(const sg_u32x4* frags, int64_t tiles, int k, int n) {
  const uint16_t* p = reinterpret_cast<const uint16_t*>(frags);
  const int lane = 16 * ((k & 31) >> 3) + (n & 15), e = k & 7;
  float s = 0.f;
#pragma unroll
  for (int part = 2; part >= 0; --part)
    s += sg_lo(p[(sg_frag(k >> 5, tiles, n >> 4, part) * 64 + lane) * 8 + e]);
  return s;
}

// Four consecutive K of one column (k0 % 4 == 0) into the fragments: half of a
// lane's 16 bytes in each part.
__device__ __forceinline__ void sg_store4(sg_u32x4* frags, int64_t tiles, int k0, int n, const float (&v)[4]) {
  const SgPair u = sg_split2_any(v[0], v[1]), w = sg_split2_any(v[2], v[3]);
  sg_u32x2* p = reinterpret_cast<sg_u32x2*>(frags) + sg_frag(k0 >> 5, tiles, n >> 4, 0) * 128 +
             (16 * ((k0 & 31) >> 3) + (n & 15)) * 2 + ((k0 >> 2) & 1);
  p[0] = sg_u32x2{u.h, w.h};
  p[128] = sg_u32x2{u.m, w.m};
  p[256] = sg_u32x2{u.l, w.l};
}

// Eight consecutive K of one column (k0 % 8 == 0).
__device__ __forceinline__ void sg_store8(sg_u32x4* frags, int64_t tiles, int k0, int n, const float (&v)[8]) {
  sg_u32x4 h, m, l;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const SgPair u = sg_split2_any(v[2 * q], v[2 * q + 1]);
    h[q] = u.h;
    m[q] = u.m;
    l[q] = u.l;
  }
  sg_u32x4* p = frags + sg_frag(k0 >> 5, tiles, n >> 4, 0) * 64 + 16 * ((k0 & 31) >> 3) + (n & 15);
  p[0] = h;
  p[64] = m;
  p[128] = l;
}

// A K x N matrix (element (k, n) at k ldk + n ldn) into fragments, zeros past K
// and N; one wave per slice and column tile, `tiles` column tiles.
__global__ __launch_bounds__(256) inline void k_sg_pack(const float* src, int64_t ldk, int64_t ldn, int K, int N,
                                                        int tiles, sg_u32x4* frags) {
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int64_t kblocks = (K + SG_K - 1) / SG_K;
  if (t >= kblocks * tiles) return;
  const int kb = static_cast<int>(t / tiles), nt = static_cast<int>(t % tiles);
  const int k0 = kb * SG_K + 8 * (lane >> 4), n = 16 * nt + (lane & 15);
  float v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = k0 + e < K && n < N ? src[(k0 + e) * ldk + n * ldn] : 0.f;
  sg_store8(frags, tiles, k0, n, v);
}

}  // namespace dbw
