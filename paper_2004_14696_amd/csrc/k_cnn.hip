// Worker minibatch gradients of the MNIST-shaped CNN (Sect. 4: two 5x5
// convolutions and two fully connected layers; Sect. 2, Eq. gradient), gfx950.
//
// Per image (28 x 28, one channel): conv 1 -> 20 channels (24 x 24), 2 x 2 max
// pooling and ReLU (20 x 12 x 12 = H1), conv 20 -> 50 (8 x 8), pooling and ReLU
// (50 x 4 x 4 = the 800 features F), then the fully connected part, which is
// the MLP 800-H-C (k_mlp.hip).  A pooling window passes its first largest
// value in row-major order; only that entry receives the gradient, and none
// when the pooled value is not positive (ReLU).  The window code 0..3 names
// the passing entry; code 4 marks a window whose ReLU is off, so unpooling
// by code applies the ReLU mask as well.
//
//  k_cnn_conv1_pool   one thread per pooled position of an image: the four
//                     conv outputs of its window for all 20 filters (vector
//                     ALU, filters in LDS), the pooled value, its ReLU and the
//                     window code; also gathers the image's label.
//  k_cnn_conv2_pool   the conv as a 64 x 64 x 500 GEMM per image (positions x
//                     filters x patches) on the split products of
//                     split_gemm.h, one image a wave, W2's fragments shared
//                     through LDS; pooling and ReLU in the epilogue.
//  k_cnn_conv2_close  the pooling and ReLU decisions of conv2 that lie within
//                     rounding, taken again on fp32 matrix-core sums.
//  k_cnn_dfeat        dF = dA Wf1^T on the matrix cores (the ReLU mask of F is
//                     in the window codes).
//  k_cnn_conv2_dgrad  gradient at H1: per image and input channel the GEMM
//                     dcols = dZ2 W2 (positions x taps, K = filters) on the
//                     matrix cores, with the filters' fragments held in
//                     registers by a persistent grid; the fold of dcols back
//                     onto the 12 x 12 map reads zero-framed tap maps in LDS at
//                     fixed offsets.
//  k_cnn_conv2_wgrad  dW2 and db2 partials over chunks of a worker's images:
//                     dW2 += dZ2^T im2col(H1) per image (filters x taps, K =
//                     positions) on the matrix cores, accumulators kept over the
//                     chunk, the next image staged in LDS meanwhile.
//  k_cnn_conv1_wgrad  dW1 and db1 partials: dW1 += dZ1 im2col(X) per image
//                     (filters x taps, K = the 576 conv1 positions) on the
//                     matrix cores, dZ1 formed from the pooled gradient and
//                     window codes as the operand is read.
//  k_cnn_wreduce      sums the chunk partials in chunk order into G.
//
// Everything runs in a fixed order: results are bitwise reproducible.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "dbw_buffer.h"
#include "dbw_internal.h"
#include "split_gemm.h"

namespace dbw {
namespace {

typedef float mfma_f32x4 __attribute__((ext_vector_type(4)));

constexpr int IMG = CNN_IMG, KS = 5, NC1 = CNN_C1, NC2 = CNN_C2;
constexpr int Q1 = 12, NPOS1 = Q1 * Q1, H1LEN = NC1 * NPOS1;   // 2880 per image
constexpr int O2 = 8, NPOS2 = O2 * O2;                          // conv2 output positions
constexpr int Q2 = 4, NQ2 = Q2 * Q2, FEAT = CNN_FEAT;           // 800
constexpr int K2 = NC1 * KS * KS;                               // 500: conv2 patch length
constexpr int W1LEN = NC1 * KS * KS;                            // 500 conv1 weights

__device__ __forceinline__ int64_t cnn_row(const CnnArgs& a, int64_t m, bool report) {
  if (!a.rows) return m;
  const int64_t r = a.rows[m];
  if (r < 0 || r >= a.S) {
    if (report) atomicOr(a.err, ERR_ROW_RANGE);
    return -1;
  }
  return r;
}

// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_cnn_conv1_pool(CnnArgs a) {
  __shared__ float sw[W1LEN + NC1];
  const int tid = threadIdx.x;
  for (int i = tid; i < W1LEN + NC1; i += 256) sw[i] = a.w[a.off_c1 + i];   // W1 then b1
  __syncthreads();
  const int64_t nB = (int64_t)a.n * a.B;
  const int64_t gidx = (int64_t)blockIdx.x * 256 + tid;
  if (gidx >= nB * NPOS1) return;
  const int64_t b = gidx / NPOS1;
  const int pos = static_cast<int>(gidx - b * NPOS1), py = pos / Q1, px = pos % Q1;
  const int64_t row = cnn_row(a, b, pos == 0);
  if (pos == 0) {
    int lab = row >= 0 ? a.y[row] : 0;
    if (lab < 0 || lab >= a.C) {
      atomicOr(a.err, ERR_LABEL_RANGE);
      lab = 0;
    }
    a.ylab[b] = lab;
  }
  // the 6 x 6 input patch under the window's four 5 x 5 filters
  float in[6][6];
  const float* img = a.X + (row >= 0 ? row : 0) * (int64_t)(IMG * IMG);
#pragma unroll
  for (int r = 0; r < 6; ++r)
#pragma unroll
    for (int c = 0; c < 6; ++c) in[r][c] = row >= 0 ? img[(2 * py + r) * IMG + 2 * px + c] : 0.f;
  float* h1 = a.H1 + b * H1LEN + pos;
  uint8_t* cd = a.code1 + b * H1LEN + pos;
#pragma unroll 1
  for (int o = 0; o < NC1; ++o) {
    float z[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int dy = q >> 1, dx = q & 1;
      float s = sw[W1LEN + o];
#pragma unroll
      for (int u = 0; u < KS; ++u)
#pragma unroll
        for (int v = 0; v < KS; ++v) s = fmaf(in[dy + u][dx + v], sw[o * 25 + u * KS + v], s);
      z[q] = s;
    }
    int code = 0;
    float best = z[0];
#pragma unroll
    for (int q = 1; q < 4; ++q)
      if (z[q] > best) {
        best = z[q];
        code = q;
      }
    h1[o * NPOS1] = best > 0.f ? best : 0.f;
    cd[o * NPOS1] = static_cast<uint8_t>(best > 0.f ? code : 4);
  }
}

// ---------------------------------------------------------------------------
// Conv2 as a GEMM per image: Z[m][o] = sum_k A[m][k] W2[o][k], m = output
// position (y, x) of the 8 x 8, k = (channel, tap), A[m][k] = H1[c][y+u][x+v], on
// the split products (split_gemm.h).  A wave takes one image at a time, all 64
// positions x 64 filters (4 x 4 tiles; 50 filters), so that every im2col value
// is read from LDS once a wave.  The image lies in the wave's LDS as its three
// bf16 parts, channels innermost; K is ordered so that a lane's eight values
// are two runs of four channels at constant offsets from the lane's own
// address:
//   slices 0 .. 12   taps 2 s and 2 s + 1, channels 4 g .. 4 g + 3 (g = lane / 16)
//   slices 13 .. 15  channels 16 .. 19, row g of the taps, columns 2 s, 2 s + 1
//   slice 16         channels 16 .. 19, row 4, columns g and (g = 0) 4
// (entries past the 5 x 5 taps have zero weights).  W2's fragments pass through
// LDS a slice at a time, shared by the block's four waves; the next image's
// values are on their way in registers meanwhile.  Bias, 2 x 2 pooling and ReLU
// run in registers: a window's two rows are in lanes 32 apart.  With few images
// (SHARED) the block's waves take the same one, a column tile each.  8000
// images: 173 - 181 us, of which 8 - 14 are the test for decisions within rounding
// (fp32 matrix cores 294), 1.2 PFLOP/s of issued bf16 products;
// one wave a SIMD, so the LDS reads are placed by hand between the products of
// the column tile before (202 us left to the compiler).
constexpr int C2_SLICES = 17, C2_TILES = 4;
constexpr int C2_POS = 148;                        // positions of a part (144; reads with zero weights pass the end)
constexpr int C2_PART = C2_POS * NC1;              // bf16 values of one part
constexpr int C2_TASKS = (NPOS1 * 5 + 63) / 64;    // (position, four channels) pieces of a lane
constexpr int kConvBlocks = 256;                   // one block of four waves per CU
static_assert(NC1 == 20 && KS == 5, "slice layout");
constexpr int C2_FRAGS = C2_SLICES * C2_TILES * 3 * 64;   // pieces of Wc2's fragments; its filters' norms follow
static_assert(kCnnW2Bytes == C2_FRAGS * 16 + C2_TILES * 16 * 4, "fragments of Wc2 and the norms of its filters");

// Tap and first channel of run j (of two) of lane group g in a slice; tap -1:
// no such tap.
__device__ __forceinline__ void c2_run(int kb, int g, int j, int& tap, int& ch) {
  if (kb < 13) {
    tap = 2 * kb + j;
    ch = 4 * g;
  } else {
    const int u = kb < 16 ? g : 4, v = kb < 16 ? 2 * (kb - 13) + j : g + 4 * j;
    tap = v < KS ? u * KS + v : -1;
    ch = 16;
  }
  if (tap >= KS * KS) tap = -1;
}

__global__ __launch_bounds__(256) void k_cnn_pack_w2(CnnArgs a) {
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
  const int t = static_cast<int>(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (t >= C2_SLICES * C2_TILES) {
    // then a wave a filter: its norm
    const int o = t - C2_SLICES * C2_TILES;
    if (o >= C2_TILES * 16) return;
    float s = 0.f;
#pragma unroll
    for (int q = 0; q < (K2 + 63) / 64; ++q) {
      const int k = lane + 64 * q;
      const float v = o < NC2 && k < K2 ? a.w[a.off_c2 + o * K2 + k] : 0.f;
      s = fmaf(v, v, s);
    }
#pragma unroll
    for (int q = 32; q > 0; q >>= 1) s += __shfl_xor(s, q);
    if (lane == 0) reinterpret_cast<float*>(a.W2p + C2_FRAGS)[o] = sqrtf(s);
    return;
  }
  const int kb = t / C2_TILES, o = 16 * (t % C2_TILES) + c;
  float v[8];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    int tap, ch;
    c2_run(kb, g, j, tap, ch);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      v[4 * j + q] = o < NC2 && tap >= 0 ? a.w[a.off_c2 + o * K2 + (ch + q) * 25 + tap] : 0.f;
  }
  sg_store8(a.W2p, C2_TILES, kb * SG_K + 8 * g, o, v);
}

// Pooling of one 16 x 16 tile of Z (positions 16 mt .. x filters) in registers:
// z[r] = Z[y = 2 mt + g / 2][x = 4 (g % 2) + r]; lanes g and g ^ 2 hold the two rows of
// the windows, the lower pair finishes the left window, the upper pair the
// right one (window column px of c2_window).  w: the window's entries in
// row-major order, code: its first largest one.
struct C2Window {
  float w[4], best;
  int code;
};
__device__ __forceinline__ int c2_px(int g) { return 2 * (g & 1) + (g >> 1); }
__device__ __forceinline__ C2Window c2_window(const sg_f32x4& acc, float bias, int g) {
  C2Window p;
  const int s = g >> 1;
  float z[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) z[r] = acc[r] + bias;
  const float r0 = __shfl_xor(s ? z[0] : z[2], 32), r1 = __shfl_xor(s ? z[1] : z[3], 32);
  p.w[0] = s ? r0 : z[0];
  p.w[1] = s ? r1 : z[1];
  p.w[2] = s ? z[2] : r0;
  p.w[3] = s ? z[3] : r1;
  p.best = p.w[0];
  p.code = 0;
#pragma unroll
  for (int q = 1; q < 4; ++q)
    if (p.w[q] > p.best) {
      p.best = p.w[q];
      p.code = q;
    }
  return p;
}
__device__ __forceinline__ void c2_store(const CnnArgs& a, int b, int o, int mt, int px, const C2Window& p) {
  const int64_t f = (int64_t)b * FEAT + o * NQ2 + mt * Q2 + px;
  a.F[f] = p.best > 0.f ? p.best : 0.f;
  a.code2[f] = static_cast<uint8_t>(p.best > 0.f ? p.code : 4);
}

// Pooling and ReLU decisions that rounding could take either way.  A decision
// moves a whole window's gradient, so those that are closer than the
// roundings of Z are taken on the sums of the fp32 matrix instruction (K in
// steps of (tap, channel quad), tap by tap): the same decisions as if all of
// Z were formed with it.  Closer than tau = 2^-21 |H1 of the image| |filter| +
// 2^-18 |largest entry less its bias| + 2^-22 |bias|.  The two forms of a sum
// differ by up to 1.2 2^-24 |H1| |filter| over uniform, normal, sparse and nearly
// constant images with filters of either sign (two such differences make 0.3
// of the first term), by 9 where all is positive (then the second term is
// three times the first).  k_cnn_conv2_pool notes the windows (close2: bit 16 nt
// + 4 mt + g of the image's word, g the lane group of the window in tile (mt,
// nt)); k_cnn_conv2_close forms their tiles again: 16 - 18 us for 8000 images of
// 28 x 28 with 80% zeros, 22 for blank ones, 520 for constant ones with 0.1%
// noise, where every window is close.  (Done at once by the waves that find
// them, the first took 53 us: the wave that found most ended last.)
//
// Windows whose four patches are the same (blank parts of an image) tie in
// both forms and are left out; they are looked for in images where all column
// tiles note the same window.  A block takes four images: wave w compares the
// neighbours of image w, then forms row tile w of all four.
__global__ __launch_bounds__(256) void k_cnn_conv2_close(CnnArgs a) {
  __shared__ uint8_t same[4][NPOS1];   // H1 at a position equals its right (1), its lower neighbour (2), in all channels
  __shared__ uint64_t words[4];
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
  const int wv = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int b0 = static_cast<int>(blockIdx.x) * 4;
  {
    uint64_t word = b0 + wv < a.n * a.B ? a.close2[b0 + wv] : 0;
    uint64_t all = word & word >> 16 & word >> 32 & word >> 48 & 0xffffu;   // bit 4 mt + g
    if (all != 0) {
      const float* img = a.H1 + (int64_t)(b0 + wv) * H1LEN;
      for (int p = lane; p < NPOS1; p += 64) {
        const int right = p % Q1 + 1 < Q1 ? p + 1 : p, down = p + Q1 < NPOS1 ? p + Q1 : p;
        bool er = true, ed = true;
#pragma unroll
        for (int ch = 0; ch < NC1; ++ch) {
          const float v = img[ch * NPOS1 + p];
          er &= v == img[ch * NPOS1 + right];
          ed &= v == img[ch * NPOS1 + down];
        }
        same[wv][p] = static_cast<uint8_t>((er ? 1 : 0) | (ed ? 2 : 0));
      }
      asm volatile("" ::: "memory");   // the wave's LDS writes precede its reads
      // lane (g, mt): the window's patches are the same if all of their
      // neighbours in it are
      const int mt = c & 3, x = 2 * c2_px(g), y = 2 * mt;
      uint32_t r = 1, d = 2;
#pragma unroll
      for (int u = 0; u <= KS; ++u)
#pragma unroll
        for (int v = 0; v < KS; ++v) {
          const uint32_t e = same[wv][(y + u) * Q1 + x + v];
          r &= e;
          if (u < KS) d &= e;
        }
      const uint64_t blank = __builtin_amdgcn_ballot_w64(r != 0 && d != 0);   // bit 16 g + mt
      uint64_t drop = 0;
#pragma unroll
      for (int q = 0; q < 16; ++q) drop |= (blank >> (16 * (q & 3) + (q >> 2)) & 1) << q;
      drop &= all;
      word &= ~(drop | drop << 16 | drop << 32 | drop << 48);
    }
    if (lane == 0) words[wv] = word;
  }
  __syncthreads();
  const int mt = wv;
#pragma unroll 1
  for (int q = 0; q < 4; ++q) {
    const uint64_t word = words[q] >> 4 * mt;
    const float* img = a.H1 + (int64_t)(b0 + q) * H1LEN;
#pragma unroll 1
    for (int nt = 0; nt < 4; ++nt) {
      if ((word >> 16 * nt & 15u) == 0) continue;
      const int o = 16 * nt + c;
      const float* h = img + g * NPOS1 + (2 * mt + (c >> 3)) * Q1 + (c & 7);
      const float* w = a.w + a.off_c2 + (o < NC2 ? o : 0) * K2 + g * 25;
      sg_f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < 25; ++t)
#pragma unroll
        for (int cq = 0; cq < NC1 / 4; ++cq)
          acc = __builtin_amdgcn_mfma_f32_16x16x4f32(h[4 * cq * NPOS1 + t / KS * Q1 + t % KS], w[4 * cq * 25 + t], acc, 0, 0, 0);
      const C2Window p = c2_window(acc, a.w[a.off_c2 + NC2 * K2 + (o < NC2 ? o : 0)], g);
      if (o < NC2) c2_store(a, b0 + q, o, mt, c2_px(g), p);
    }
  }
}

template <bool SHARED>
__global__ __launch_bounds__(256, 1) void k_cnn_conv2_pool(CnnArgs a) {
  constexpr int NT = SHARED ? 1 : C2_TILES;         // column tiles of a wave
  constexpr int IMAGES = SHARED ? 1 : 4;            // images of a block
  __shared__ __align__(16) uint16_t img[4][3][C2_PART];
  __shared__ SgLds<C2_TILES, 4> L;
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const float* b2 = a.w + a.off_c2 + NC2 * K2;
  const int nt0 = SHARED ? wv : 0;
  float bias[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) bias[nt] = 16 * (nt0 + nt) + c < NC2 ? b2[16 * (nt0 + nt) + c] : 0.f;
  float wnorm[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) wnorm[nt] = reinterpret_cast<const float*>(a.W2p + C2_FRAGS)[16 * (nt0 + nt) + c];
  for (int e = lane; e < 3 * C2_PART; e += 64) (&img[wv][0][0])[e] = 0;
  const int nB = a.n * a.B;
  float4 h[C2_TASKS];
  auto fetch = [&](int b) {
#pragma unroll
    for (int s = 0; s < C2_TASKS; ++s) {
      const int e = lane + 64 * s, cq = e / NPOS1, pos = e - cq * NPOS1;
      const bool ok = b < nB && e < NPOS1 * 5;
      const float* src = a.H1 + (int64_t)(ok ? b : 0) * H1LEN + (ok ? 4 * cq * NPOS1 + pos : 0);
      h[s] = make_float4(src[0], src[NPOS1], src[2 * NPOS1], src[3 * NPOS1]);
    }
  };
  // into LDS as parts; returns the sum of the image's squares
  auto put = [&]() {
    float sq = 0.f;
#pragma unroll
    for (int s = 0; s < C2_TASKS; ++s) {
      const int e = lane + 64 * s, cq = e / NPOS1, pos = e - cq * NPOS1;
      if (e >= NPOS1 * 5) break;
      const SgPair u = sg_split2(h[s].x, h[s].y), v = sg_split2(h[s].z, h[s].w);
      uint16_t* p = &img[wv][0][pos * NC1 + 4 * cq];
      *reinterpret_cast<sg_u32x2*>(p) = sg_u32x2{u.h, v.h};
      *reinterpret_cast<sg_u32x2*>(p + C2_PART) = sg_u32x2{u.m, v.m};
      *reinterpret_cast<sg_u32x2*>(p + 2 * C2_PART) = sg_u32x2{u.l, v.l};
      sq = fmaf(h[s].x, h[s].x, fmaf(h[s].y, h[s].y, fmaf(h[s].z, h[s].z, fmaf(h[s].w, h[s].w, sq))));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o);
    return sq;
  };
  sg_u32x4 rb[3];
  auto fetch_w = [&](int kb) {
#pragma unroll
    for (int q = 0; q < 3; ++q) rb[q] = a.W2p[(sg_frag(kb, C2_TILES, 0, 0) + wv + 4 * q) * 64 + lane];
  };
  auto stage_w = [&](int buf) {
#pragma unroll
    for (int q = 0; q < 3; ++q) L.B[buf][wv + 4 * q][lane] = rb[q];
  };
  // position of tile row c (m = 16 mt + c: y = 2 mt + c / 8, x = c % 8)
  const int pos0 = (c >> 3) * Q1 + (c & 7);
  const uint16_t* im = &img[wv][0][0];
  const uint16_t* base1 = im + pos0 * NC1 + 4 * g;
  const uint16_t* base2 = im + (pos0 + g * Q1) * NC1 + 16;
  const uint16_t* base3 = im + (pos0 + 4 * Q1 + g) * NC1 + 16;
  const int stride = static_cast<int>(gridDim.x) * IMAGES;
  int b = static_cast<int>(blockIdx.x) * IMAGES + (SHARED ? 0 : wv);
  fetch_w(0);
  fetch(b);
  stage_w(0);
  __syncthreads();
  int buf = 0;
  for (int b0 = static_cast<int>(blockIdx.x) * IMAGES; b0 < nB; b0 += stride, b += stride) {
    const float hnorm = sqrtf(put());
    asm volatile("" ::: "memory");   // the wave's LDS writes precede its reads
    fetch(b + stride);
    sg_f32x4 acc[NT][4];
    sg_zero<4, NT>(acc);
    // tile mt of a slice's A operand
    auto operand = [&](int kb, int mt, SgParts& A) {
      sg_u32x4 v[3];
#pragma unroll
      for (int part = 0; part < 3; ++part) {
        sg_u32x2 run[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const uint16_t* p;
          if (kb < 13) {
            const int t = 2 * kb + j < 25 ? 2 * kb + j : 24;
            p = base1 + (t / KS * Q1 + t % KS) * NC1;
          } else if (kb < 16) {
            p = base2 + (2 * (kb - 13) + j) * NC1;
          } else {
            p = base3 + 4 * j * NC1;
          }
          run[j] = *reinterpret_cast<const sg_u32x2*>(p + part * C2_PART + 2 * mt * Q1 * NC1);
        }
        v[part] = sg_u32x4{run[0].x, run[0].y, run[1].x, run[1].y};
      }
      A.h = v[0];
      A.m = v[1];
      A.l = v[2];
    };
    SgParts A[2][4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) operand(0, mt, A[0][mt]);
#pragma unroll
    for (int kb = 0; kb < C2_SLICES; ++kb) {
      // while a column tile is multiplied, the next one's fragments and a
      // quarter of the next slice's A operand are read
      sg_u32x4 w[2][3];
#pragma unroll
      for (int q = 0; q < 3; ++q) w[0][q] = L.B[buf][3 * nt0 + q][lane];
      fetch_w(kb + 1 < C2_SLICES ? kb + 1 : 0);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        if (nt + 1 < NT)
#pragma unroll
          for (int q = 0; q < 3; ++q) w[(nt + 1) & 1][q] = L.B[buf][3 * (nt + 1) + q][lane];
        if (kb + 1 < C2_SLICES)
#pragma unroll
          for (int mt = nt; mt < (SHARED ? 4 : nt + 1); ++mt) operand(kb + 1, mt, A[(kb + 1) & 1][mt]);
        __builtin_amdgcn_sched_barrier(0);
        sg_products<false, 4>(A[kb & 1], w[nt & 1][0], w[nt & 1][1], w[nt & 1][2], acc[nt]);
        __builtin_amdgcn_sched_barrier(0);
      }
      stage_w(buf ^ 1);
      sg_barrier();
      buf ^= 1;
    }
    const bool have = b < nB;
    // (K index 20 tap + channel, the order of k_cnn_conv2_close)
    sg_redo<4, NT>(
        acc, K2,
        [&](int mt, int k) {
          const int t = k / NC1, ch = k % NC1;
          return a.H1[(int64_t)(have ? b : 0) * H1LEN + ch * NPOS1 + (2 * mt + (c >> 3) + t / KS) * Q1 + (c & 7) + t % KS];
        },
        [&](int nt, int k) {
          const int o = 16 * (nt0 + nt) + c;
          const float v = a.w[a.off_c2 + min(o, NC2 - 1) * K2 + k % NC1 * 25 + k / NC1];
          return o < NC2 ? v : 0.f;
        });
    uint64_t close = 0;   // windows decided within rounding (k_cnn_conv2_close)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int o = 16 * (nt0 + nt) + c;
      const float tau0 = 0x1p-21f * hnorm * wnorm[nt] + 0x1p-22f * fabsf(bias[nt]);
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        const C2Window p = c2_window(acc[nt][mt], bias[nt], g);
        if (have && o < NC2) c2_store(a, b, o, mt, c2_px(g), p);
        const float tau = fmaf(0x1p-18f, fabsf(p.best - bias[nt]), tau0);
        int within = fabsf(p.best) < tau ? 2 : 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) within += p.best - p.w[q] < tau;   // (the largest itself is one)
        const uint64_t m = __builtin_amdgcn_ballot_w64(within >= 2 && o < NC2);
        if (m != 0)
#pragma unroll
          for (int q = 0; q < 4; ++q) close |= (m >> 16 * q & 0xffffu) != 0 ? uint64_t{1} << (16 * nt + 4 * mt + q) : 0u;
      }
    }
    if (have && lane == 0) {
      if (SHARED) reinterpret_cast<uint16_t*>(a.close2 + b)[wv] = static_cast<uint16_t>(close);
      else a.close2[b] = close;
    }
  }
}

// ---------------------------------------------------------------------------
// dP2[m][f] = sum_h dA[m][h] Wf1[f][h] on MT x DF_NT tiles of 16 x 16 per wave
// (split_gemm.h), Wf1^T as fragments; blockIdx.x = 4 MT row tiles, y = DF_NT
// column tiles.  8000 x 800 x 500: 92 us on the fp32 matrix cores.
constexpr int DF_NT = 5, DF_TILES = FEAT / 16;
static_assert(DF_TILES % DF_NT == 0, "whole column chunks");
template <int MT, bool TINY>
__global__ __launch_bounds__(256, 2) void k_cnn_dfeat(CnnArgs a) {
  __shared__ SgLds<DF_NT, 4> L;
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nB = a.n * a.B, H = a.H;   // nB below 2^30
  const int m0 = (static_cast<int>(blockIdx.x) * 4 + wv) * MT * 16, nt0 = static_cast<int>(blockIdx.y) * DF_NT;
  SgRows<MT, TINY> A(make_rsrc(a.dA, static_cast<uint32_t>((int64_t)nB * H * 4)), H);
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    const int m = m0 + 16 * t + c;
    A.roff[t] = m < nB ? static_cast<uint32_t>((int64_t)m * H * 4) + 32 * g : kOutOfRange;
  }
  sg_f32x4 acc[DF_NT][MT];
  sg_zero<MT, DF_NT>(acc);
  sg_loop<true, MT, DF_NT, 4, 2>(
      L, 0, A.slices(), A, [&](int kb, float (&x)[MT][8]) { A.prep(kb, x); },
      [&](int kb) { return a.Wp + sg_frag(kb, DF_TILES, nt0, 0) * 64; }, acc);
  sg_redo<MT, DF_NT>(
      acc, H,
      [&](int t, int k) {
        const int m = m0 + 16 * t + c;
        const float v = a.dA[(int64_t)min(m, nB - 1) * H + k];
        return m < nB ? v : 0.f;
      },
      [&](int nt, int k) { return a.w[(int64_t)((nt0 + nt) * 16 + c) * H + k]; });
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = m0 + 16 * t + 4 * g + r;
      if (m >= nB) continue;
#pragma unroll
      for (int nt = 0; nt < DF_NT; ++nt) a.dP2[(int64_t)m * FEAT + (nt0 + nt) * 16 + c] = acc[nt][t][r];
    }
}

// ---------------------------------------------------------------------------
// Gradient at H1.  Per image the pooled gradient is unpooled into dZ2[m][o]
// (its value at the window's passing entry, 0 at the other three), and
// dcols[m][(c, t)] = sum_o dZ2[m][o] W2[o][c][t] is a 64 x 25 x 50 GEMM per
// input channel c on the matrix cores (4 x 2 tiles of 16 x 16, K = 50 padded
// to 52).  Each wave owns five channels and holds their W2 fragments in
// registers for the whole (persistent) launch.  The fold back onto H1,
// dH1[c][p] = sum_{t = (u, v)} dcols[p - (u, v)][(c, t)], goes through a
// wave-private LDS copy of the channel's 25 tap maps, each stored in a
// zero-framed 12 x 12 tile (data in rows and columns 4..11) so that a target's
// 25 reads sit at fixed offsets from it and out-of-range taps read zeros.
constexpr int DG_CPW = NC1 / 4;          // channels per wave (4 waves)
constexpr int DG_KS = (NC2 + 3) / 4;     // 13 K steps of 4 filters
constexpr int SA_LD = 80;                // unpooled-gradient row stride (bank spread)
constexpr int DT = 12 * 12;              // one framed tap map
constexpr int DLEN = 25 * DT + 64;       // 25 maps and a zero tail
constexpr int kDgradBlocks = 512;        // two blocks per CU

__global__ __launch_bounds__(256, 2) void k_cnn_conv2_dgrad(CnnArgs a) {
  __shared__ float sA[52 * SA_LD];                     // [o][m]
  __shared__ __align__(16) float sD[4][DLEN];           // per wave
  // the next image's pooled gradient and codes, loaded straight into LDS
  // while the current image is multiplied
  __shared__ float rawg[FEAT];
  __shared__ uint32_t rawc[FEAT / 4];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, g = lane >> 4, j = lane & 15;
  for (int i = tid; i < 4 * DLEN; i += 256) (&sD[0][0])[i] = 0.f;
  for (int i = tid; i < 2 * SA_LD; i += 256) sA[NC2 * SA_LD + i] = 0.f;   // rows o = 50, 51
  // B fragments: W2[o = 4 ks + g][c][t = 16 nt + j] of the wave's channels
  const float* W2 = a.w + a.off_c2;
  float wb[DG_CPW][2][DG_KS];
#pragma unroll
  for (int ci = 0; ci < DG_CPW; ++ci)
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
      for (int ks = 0; ks < DG_KS; ++ks) {
        const int o = 4 * ks + g, t = 16 * nt + j, c = DG_CPW * wv + ci;
        wb[ci][nt][ks] = o < NC2 && t < 25 ? W2[o * K2 + c * 25 + t] : 0.f;
      }
  float* D = sD[wv];
  const int64_t nB = (int64_t)a.n * a.B;
  auto fetch = [&](int64_t bn) {
    // wave wv copies pieces wv, wv + 4, .. of 64 dwords; lanes past the end
    // stay idle
    for (int k = wv; k * 64 < FEAT + FEAT / 4; k += 4) {
      const int e = 64 * k + lane;
      if (e < FEAT)
        __builtin_amdgcn_global_load_lds(a.dP2 + bn * FEAT + e, rawg + 64 * k, 4, 0, 0);
      else if (e < FEAT + FEAT / 4)
        __builtin_amdgcn_global_load_lds(reinterpret_cast<const uint32_t*>(a.code2 + bn * FEAT) + (e - FEAT),
                                         rawc + (64 * k - FEAT), 4, 0, 0);
    }
  };
  if (blockIdx.x < nB) fetch(blockIdx.x);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  for (int64_t b = blockIdx.x; b < nB; b += gridDim.x) {
    // unpool: task (o, q) writes the four entries of its window in row o
    const uint8_t* rc = reinterpret_cast<const uint8_t*>(rawc);
    for (int e = tid; e < FEAT; e += 256) {
      const int o = e / NQ2, q = e % NQ2;
      const int m0 = 2 * (q / Q2) * O2 + 2 * (q % Q2);
      const float gv = rawg[e];
      const int cd = rc[e];
      float* row = sA + o * SA_LD + m0;
      row[0] = cd == 0 ? gv : 0.f;
      row[1] = cd == 1 ? gv : 0.f;
      row[O2] = cd == 2 ? gv : 0.f;
      row[O2 + 1] = cd == 3 ? gv : 0.f;
    }
    __syncthreads();
    if (b + gridDim.x < nB) fetch(b + gridDim.x);
    // dcols of channel ci on the matrix cores
    auto products = [&](int ci, mfma_f32x4 (&acc)[4][2]) {
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) acc[mt][nt] = mfma_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < DG_KS; ++ks) {
        float av[4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) av[mt] = sA[(4 * ks + g) * SA_LD + 16 * mt + j];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
          for (int nt = 0; nt < 2; ++nt)
            acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[mt], wb[ci][nt][ks], acc[mt][nt], 0, 0, 0);
      }
    };
    // acc[mt][nt][r]: m = 16 mt + 4 g + r (y = 2 mt + g / 2, x = 4 (g % 2) + r),
    // tap t = 16 nt + j, into the framed tap maps
    auto store = [&](const mfma_f32x4 (&acc)[4][2]) {
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
          const int t = 16 * nt + j;
          if (t < 25) {
            float* cell = D + t * DT + (2 * mt + (g >> 1) + 4) * 12 + 4 * (g & 1) + 4;
            *reinterpret_cast<float4*>(cell) =
                make_float4(acc[mt][nt][0], acc[mt][nt][1], acc[mt][nt][2], acc[mt][nt][3]);
          }
        }
    };
    auto fold = [&](int c) {
      float* dp1 = a.dP1 + b * H1LEN + c * NPOS1;
#pragma unroll
      for (int pp = 0; pp < 3; ++pp) {
        const int p = lane + 64 * pp;
        if (p < NPOS1) {
          // framed cell of (t, y = py - u, x = px - v) = p + 52 + 708 u + 143 v
          const float* src = D + p + 52;
          float su[KS];                  // one short add chain per tap row
#pragma unroll
          for (int u = 0; u < KS; ++u) {
            su[u] = src[708 * u];
#pragma unroll
            for (int v = 1; v < KS; ++v) su[u] += src[708 * u + 143 * v];
          }
          dp1[p] = ((su[0] + su[1]) + (su[2] + su[3])) + su[4];
        }
        // one target's reads in flight at a time; matrix-core work may cross
        __builtin_amdgcn_sched_barrier(0x8);
      }
    };
    // channel ci + 1's products run while channel ci is folded: they need
    // neither its maps nor its results
    mfma_f32x4 acc[4][2];
    products(0, acc);
#pragma unroll   // register index ci
    for (int ci = 0; ci < DG_CPW; ++ci) {
      store(acc);
      asm volatile("" ::: "memory");   // the wave's LDS ops stay in program order
      if (ci + 1 < DG_CPW) products(ci + 1, acc);
      fold(DG_CPW * wv + ci);
      asm volatile("" ::: "memory");
    }
    __builtin_amdgcn_s_waitcnt(0);   // the next image's copy has landed
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// dW2, db2 partial of chunk j of worker i (images i B + j chunk .., in order):
// dW2[o][n] += sum_m dZ2[m][o] H1[c][m + t] with n = (c, t) = 25 c + t, a
// 64 x 512 x 64 GEMM per image on the matrix cores (o padded to 64, n to 512;
// the padded columns read a zero region, except column 500, which reads ones
// and so collects db2).  Each of the four waves owns 8
// column tiles and keeps its 4 x 8 accumulator tiles over the chunk; the
// image's H1 and unpooled gradient are staged in LDS, the next image's loads
// in flight meanwhile.
constexpr int WG_NT = 8;                 // column tiles per wave
constexpr int WG_ZERO = H1LEN;           // zero region after the image's H1
constexpr int WG_ONES = H1LEN + 96;      // then a region of ones
constexpr int WG_H1 = H1LEN + 192;
struct WgradBuf {
  float h1[WG_H1];
  float A[NPOS2 * SA_LD];                // [m][o]
};

__global__ __launch_bounds__(256) void k_cnn_conv2_wgrad(CnnArgs a) {
  __shared__ __align__(16) WgradBuf L[2];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, g = lane >> 4, j = lane & 15;
  const int i = blockIdx.y, jc = blockIdx.x;
  const int b0 = jc * a.chunk, b1 = min(a.B, b0 + a.chunk);
  for (int e = tid; e < 2 * 192; e += 256) L[e / 192].h1[WG_ZERO + e % 192] = e % 192 < 96 ? 0.f : 1.f;
  for (int e = tid; e < 2 * NPOS2 * (SA_LD - NC2); e += 256) {
    const int bi = e / (NPOS2 * (SA_LD - NC2)), r = e % (NPOS2 * (SA_LD - NC2));
    L[bi].A[(r / (SA_LD - NC2)) * SA_LD + NC2 + r % (SA_LD - NC2)] = 0.f;
  }
  // per column tile: the lane's H1 offset of tap (c, u, v), or the zero region
  int colbase[WG_NT];
#pragma unroll
  for (int nt = 0; nt < WG_NT; ++nt) {
    const int n = 16 * (WG_NT * wv + nt) + j;
    const int c = n / 25, t = n % 25;
    colbase[nt] = (n < K2 ? c * NPOS1 + (t / 5) * Q1 + t % 5 : n == K2 ? WG_ONES : WG_ZERO) + g;
  }
  float4 rh[3];
  float rg[4];
  uint8_t rc[4];
  auto fetch = [&](int64_t b) {
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      const int e = tid + 256 * s;
      rh[s] = e < H1LEN / 4 ? reinterpret_cast<const float4*>(a.H1 + b * H1LEN)[e] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int e = tid + 256 * s;
      rg[s] = e < FEAT ? a.dP2[b * FEAT + e] : 0.f;
      rc[s] = e < FEAT ? a.code2[b * FEAT + e] : 0;
    }
  };
  auto stage = [&](WgradBuf& B) {
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      const int e = tid + 256 * s;
      if (e < H1LEN / 4) reinterpret_cast<float4*>(B.h1)[e] = rh[s];
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int e = tid + 256 * s;
      if (e < FEAT) {
        const int o = e / NQ2, q = e % NQ2, m0 = 2 * (q / Q2) * O2 + 2 * (q % Q2);
        float* col = B.A + m0 * SA_LD + o;
        col[0] = rc[s] == 0 ? rg[s] : 0.f;
        col[SA_LD] = rc[s] == 1 ? rg[s] : 0.f;
        col[O2 * SA_LD] = rc[s] == 2 ? rg[s] : 0.f;
        col[(O2 + 1) * SA_LD] = rc[s] == 3 ? rg[s] : 0.f;
      }
    }
  };
  mfma_f32x4 acc[4][WG_NT];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int nt = 0; nt < WG_NT; ++nt) acc[mt][nt] = mfma_f32x4{0.f, 0.f, 0.f, 0.f};
  if (b0 < b1) {
    fetch((int64_t)i * a.B + b0);
    stage(L[0]);
  }
  __syncthreads();
  for (int bb = b0; bb < b1; ++bb) {
    const int cur = (bb - b0) & 1;
    const int64_t b = (int64_t)i * a.B + bb;
    if (bb + 1 < b1) fetch(b + 1);
    const float* A = L[cur].A + g * SA_LD + j;
    const float* H = L[cur].h1;
#pragma unroll
    for (int ks = 0; ks < NPOS2 / 4; ++ks) {
      // K index m = 4 ks + g: y = ks / 2, x = 4 (ks % 2) + g
      const int moff = (ks >> 1) * Q1 + 4 * (ks & 1);
      float av[4], bv[WG_NT];
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) av[mt] = A[4 * ks * SA_LD + 16 * mt];
#pragma unroll
      for (int nt = 0; nt < WG_NT; ++nt) bv[nt] = H[colbase[nt] + moff];
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int nt = 0; nt < WG_NT; ++nt)
          acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[mt], bv[nt], acc[mt][nt], 0, 0, 0);
    }
    if (bb + 1 < b1) stage(L[cur ^ 1]);
    __syncthreads();
  }
  // partial [i][jc][W2 (50 x 500) | b2 (50)]; acc[mt][nt][r] is (o = 16 mt + 4 g + r, n)
  float* p = a.part2 + ((int64_t)i * gridDim.x + jc) * (NC2 * K2 + NC2);
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int nt = 0; nt < WG_NT; ++nt) {
      const int n = 16 * (WG_NT * wv + nt) + j;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int o = 16 * mt + 4 * g + r;
        if (o < NC2 && n <= K2) p[n < K2 ? o * K2 + n : NC2 * K2 + o] = acc[mt][nt][r];
      }
    }
}

// ---------------------------------------------------------------------------
// dW1, db1 partial of chunk j of worker i: dW1[o][t] += sum_m dZ1[o][m]
// X[m + t] over the 24 x 24 conv1 outputs m of each image, a GEMM (filters x
// taps, K = positions) on the matrix cores.  K runs over (pooled position p,
// window offset d): the lanes of group d = lane / 16 take the pooled gradient
// of p where the window's code is d and 0 elsewhere, which is the unpooled
// dZ1.  Tap column 25 is all ones, so it collects db1.  Each wave takes whole
// images of the chunk (every fourth), staged in its own LDS region while the
// next one is loaded into registers; the four waves' partial tiles are
// summed in wave order at the end.
constexpr int C1_LD = NPOS1 + 1;         // bank spread of the [o][p] rows
struct Wg1Buf {
  float x[IMG * IMG];
  float g[NC1 * C1_LD];
  uint8_t cd[NC1 * C1_LD + 12];
};
constexpr int C1_X4 = (IMG * IMG / 4 + 63) / 64;     // float4 pieces per lane
constexpr int C1_G4 = (H1LEN / 4 + 63) / 64;

__global__ __launch_bounds__(256, 2) void k_cnn_conv1_wgrad(CnnArgs a) {
  __shared__ __align__(16) Wg1Buf L[4];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, g = lane >> 4, j = lane & 15;
  const int i = blockIdx.y, jc = blockIdx.x;
  const int b0 = jc * a.chunk, b1 = min(a.B, b0 + a.chunk);
  Wg1Buf& B = L[wv];
  // B operand of lane (d = g, tap t = 16 nt + j): X[(2 py + d / 2 + u) 28 + 2 px + d % 2 + v]
  int xb[2];
  float bconst[2];
  bool bx[2];
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    const int t = 16 * nt + j;
    bx[nt] = t < 25;
    xb[nt] = t < 25 ? ((g >> 1) + t / 5) * IMG + (g & 1) + t % 5 : 0;
    bconst[nt] = t == 25 ? 1.f : 0.f;
  }
  // A operand row o = 16 mt + j (filters 20 .. 31 read row 0 and contribute 0)
  int arow[2];
  bool aval[2];
#pragma unroll
  for (int mt = 0; mt < 2; ++mt) {
    aval[mt] = 16 * mt + j < NC1;
    arow[mt] = aval[mt] ? (16 * mt + j) * C1_LD : 0;
  }
  float4 rx[C1_X4], rg[C1_G4];
  uint32_t rc[C1_G4];
  auto fetch = [&](int64_t b) {
    const int64_t row = cnn_row(a, b, false);
#pragma unroll
    for (int s = 0; s < C1_X4; ++s) {
      const int e = lane + 64 * s;
      rx[s] = e < IMG * IMG / 4 && row >= 0 ? reinterpret_cast<const float4*>(a.X + row * (IMG * IMG))[e]
                                            : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int s = 0; s < C1_G4; ++s) {
      const int e = lane + 64 * s;
      rg[s] = e < H1LEN / 4 ? reinterpret_cast<const float4*>(a.dP1 + b * H1LEN)[e] : make_float4(0.f, 0.f, 0.f, 0.f);
      rc[s] = e < H1LEN / 4 ? reinterpret_cast<const uint32_t*>(a.code1 + b * H1LEN)[e] : 0u;
    }
  };
  auto stage = [&]() {
#pragma unroll
    for (int s = 0; s < C1_X4; ++s) {
      const int e = lane + 64 * s;
      if (e < IMG * IMG / 4) reinterpret_cast<float4*>(B.x)[e] = rx[s];
    }
#pragma unroll
    for (int s = 0; s < C1_G4; ++s) {
      const int e = lane + 64 * s;
      if (e < H1LEN / 4) {
        const int o = (4 * e) / NPOS1, p = (4 * e) % NPOS1;   // 144 % 4 == 0: one row
        float* gd = B.g + o * C1_LD + p;
        uint8_t* cd = B.cd + o * C1_LD + p;
        gd[0] = rg[s].x; gd[1] = rg[s].y; gd[2] = rg[s].z; gd[3] = rg[s].w;
        cd[0] = rc[s] & 0xff; cd[1] = (rc[s] >> 8) & 0xff; cd[2] = (rc[s] >> 16) & 0xff; cd[3] = rc[s] >> 24;
      }
    }
  };
  mfma_f32x4 acc[2][2];
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) acc[mt][nt] = mfma_f32x4{0.f, 0.f, 0.f, 0.f};
  int bb = b0 + wv;
  if (bb < b1) fetch((int64_t)i * a.B + bb);
  for (; bb < b1; bb += 4) {
    stage();
    asm volatile("" ::: "memory");       // the wave's LDS writes precede its reads
    if (bb + 4 < b1) fetch((int64_t)i * a.B + bb + 4);
    // pooled row py, column px: every read is unconditional (padding lanes
    // read valid cells and select), offsets are immediates within a row
#pragma unroll 1
    for (int py = 0; py < Q1; ++py) {
      const float* gr0 = B.g + arow[0] + py * Q1;
      const float* gr1 = B.g + arow[1] + py * Q1;
      const uint8_t* cr0 = B.cd + arow[0] + py * Q1;
      const uint8_t* cr1 = B.cd + arow[1] + py * Q1;
      const float* xr0 = B.x + xb[0] + 2 * py * IMG;
      const float* xr1 = B.x + xb[1] + 2 * py * IMG;
#pragma unroll
      for (int px = 0; px < Q1; ++px) {
        const float g0 = gr0[px], g1 = gr1[px];
        const int c0 = cr0[px], c1 = cr1[px];
        const float x0 = xr0[2 * px], x1 = xr1[2 * px];
        const float av0 = ((c0 == g) & aval[0]) ? g0 : 0.f;
        const float av1 = ((c1 == g) & aval[1]) ? g1 : 0.f;
        const float bv0 = bx[0] ? x0 : bconst[0];
        const float bv1 = bx[1] ? x1 : bconst[1];
        acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(av0, bv0, acc[0][0], 0, 0, 0);
        acc[0][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(av0, bv1, acc[0][1], 0, 0, 0);
        acc[1][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(av1, bv0, acc[1][0], 0, 0, 0);
        acc[1][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(av1, bv1, acc[1][1], 0, 0, 0);
      }
    }
    asm volatile("" ::: "memory");       // reads done before the next image's writes
  }
  // acc[mt][nt][r] = (o = 16 mt + 4 g + r, t = 16 nt + j); the four waves'
  // tiles meet in the staging LDS, now free
  __syncthreads();
  float (*red)[32][33] = reinterpret_cast<float (*)[32][33]>(&L[0]);
  static_assert(sizeof(float) * 4 * 32 * 33 <= sizeof(L), "reduction tiles fit in the staging LDS");
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wv][16 * mt + 4 * g + r][16 * nt + j] = acc[mt][nt][r];
  __syncthreads();
  // partial [i][jc][W1 (20 x 25) | b1 (20)]
  float* part = a.part1 + ((int64_t)i * gridDim.x + jc) * (W1LEN + NC1);
  for (int e = tid; e < NC1 * 26; e += 256) {
    const int o = e / 26, t = e % 26;
    const float s = ((red[0][o][t] + red[1][o][t]) + red[2][o][t]) + red[3][o][t];
    part[t < 25 ? o * 25 + t : W1LEN + o] = s;
  }
}

// ---------------------------------------------------------------------------
// G[i][off_c1 + e] = sum over chunks in order of the partials (conv1 block
// then conv2 block, which are contiguous in w).
__global__ __launch_bounds__(256) void k_cnn_wreduce(CnnArgs a, int chunks) {
  const int i = blockIdx.y;
  const int e = blockIdx.x * 256 + threadIdx.x;
  constexpr int L1 = W1LEN + NC1, L2 = NC2 * K2 + NC2;
  if (e >= L1 + L2) return;
  const float* src = e < L1 ? a.part1 + (int64_t)i * chunks * L1 + e : a.part2 + (int64_t)i * chunks * L2 + (e - L1);
  const int64_t stride = e < L1 ? L1 : L2;
  float s = 0.f;
  for (int j0 = 0; j0 < chunks; j0 += 8) {
    // eight chunks' partials in flight, then added in chunk order (a plain
    // loop over the run-time chunk count waits for each load in turn)
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = j0 + u < chunks ? src[(j0 + u) * stride] : 0.f;
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (j0 + u < chunks) s += v[u];
  }
  if (!a.row_mask || a.row_mask[i]) a.G[(int64_t)i * a.P + a.off_c1 + e] = s;
}

}  // namespace

int cnn_chunks(int B) { return (B + kCnnChunk - 1) / kCnnChunk; }

hipError_t launch_cnn_grads(const MlpPlan& mplan, const CnnArgs& a, hipStream_t s) {
  const int64_t nB = (int64_t)a.n * a.B;
  hipLaunchKernelGGL(k_cnn_conv1_pool, dim3(static_cast<unsigned>((nB * NPOS1 + 255) / 256)), dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_cnn_pack_w2, dim3((C2_SLICES + 16) * C2_TILES / 4), dim3(256), 0, s, a);
  // up to two images a CU the four waves of a block share one (a wave takes
  // about 20 us over an image of its own)
  if (nB <= 2 * kConvBlocks)
    hipLaunchKernelGGL(k_cnn_conv2_pool<true>, dim3(static_cast<unsigned>(std::min<int64_t>(nB, kConvBlocks))), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL(k_cnn_conv2_pool<false>, dim3(static_cast<unsigned>(std::min<int64_t>((nB + 3) / 4, kConvBlocks))),
                       dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_cnn_conv2_close, dim3(static_cast<unsigned>((nB + 3) / 4)), dim3(256), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // the fully connected part: the MLP 800-H-C on the features, its G block
  // at the start of each row of G
  MlpArgs m{};
  m.w = a.w; m.X = a.F; m.y = a.ylab; m.rows = nullptr; m.S = 0;
  m.n = a.n; m.B = a.B; m.d = FEAT; m.H = a.H; m.C = a.C;
  m.G = a.G; m.ldG = a.P; m.loss = a.loss;
  m.Hh = a.Hh; m.Wp = a.Wp; m.Dp = a.Dp; m.dA = a.dA; m.Gp = a.Gp; m.lossp = a.lossp; m.err = a.err; m.row_mask = a.row_mask;
  e = launch_mlp_grads(mplan, m, s);
  if (e != hipSuccess) return e;
  // Wf1's own fragments are no longer needed: its transpose takes their place
  const int64_t tasks = (int64_t)((a.H + SG_K - 1) / SG_K) * DF_TILES;
  hipLaunchKernelGGL(k_sg_pack, dim3(static_cast<unsigned>((tasks + 3) / 4)), dim3(256), 0, s, a.w, int64_t{1}, (int64_t)a.H,
                     a.H, FEAT, DF_TILES, a.Wp);
  auto dfeat = [&](auto kernel, int rows) {
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>((nB + rows - 1) / rows), DF_TILES / DF_NT), dim3(256), 0, s, a);
  };
  if (a.H < 8) dfeat(k_cnn_dfeat<1, true>, 64);
  else if (nB < 4096) dfeat(k_cnn_dfeat<1, false>, 64);
  else dfeat(k_cnn_dfeat<2, false>, 128);
  const int64_t dg_blocks = nB < kDgradBlocks ? nB : kDgradBlocks;
  hipLaunchKernelGGL(k_cnn_conv2_dgrad, dim3(static_cast<unsigned>(dg_blocks)), dim3(256), 0, s, a);
  const int chunks = cnn_chunks(a.B);
  hipLaunchKernelGGL(k_cnn_conv2_wgrad, dim3(chunks, a.n), dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_cnn_conv1_wgrad, dim3(chunks, a.n), dim3(256), 0, s, a);
  constexpr int LW = W1LEN + NC1 + NC2 * K2 + NC2;
  hipLaunchKernelGGL(k_cnn_wreduce, dim3((LW + 255) / 256, a.n), dim3(256), 0, s, a, chunks);
  return hipGetLastError();
}

}  // namespace dbw
