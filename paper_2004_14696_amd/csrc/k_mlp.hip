// Worker minibatch gradients of the two-layer ReLU MLP (Sect. 2, Eq. gradient), gfx950.
//
// For worker i with rows x_b (b < B), parameters [W1 (d x H) | b1 | W2 (H x C) | b2]:
//   A = X W1 + b1,  Hh = relu(A),  Z = Hh W2 + b2,  R = (softmax(Z) - Y) / B
//   dW2 = Hh^T R,  db2 = sum_b R,  dA = (R W2^T) * [A > 0],
//   dW1 = X^T dA,  db1 = sum_b dA,  loss = mean_b CE.
// ReLU'(0) = 0; [A > 0] is read from Hh > 0, which is the same predicate.
//
// Kernels (one stream, in order); the two products run on the bf16 matrix
// cores with every fp32 operand in three parts (split_gemm.h):
//  k_mlp_hidden  Hh for all n*B rows, bias + ReLU in the epilogue.
//  k_mlp_head    per (worker, slab of rows): logits from Hh and W2 held in
//                registers (thread = hidden unit), LDS reduction, softmax in
//                wave 0, then dA as fragments of the next product and the
//                slab partials of db1 | dW2 | db2.
//  k_mlp_dw1     per worker: dW1 = X_i^T dA_i, K = B; extra blocks sum the head's
//                slab partials into G[i][d*H ...] (fixed order) and the loss.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "dbw_buffer.h"
#include "dbw_internal.h"
#include "split_gemm.h"

namespace dbw {
namespace {

constexpr int WAVE = 64;
constexpr int NXCD = 8;
constexpr int DW1_ROWS = 1024;   // row offsets staged in LDS at a time

__device__ __forceinline__ int64_t mlp_row(const MlpArgs& a, int64_t m, bool report) {
  if (!a.rows) return m;
  const int64_t r = a.rows[m];
  if (r < 0 || r >= a.S) {
    if (report) atomicOr(a.err, ERR_ROW_RANGE);
    return 0;
  }
  return r;
}

__device__ __forceinline__ int64_t mlp_row(const MlpArgs& a, int i, int b, bool report) {
  return mlp_row(a, (int64_t)i * a.B + b, report);
}

// A label loaded by the caller, range-checked (bad labels are reported and
// read as class 0).
__device__ __forceinline__ int checked_label(const MlpArgs& a, int lab) {
  if (lab < 0 || lab >= a.C) {
    atomicOr(a.err, ERR_LABEL_RANGE);
    return 0;
  }
  return lab;
}

// ---------------------------------------------------------------------------
// Hh[m][h] = relu(sum_j X[row(m)][j] W1[j][h] + b1[h]), m < n*B, on MT x NT tiles
// of 16 x 16 per wave (split_gemm.h); blockIdx.x = NW MT row tiles, y = NT
// column tiles.  KS: the block's waves share MT row tiles, split K and read W1
// itself; else W1 comes as fragments (`tiles` column tiles).  4096 x 3072 x
// 1024: 135 us, 1.15 PFLOP/s of issued bf16 products (fp32 matrix cores 230
// us); 2048 x 784 x 512: 18 us, of which 8 are there with one slice of K
// (launch, first loads, stores).
template <int MT, int NT, int NW, int OCC, bool KS, bool TINY = false>
__global__ __launch_bounds__(64 * NW, OCC) void k_mlp_hidden(MlpArgs a, int tiles) {
  __shared__ std::conditional_t<KS, SgRed<MT, NT, NW>, SgLds<NT, NW>> L;
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, c = lane & 15;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int Mrows = a.n * a.B;   // below 2^30
  const int d = a.d, H = a.H;
  const int64_t xrows = a.rows ? a.S : Mrows;
  const __amdgpu_buffer_rsrc_t xs = make_rsrc(a.X, static_cast<uint32_t>(xrows * d * 4));
  const int m0 = (KS ? static_cast<int>(blockIdx.x) : static_cast<int>(blockIdx.x) * NW + wv) * MT * 16;
  const int nt0 = static_cast<int>(blockIdx.y) * NT;
  SgRows<MT, TINY> X(xs, d);
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    const int m = m0 + 16 * t + c;
    X.roff[t] = kOutOfRange;
    if (m < Mrows) {
      const bool report = blockIdx.y == 0 && g == 0 && (!KS || wv == 0);
      const int64_t row = mlp_row(a, m, report);
      X.roff[t] = static_cast<uint32_t>(row * d * 4) + 32 * g;
    }
  }
  const float* b1 = a.w + (int64_t)d * H;
  float bias[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int h = (nt0 + nt) * 16 + c;
    bias[nt] = h < H ? b1[h] : 0.f;
  }
  sg_f32x4 acc[NT][MT];
  sg_zero<MT, NT>(acc);
  {
    auto prep = [&](int kb, float (&x)[MT][8]) { X.prep(kb, x); };
    const __amdgpu_buffer_rsrc_t ws = make_rsrc(a.w, static_cast<uint32_t>((int64_t)d * H * 4));
    if constexpr (KS)
      sg_loop_k<true, MT, NT, NW>(L, 0, X.slices(), X, prep, SgMatrix<NT>(ws, H, nt0 * 16), acc);
    else
      sg_loop<true, MT, NT, NW, 2>(L, 0, X.slices(), X, prep, [&](int kb) { return a.Wp + sg_frag(kb, tiles, nt0, 0) * 64; }, acc);
  }
  if (KS && wv > 0) return;
  sg_redo<MT, NT>(
      acc, d,
      [&](int t, int k) {
        const int m = m0 + 16 * t + c;
        const float v = a.X[mlp_row(a, min(m, Mrows - 1), false) * d + k];
        return m < Mrows ? v : 0.f;
      },
      [&](int nt, int k) {
        const int h = (nt0 + nt) * 16 + c;
        const float v = a.w[(int64_t)k * H + min(h, H - 1)];
        return h < H ? v : 0.f;
      });
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int h = (nt0 + nt) * 16 + c;
    if (h >= H) continue;
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + 16 * t + 4 * g + r;
        if (m < Mrows) a.Hh[(int64_t)m * H + h] = fmaxf(acc[nt][t][r] + bias[nt], 0.f);
      }
  }
}

// G[i][d*H + e] = sum_q Gp[i][q][e] for e < len (fixed slab order) and the
// loss of worker i: the head's slab partials, summed by the extra grid row of
// the dW1 kernels (part `part` of `nparts` blocks of 256 threads), which run
// beside the X^T dA tiles and write a disjoint part of G.
__device__ __forceinline__ void mlp_tail_sum(const MlpArgs& a, int slabs, int64_t len, int i, int part, int nparts) {
  const int64_t P = a.ldG ? a.ldG : (int64_t)a.d * a.H + len;   // row stride of G
  const bool keep = !a.row_mask || a.row_mask[i];
  for (int64_t e = (int64_t)part * 256 + threadIdx.x; e < len; e += (int64_t)nparts * 256) {
    const float* src = a.Gp + (int64_t)i * slabs * len + e;
    float s = 0.f;
    for (int q0 = 0; q0 < slabs; q0 += 8) {
      // eight slabs' loads in flight, then added in slab order
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = q0 + u < slabs ? src[(int64_t)(q0 + u) * len] : 0.f;
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (q0 + u < slabs) s += v[u];
    }
    if (keep) a.G[(int64_t)i * P + (int64_t)a.d * a.H + e] = s;
  }
  if (part == 0 && threadIdx.x == 0) {
    float s = 0.f;
    for (int q = 0; q < slabs; ++q) s += a.lossp[(int64_t)i * slabs + q];
    a.loss[i] = s / static_cast<float>(a.B);
  }
}

// dW1[j][h] = sum_b X[row(i,b)][j] dA_i[b][h] on MT x NT tiles per wave (lane
// (g, c) loads MT consecutive features of eight rows), dA as fragments from the
// head.  A linear grid, a worker's blocks on one XCD (its fragments of dA meet
// in one L2), the column chunks of one feature block neighbours; the last
// n * parts blocks sum the head's slab partials.
template <int MT, int NT, int NW, int OCC>
__global__ __launch_bounds__(64 * NW, OCC) void k_mlp_dw1(MlpArgs a, int slabs, int64_t tail, int tiles, int kblocks,
                                                         int fblocks, int chunks, int64_t per_xcd, int parts) {
  static_assert(NW == 4, "the tail sum takes blocks of 256 threads");
  if (blockIdx.x >= per_xcd * NXCD) {
    const int q = static_cast<int>(blockIdx.x - per_xcd * NXCD);
    mlp_tail_sum(a, slabs, tail, q / parts, q % parts, parts);
    return;
  }
  __shared__ SgLds<NT, NW> L;
  __shared__ __attribute__((aligned(16))) uint32_t srow[DW1_ROWS];
  const int64_t logical = (int64_t)(blockIdx.x % NXCD) * per_xcd + blockIdx.x / NXCD;
  if (logical >= (int64_t)a.n * fblocks * chunks) return;
  const int i = static_cast<int>(logical / (fblocks * chunks));
  const int rem = static_cast<int>(logical % (fblocks * chunks));
  const int fb = rem / chunks, nt0 = rem % chunks * NT;
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, c = lane & 15;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int d = a.d, H = a.H, B = a.B;
  const int64_t P = a.ldG ? a.ldG : (int64_t)d * H + tail;   // row stride of G
  const int64_t xrows = a.rows ? a.S : (int64_t)a.n * B;
  const __amdgpu_buffer_rsrc_t xs = make_rsrc(a.X, static_cast<uint32_t>(xrows * d * 4));
  const sg_u32x4* dp = a.Dp + (int64_t)i * kblocks * tiles * 192;
  const int f0 = (fb * NW + wv) * 16 * MT;
  uint32_t foff;
  int shift;
  sg_feature<MT>(f0 + MT * c, d, foff, shift);
  const bool edge = f0 + 16 * MT > d;
  sg_f32x4 acc[NT][MT];
  sg_zero<MT, NT>(acc);
  for (int c0 = 0; c0 < B; c0 += DW1_ROWS) {
    const int nr = min(B - c0, DW1_ROWS), nb = (nr + SG_K - 1) / SG_K;
    __syncthreads();
    for (int b = tid; b < nb * SG_K; b += 64 * NW)
      srow[b] = b < nr ? static_cast<uint32_t>(mlp_row(a, i, c0 + b, false) * d * 4) : kOutOfRange;
    __syncthreads();
    sg_loop<MT == 1, MT, NT, NW, 1>(
        L, c0 / SG_K, c0 / SG_K + nb,
        [&](int kb, float (&x)[MT][8], uint32_t dead = 0) { sg_load_cols<MT>(xs, srow + (kb * SG_K - c0) + 8 * g, foff, x, dead); },
        [&](int, float (&x)[MT][8]) { sg_shift<MT>(shift, edge, x); },
        [&](int kb) { return dp + sg_frag(kb, tiles, nt0, 0) * 64; }, acc);
  }
  sg_redo<MT, NT>(
      acc, B,
      [&](int t, int b) {
        const int j = f0 + MT * c + t;
        const float v = a.X[mlp_row(a, i, b, false) * d + min(j, d - 1)];
        return j < d ? v : 0.f;
      },
      [&](int nt, int b) { return sg_unpack(dp, tiles, b, (nt0 + nt) * 16 + c); });
  // the G rows of workers outside the row mask are computed but not stored
  if (a.row_mask && !a.row_mask[i]) return;
  float* Gi = a.G + (int64_t)i * P;
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const int j = f0 + MT * (4 * g + r) + t;
      if (j >= d) continue;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const int h = (nt0 + nt) * 16 + c;
        if (h < H) Gi[(int64_t)j * H + h] = acc[nt][t][r];
      }
    }
}

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}

// Max / sum over the 16 lanes of a DPP row: butterflies (xor 1, xor 2, half
// mirror, mirror) that leave the identical value in every lane of the row.
__device__ __forceinline__ float row16_max(float v) {
  v = fmaxf(v, dpp<0xB1>(v));
  v = fmaxf(v, dpp<0x4E>(v));
  v = fmaxf(v, dpp<0x141>(v));
  return fmaxf(v, dpp<0x140>(v));
}
__device__ __forceinline__ float row16_sum(float v) {
  v += dpp<0xB1>(v);
  v += dpp<0x4E>(v);
  v += dpp<0x141>(v);
  return v + dpp<0x140>(v);
}

// ---------------------------------------------------------------------------
// Head: thread j < H owns hidden unit j (T == H rounded up to a wave multiple
// is handled by the plan: T threads cover H with M units each).
template <int CP, int M, int T>
__global__ __launch_bounds__(T) void k_mlp_head(MlpArgs a, int slabs, int rps, int64_t L, int tiles, int kblocks) {
  constexpr int R = 4;
  constexpr int V = R * CP;
  constexpr int G = T / V;
  static_assert(G >= 1 && CP <= 16, "head layout");
  __shared__ float red[T][V + 1];
  __shared__ float red2[G][V];
  __shared__ float rr[V];
  __shared__ float sh_loss[R];
  __shared__ float sh_db2[R][CP];
  __shared__ int sh_lab[1024];
  const int i = blockIdx.x / slabs, q = blockIdx.x % slabs;
  const int tid = threadIdx.x;
  const int H = a.H, C = a.C, d = a.d;
  const int b0 = q * rps, b1 = min(a.B, b0 + rps), nrows = b1 - b0;
  // Nothing waits on the row indices but the labels, and nothing on the
  // labels until the first softmax: the indices are loaded first, then the
  // first rows and W2, then the labels, which are checked and staged in LDS
  // before the first step's first barrier.
  constexpr int LPT = (1024 + T - 1) / T;   // slab rows per thread
  int64_t rowv[LPT];
#pragma unroll
  for (int k = 0; k < LPT; ++k) {
    const int r = tid + k * T;
    rowv[k] = r < nrows ? mlp_row(a, i, b0 + r, false) : 0;
  }
  const int64_t hrow0 = (int64_t)i * a.B;
  // rows cb .. cb + R - 1.  The next rows are loaded one step ahead, so their
  // latency overlaps a step's reductions.
  auto load_rows = [&](int cb, float (&h1)[R][M]) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const bool ok = cb + r < nrows;
      const int64_t hoff = (hrow0 + b0 + (ok ? cb + r : 0)) * H;
      const __amdgpu_buffer_rsrc_t hs = make_rsrc(a.Hh + hoff, ok ? static_cast<uint32_t>(H * 4) : 0u);
#pragma unroll
      for (int m = 0; m < M; ++m) h1[r][m] = buf_f32(hs, static_cast<uint32_t>((tid + m * T) * 4));
    }
  };
  float h1[R][M];
  load_rows(0, h1);
  const float* W2 = a.w + (int64_t)d * H + H;
  const float* bias2 = W2 + (int64_t)H * C;
  const __amdgpu_buffer_rsrc_t w2s = make_rsrc(W2, static_cast<uint32_t>((int64_t)H * C * 4));
  float wr[M][CP], gw2[M][CP], gb1[M];
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const int j = tid + m * T;
    gb1[m] = 0.f;
#pragma unroll
    for (int c = 0; c < CP; ++c) {
      wr[m][c] = buf_f32(w2s, c < C ? static_cast<uint32_t>((j * C + c) * 4) : kOutOfRange);
      gw2[m][c] = 0.f;
    }
  }
  float loss_acc = 0.f, db2_acc = 0.f;
  sg_u32x2 first[M][3];   // parts of dA's rows 0 .. 3 of a group of eight
  sg_u32x4* dp = a.Dp + (int64_t)i * kblocks * tiles * 192;
  const float invB = 1.0f / static_cast<float>(a.B);
  int labv[LPT];
#pragma unroll
  for (int k = 0; k < LPT; ++k) labv[k] = tid + k * T < nrows ? a.y[rowv[k]] : 0;
  for (int cb = 0; cb < nrows; cb += R) {
    float x[R][M];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int m = 0; m < M; ++m) x[r][m] = h1[r][m];
    if (cb + R < nrows) load_rows(cb + R, h1);
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int c = 0; c < CP; ++c) {
        float z = 0.f;
#pragma unroll
        for (int m = 0; m < M; ++m) z = fmaf(x[r][m], wr[m][c], z);
        red[tid][r * CP + c] = z;
      }
    if (cb == 0) {
#pragma unroll
      for (int k = 0; k < LPT; ++k)
        if (tid + k * T < nrows) sh_lab[tid + k * T] = checked_label(a, labv[k]);
    }
    __syncthreads();
    if (tid < V * G) {
      // four interleaved partial sums keep four LDS reads in flight
      const int v = tid % V, g = tid / V;
      float s4[4] = {0.f, 0.f, 0.f, 0.f};
      int t = g;
      for (; t + 3 * G < T; t += 4 * G) {
#pragma unroll
        for (int u = 0; u < 4; ++u) s4[u] += red[t + u * G][v];
      }
#pragma unroll
      for (int u = 0; u < 3; ++u)
        if (t + u * G < T) s4[u] += red[t + u * G][v];
      red2[g][v] = (s4[0] + s4[1]) + (s4[2] + s4[3]);
    }
    __syncthreads();
    if (tid < WAVE) {
      const int r = tid / 16, c = tid % 16;
      const int rb = cb + r;
      float z = 0.f;
      if (c < CP) {
#pragma unroll
        for (int g = 0; g < G; ++g) z += red2[g][r * CP + c];
      }
      const bool valid = c < C;
      if (valid) z += bias2[c];
      const float zmax = row16_max(valid ? z : -INFINITY);
      const float sh = z - zmax;
      const float e = valid ? expf(sh) : 0.f;
      const float se = row16_sum(e);
      const bool row_ok = rb < nrows;
      const int lab = row_ok ? sh_lab[rb] : 0;
      const float zy = __shfl(sh, r * 16 + lab, WAVE);
      const float res = row_ok ? (e / se - (c == lab ? 1.f : 0.f)) * invB : 0.f;
      if (c < CP) rr[r * CP + c] = res;
      db2_acc += (c < C) ? res : 0.f;
      if (c == 0 && row_ok) loss_acc += logf(se) - zy;
    }
    __syncthreads();
    float da[M][R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      float rv[CP];
#pragma unroll
      for (int c = 0; c < CP; ++c) rv[c] = rr[r * CP + c];
      const bool ok = cb + r < nrows;
#pragma unroll
      for (int m = 0; m < M; ++m) {
        const int j = tid + m * T;
        float dh = 0.f;
#pragma unroll
        for (int c = 0; c < CP; ++c) {
          dh = fmaf(rv[c], wr[m][c], dh);
          gw2[m][c] = fmaf(x[r][m], rv[c], gw2[m][c]);
        }
        da[m][r] = ok && x[r][m] > 0.f ? dh : 0.f;
        gb1[m] += da[m][r];
        if (a.dA && ok && j < H) a.dA[(hrow0 + b0 + cb + r) * H + j] = da[m][r];
      }
    }
    // the step's four rows of dA as fragments of the dW1 product (slabs start
    // at multiples of 4 rows; rows past B stay as they were created, zero): half
    // of a lane's 16 bytes, kept for the next step where that has the other half
    // (9 x 21 x 104-552-7 25.9 -> 24.0 us a call, 18 x 34 x 508-868-5 45.8 -> 44.3)
    const bool second = ((b0 + cb) >> 2 & 1) != 0;
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const int j = tid + m * T;
      const SgPair u = sg_split2_any(da[m][0], da[m][1]), v = sg_split2_any(da[m][2], da[m][3]);
      const sg_u32x2 part[3] = {{u.h, v.h}, {u.m, v.m}, {u.l, v.l}};
      if (!second && cb + R < nrows) {
#pragma unroll
        for (int p = 0; p < 3; ++p) first[m][p] = part[p];
      } else if (j < H) {
        sg_u32x4* frag = dp + sg_frag((b0 + cb) >> 5, tiles, j >> 4, 0) * 64 + 16 * (((b0 + cb) & 31) >> 3) + (j & 15);
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          if (second && cb > 0) frag[64 * p] = sg_u32x4{first[m][p].x, first[m][p].y, part[p].x, part[p].y};
          else reinterpret_cast<sg_u32x2*>(frag + 64 * p)[second ? 1 : 0] = part[p];
        }
      }
    }
  }
  if (tid < WAVE) {
    const int r = tid / 16, c = tid % 16;
    if (c == 0) sh_loss[r] = loss_acc;
    if (c < CP) sh_db2[r][c] = db2_acc;
  }
  __syncthreads();
  // slab partial, laid out like G's tail: [db1 (H) | dW2 (H x C) | db2 (C)],
  // assembled in the LDS of the reduction and written in 8-byte pieces (a
  // thread's C classes are C floats apart from the next thread's)
  static_assert(M * T + M * T * CP + CP <= T * (V + 1), "slab partial fits the reduction LDS");
  float* stage = &red[0][0];
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const int j = tid + m * T;
    if (j < H) {
      stage[j] = gb1[m];
#pragma unroll
      for (int c = 0; c < CP; ++c)
        if (c < C) stage[H + j * C + c] = gw2[m][c];
    }
  }
  if (tid < C) {
    float s = 0.f;
#pragma unroll
    for (int r = 0; r < R; ++r) s += sh_db2[r][tid];
    stage[H + H * C + tid] = s;
  }
  if (tid == 0) {
    float s = 0.f;
#pragma unroll
    for (int r = 0; r < R; ++r) s += sh_loss[r];
    a.lossp[(int64_t)i * slabs + q] = s;
  }
  __syncthreads();
  float* gp = a.Gp + ((int64_t)i * slabs + q) * L;
  const int len = static_cast<int>(L);
  if ((len & 1) == 0) {
    // L even: every slab's partial starts 8-byte aligned
    for (int k = tid; k < len / 2; k += T)
      reinterpret_cast<float2*>(gp)[k] = make_float2(stage[2 * k], stage[2 * k + 1]);
  } else {
    for (int k = tid; k < len; k += T) gp[k] = stage[k];
  }
}

template <int CP, int M, int T>
hipError_t launch_head(const MlpPlan& p, const MlpArgs& a, hipStream_t s) {
  hipLaunchKernelGGL((k_mlp_head<CP, M, T>), dim3(static_cast<unsigned>(a.n * p.slabs)), dim3(T), 0, s, a,
                     p.slabs, p.rows_per_slab, p.tail, p.tiles, (a.B + SG_K - 1) / SG_K);
  return hipGetLastError();
}

template <int NT>
hipError_t launch_dw1(const MlpPlan& p, const MlpArgs& a, hipStream_t s) {
  const int kblocks = (a.B + SG_K - 1) / SG_K, chunks = p.tiles / NT;
  const int parts = static_cast<int>(std::min<int64_t>(8, (p.tail + 1023) / 1024));
  auto go = [&](auto kernel, int feats) {
    const int fblocks = (a.d + feats - 1) / feats;
    const int64_t per_xcd = ((int64_t)a.n * fblocks * chunks + NXCD - 1) / NXCD;
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(per_xcd * NXCD + (int64_t)a.n * parts)), dim3(256), 0, s, a,
                       p.slabs, p.tail, p.tiles, kblocks, fblocks, chunks, per_xcd, parts);
  };
  const int64_t w16 = (int64_t)a.n * chunks * ((a.d + 15) / 16);
  // one feature a lane, or two (half the reads of dA) from 16384 tiles of 16
  // features on, with more than 7 slices of rows from 2048 on: 32 x 64 x 784 x 512
  // (6272 tiles) 19.5 / 21.9 us, 16 x 256 x 3072 x 1024 (24576) 135 / 119, 16 x 500 x 800 x
  // 500 (3200, 16 slices) 44.7 / 42.3; the whole call 18 x 495 x 440-492-7 (2016, 16)
  // 97 / 109
  if (a.d < 2 || w16 < 2048 || (w16 < 16384 && kblocks < 8)) go(k_mlp_dw1<1, NT, 4, 2>, 64);
  else go(k_mlp_dw1<2, NT, 4, 3>, 128);
  return hipGetLastError();
}

}  // namespace

MlpPlan mlp_plan(int n, int B, int d, int H, int C) {
  MlpPlan p;
  p.tail = (int64_t)H + (int64_t)H * C + C;
  p.cpad = C <= 4 ? 4 : C <= 10 ? 10 : C <= 16 ? 16 : 0;
  p.threads = H <= 256 ? 256 : 512;
  p.per_thread = (H + p.threads - 1) / p.threads;
  if (p.cpad == 0 || p.per_thread > 2 || (p.cpad == 16 && p.per_thread > 1)) return p;   // ok = 0
  int slabs = 256 / n;
  int max_slabs = B / 8;
  slabs = slabs < 1 ? 1 : slabs;
  max_slabs = max_slabs < 1 ? 1 : max_slabs;
  slabs = slabs > max_slabs ? max_slabs : slabs;
  p.rows_per_slab = (B + slabs - 1) / slabs;
  p.rows_per_slab = (p.rows_per_slab + 3) / 4 * 4;
  if (p.rows_per_slab > 1024) p.rows_per_slab = 1024;
  p.slabs = (B + p.rows_per_slab - 1) / p.rows_per_slab;
  // column tiles: of the hidden layer's W1 fragments, and of dA's (chunks of
  // equal width, up to 8 tiles; narrower ones where they would leave the chip
  // idle: 7 x 406 x 172-108-9, 77 tiles of 7 columns or 308 of 2: 41.8 / 31.2 us)
  const int need = (H + 15) / 16;
  int chunks = (need + 7) / 8;
  p.nt = (need + chunks - 1) / chunks;
  while (p.nt > 2 && (int64_t)n * chunks * ((d + 15) / 16) < 256) {
    p.nt = (p.nt + 1) / 2;
    chunks = (need + p.nt - 1) / p.nt;
  }
  p.tiles = p.nt * chunks;
  p.wtiles = (need + 7) / 8 * 8;
  p.w_bytes = sg_frag_bytes((d + SG_K - 1) / SG_K, p.wtiles);
  p.d_bytes = sg_frag_bytes((int64_t)n * ((B + SG_K - 1) / SG_K), p.tiles);
  p.ok = 1;
  return p;
}

hipError_t launch_mlp_grads(const MlpPlan& p, const MlpArgs& a, hipStream_t s) {
  if (!p.ok) return hipErrorNotSupported;
  const int64_t rt = ((int64_t)a.n * a.B + 15) / 16;
  const int ct = (a.H + 15) / 16;
  auto hidden = [&](auto kernel, int rows, int cols, int threads) {
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>((rt + rows - 1) / rows), (ct + cols - 1) / cols), dim3(threads), 0,
                       s, a, p.wtiles);
  };
  auto pack = [&]() {
    const int64_t tasks = (int64_t)((a.d + SG_K - 1) / SG_K) * p.wtiles;
    hipLaunchKernelGGL(k_sg_pack, dim3(static_cast<unsigned>((tasks + 3) / 4)), dim3(256), 0, s, a.w, (int64_t)a.H, int64_t{1}, a.d, a.H,
                       p.wtiles, a.Wp);
  };
  // Hidden layer by the number of row tiles times column chunks: with few, a
  // block's eight waves split K of one row tile and read W1 itself; then 32
  // columns a wave (512 blocks of 64 x 32 at 2048 x 512), from two blocks of 64
  // x 128 per CU on those.  us, K-split / 32 / 64 / 128 columns: 114 x 836 x 784
  // 11.8 / - / 20 / -; 2048 x 784 x 512 30.6 / 17.9 / 19.4 / 29.7; 8000 x 800 x
  // 500 - / 69 / 46 / 43; 4096 x 3072 x 1024 - / - / 149 / 136.
  if (a.d < 8) {
    pack();
    hidden(k_mlp_hidden<1, 4, 4, 2, false, true>, 4, 4, 256);
  } else if (rt * ((ct + 3) / 4) <= 512) {
    hidden(k_mlp_hidden<1, 4, 8, 2, true>, 1, 4, 512);
  } else if (rt * ((ct + 7) / 8) < 1024) {
    pack();
    hidden(k_mlp_hidden<1, 2, 4, 2, false>, 4, 2, 256);
  } else {
    pack();
    hidden(k_mlp_hidden<1, 8, 4, 2, false>, 4, 8, 256);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  switch (p.cpad * 100 + p.per_thread * 10 + (p.threads == 512)) {
    case 410: e = launch_head<4, 1, 256>(p, a, s); break;
    case 420: e = launch_head<4, 2, 256>(p, a, s); break;
    case 411: e = launch_head<4, 1, 512>(p, a, s); break;
    case 421: e = launch_head<4, 2, 512>(p, a, s); break;
    case 1010: e = launch_head<10, 1, 256>(p, a, s); break;
    case 1020: e = launch_head<10, 2, 256>(p, a, s); break;
    case 1011: e = launch_head<10, 1, 512>(p, a, s); break;
    case 1021: e = launch_head<10, 2, 512>(p, a, s); break;
    case 1610: e = launch_head<16, 1, 256>(p, a, s); break;
    case 1611: e = launch_head<16, 1, 512>(p, a, s); break;
    default: return hipErrorNotSupported;
  }
  if (e != hipSuccess) return e;
  switch (p.nt) {
    case 1: return launch_dw1<1>(p, a, s);
    case 2: return launch_dw1<2>(p, a, s);
    case 3: return launch_dw1<3>(p, a, s);
    case 4: return launch_dw1<4>(p, a, s);
    case 5: return launch_dw1<5>(p, a, s);
    case 6: return launch_dw1<6>(p, a, s);
    case 7: return launch_dw1<7>(p, a, s);
    case 8: return launch_dw1<8>(p, a, s);
  }
  return hipErrorNotSupported;
}

}  // namespace dbw
