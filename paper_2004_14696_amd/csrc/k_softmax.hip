// Worker minibatch gradients of softmax regression (Sect. 2, Eq. gradient), gfx950.
//
// For worker i with minibatch rows x_{i,b} (b < B) and labels y_{i,b}:
//   z_b = x_b W,  p_b = softmax(z_b),  r_b = (p_b - onehot(y_b)) / B
//   G_i = sum_b x_b^T r_b  (d x C, laid out like W)
//   loss_i = (1/B) sum_b (logsumexp(z_b) - z_{b,y_b})
//
// Two implementations:
//  * k_softmax_mfma -- small C (<= 16), large minibatches: one pass over X
//    (each wave keeps its slice of the features and of the gradient in
//    registers; rows stream through in chunks).  A worker's rows are split
//    over `slabs` blocks to fill the 256 CUs; a second kernel sums the slab
//    partials in a fixed order.
//  * GEMM path -- everything else: logits Z = X W, row softmax (residuals), then
//    a per-worker product G_i = X_i^T R_i, on the bf16 matrix cores with every
//    fp32 operand in three parts (split_gemm.h).
//
// Minibatch rows are read either from a materialised X [n][B][d] or by row
// index from a resident dataset; both read each sample once per pass.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "dbw_buffer.h"
#include "dbw_internal.h"
#include "split_gemm.h"

namespace dbw {
namespace {

constexpr int WAVE = 64;
constexpr int NXCD = 8;

// Row pointer and label of sample b of worker i; invalid indices are
// reported and replaced by 0 so that no access leaves the buffers.
__device__ __forceinline__ int64_t sample_row(const SoftmaxArgs& a, int i, int b, bool report) {
  const int64_t m = (int64_t)i * a.B + b;
  if (!a.rows) return m;
  const int64_t r = a.rows[m];
  if (r < 0 || r >= a.S) {
    if (report) atomicOr(a.err, ERR_ROW_RANGE);
    return 0;
  }
  return r;
}

__device__ __forceinline__ int sample_label(const SoftmaxArgs& a, int64_t row, bool report) {
  const int lab = a.y[row];
  if (lab < 0 || lab >= a.C) {
    if (report) atomicOr(a.err, ERR_LABEL_RANGE);
    return 0;
  }
  return lab;
}

// A label loaded by the caller, range-checked as in sample_label.
__device__ __forceinline__ int checked_label(const SoftmaxArgs& a, int lab) {
  if (lab < 0 || lab >= a.C) {
    atomicOr(a.err, ERR_LABEL_RANGE);
    return 0;
  }
  return lab;
}

// Block index -> logical (worker, slab) so that a worker's slabs run on the
// same XCD (dispatch places block b on XCD b % 8): their partials then meet
// in one L2.
__device__ __forceinline__ int64_t xcd_logical(int64_t b, int64_t per_xcd) {
  return (b % NXCD) * per_xcd + b / NXCD;
}

constexpr int FUSED_MAX_ROWS = 1024;   // rows of one slab staged in LDS

// ---------------------------------------------------------------------------
// The single pass over X (C <= 16, 4 <= d <= 3072).
//
// Eight waves split the feature dimension; wave w owns features
// w*64U + 64u + 4m + j (u < U, m < 16, j < 4).  Rows stream through in
// chunks of 8; lane (m, g) = (lane % 16, lane / 16) holds the float4
// X[row g + 4e][w*64U + 64u + 4m .. +3] for e = 0, 1 -- exactly the A
// operand of a 16x16x4 MFMA whose k index runs over rows and whose m index
// runs over 16 features.  So the gradient G_i += X^T R (contraction over
// rows) is a chain of MFMAs on the loaded registers, accumulated in 16U
// tiles of 16 features x 16 classes.  The logits (contraction over
// features, which sit on lane % 16) are computed on the vector ALUs: each
// lane dots its 4U features of a row with W (staged once per block in LDS,
// in lane order), a 16-lane DPP reduction sums the row group, and the eight
// waves' partials meet in LDS.  After one block barrier every wave sums the
// partials of the rows its lanes hold and runs their softmax (16-lane DPP
// max and sum), so lane (m, g) forms r[row g + 4e][class m] itself -- the
// B operand of the same MFMAs.  One block barrier per chunk.
//
// RAG (d % 4 != 0): rows start at any 4-byte boundary, which the loads allow; the
// lane whose four features pass the row's end loads the row's last four and
// shifts them down before they are used, zeros behind.  The last P % 4 values
// of W and of G go one by one.
constexpr int MF_WAVES = 8;
constexpr int MF_T = MF_WAVES * WAVE;
constexpr int MF_ROWS = 8;
static_assert(MF_ROWS == 8, "lane (m, g) holds rows g and g + 4 of a chunk");

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}

// Sum / max over the 16 lanes of a DPP row; butterfly pairs (xor 1, xor 2,
// half-mirror, mirror) leave the identical value in all 16 lanes.
__device__ __forceinline__ float row16_sum(float v) {
  v += dpp<0xB1>(v);
  v += dpp<0x4E>(v);
  v += dpp<0x141>(v);
  v += dpp<0x140>(v);
  return v;
}
__device__ __forceinline__ float row16_max(float v) {
  v = fmaxf(v, dpp<0xB1>(v));
  v = fmaxf(v, dpp<0x4E>(v));
  v = fmaxf(v, dpp<0x141>(v));
  v = fmaxf(v, dpp<0x140>(v));
  return v;
}

__device__ __forceinline__ float f4_at(const float4& v, int j) {
  return j == 0 ? v.x : j == 1 ? v.y : j == 2 ? v.z : v.w;
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int U, int CW, bool RAG>
__global__ __launch_bounds__(MF_T) void k_softmax_mfma(SoftmaxArgs a, int slabs, int rps, int64_t per_xcd) {
  static_assert(CW % 2 == 0 && CW <= 16, "class padding");
  // W in lane order: lane (w, m) reads its 4U features x CW classes from one
  // contiguous run (features w 64U + 64u + 4m + j at (4u + j) CW); with the
  // run length SL = 4 U CW + 2 floats, SL / 2 is odd, so the 16 distinct
  // 8-byte reads of a row group fall on distinct bank pairs of the 32 banks
  // (runs start 8-byte aligned, so W is staged with 8-byte stores).  The same
  // LDS later assembles the block's slice of G ([d][C]).
  constexpr int SL = 4 * U * CW + 2;
  constexpr int WS = MF_WAVES * 16 * SL;
  __shared__ __attribute__((aligned(16))) float Ws[WS];
  __shared__ __attribute__((aligned(16))) float zb[2][MF_WAVES][MF_ROWS][16];  // per-wave partial logits
  __shared__ int sh_row[FUSED_MAX_ROWS];
  __shared__ int sh_lab[FUSED_MAX_ROWS];

  const int64_t logical = xcd_logical(blockIdx.x, per_xcd);
  if (logical >= (int64_t)a.n * slabs) return;
  const int i = static_cast<int>(logical / slabs);
  const int q = static_cast<int>(logical % slabs);
  const int tid = threadIdx.x;
  const int lane = tid & (WAVE - 1), w = tid >> 6;
  const int m = lane & 15, g = lane >> 4;
  const int d = a.d, C = a.C;
  const int64_t P = (int64_t)d * C;
  const int b0 = q * rps;
  const int nrows = min(a.B, b0 + rps) - b0;

  // The chain to the first products is the row indices, then the rows: the
  // indices are loaded first, then W (coalesced float4 pieces), then the
  // labels, which are checked and staged only after the first rows are on
  // their way (the wait for a load also waits
  // for every load issued before it, so the labels go out before the rows).
  constexpr int RPT = FUSED_MAX_ROWS / MF_T;   // slab rows per thread
  int64_t rowv[RPT];
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    const int r = tid + k * MF_T;
    rowv[k] = r < nrows ? sample_row(a, i, b0 + r, true) : 0;
  }
  const int n4 = static_cast<int>(P / 4);
  constexpr int KMAX = (MF_T * U * CW / 4 + MF_T - 1) / MF_T;   // P <= 512 U CW
  float4 wl[KMAX];
  {
    const __amdgpu_buffer_rsrc_t wrs = make_rsrc(a.W, static_cast<uint32_t>(P * 4));
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
      const int e4 = tid + k * MF_T;
      wl[k] = buf_f32x4(wrs, e4 < n4 ? static_cast<uint32_t>(e4 * 16) : kOutOfRange);
    }
  }
  const float wrest = RAG && tid < static_cast<int>(P & 3) ? a.W[4 * (int64_t)n4 + tid] : 0.f;
  float4* w4 = reinterpret_cast<float4*>(Ws);
  if (d < MF_T * U) {
    // slots of features past d must read as 0 (their rows carry finite values
    // of the same row)
    for (int k = tid; k < WS / 4; k += MF_T) w4[k] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  int labv[RPT];
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    const int r = tid + k * MF_T;
    labv[k] = 0;
    if (r < nrows) {
      sh_row[r] = static_cast<int>(rowv[k]);
      labv[k] = a.y[rowv[k]];
    }
  }
  __syncthreads();

  const int64_t xrows = a.rows ? a.S : (int64_t)a.n * a.B;
  const __amdgpu_buffer_rsrc_t xr = make_rsrc(a.X, static_cast<uint32_t>(xrows * d * 4));
  const int fbase = w * 64 * U + 4 * m;
  // byte offset of row cb + g + 4e of the slab, or kOutOfRange past the slab
  auto row_off = [&](int cb, int e) -> uint32_t {
    const int r = cb + g + 4 * e;
    const int rc = r < nrows ? r : 0;
    const int64_t row = a.rows ? (int64_t)sh_row[rc] : (int64_t)i * a.B + b0 + rc;
    return r < nrows ? static_cast<uint32_t>(row * d * 4) : kOutOfRange;
  };
  // this lane's float4 of group u of a row.  A group past d reads features
  // 0..3 of the same row instead: its W entries are 0 and its gradient rows
  // are never stored, so only the row's own values enter (no bounds select
  // per load; kOutOfRange + 12 KiB stays out of range).
  auto load_u = [&](uint32_t roff, int u) -> float4 {
    const int f = fbase + 64 * u;
    if (RAG) return buf_f32x4(xr, roff + (f + 4 <= d ? static_cast<uint32_t>(f * 4) : f < d ? static_cast<uint32_t>((d - 4) * 4) : 0u));
    return buf_f32x4(xr, roff + (f < d ? static_cast<uint32_t>(f * 4) : 0u));
  };
  // the row's end in its place (only the wave and group that hold it)
  auto ragged = [&](float4 (&x)[2][U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int g0 = __builtin_amdgcn_readfirstlane(w) * 64 * U + 64 * u;
      if (g0 >= d || g0 + 64 < d) continue;
      const int f = fbase + 64 * u, sh = f < d ? max(0, f + 4 - d) : 0;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const float4 v = x[e][u];
        x[e][u] = make_float4(sh == 0 ? v.x : sh == 1 ? v.y : sh == 2 ? v.z : v.w, sh == 0 ? v.y : sh == 1 ? v.z : sh == 2 ? v.w : 0.f,
                              sh == 0 ? v.z : sh == 1 ? v.w : 0.f, sh == 0 ? v.w : 0.f);
      }
    }
  };
  float4 xa[2][U], xb[2][U];   // two chunks in flight, roles alternate
  {
    const uint32_t r0 = row_off(0, 0), r1 = row_off(0, 1);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      xa[0][u] = load_u(r0, u);
      xa[1][u] = load_u(r1, u);
    }
  }
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    const int r = tid + k * MF_T;
    if (r < nrows) sh_lab[r] = checked_label(a, labv[k]);
  }

  // Stage W.  Features 4h .. 4h+3 (group h = w' 16U + 16u + m') are 4C
  // contiguous elements of W and 4CW contiguous floats of run (w', m') at
  // 4u CW, so with C == CW a float4 of W lands as two float2 stores.
  {
    // float index in Ws of element r of group h's 4CW floats
    auto slot = [](int h, int r) { return ((h / (16 * U)) * 16 + h % 16) * SL + ((h % (16 * U)) / 16) * 4 * CW + r; };
    if (C == CW) {
#pragma unroll
      for (int k = 0; k < KMAX; ++k) {
        const int e = 4 * (tid + k * MF_T);
        if (e < 4 * n4) {
          float2* w2 = reinterpret_cast<float2*>(Ws) + slot(e / (4 * CW), e % (4 * CW)) / 2;
          w2[0] = make_float2(wl[k].x, wl[k].y);
          w2[1] = make_float2(wl[k].z, wl[k].w);
        }
      }
    } else {
#pragma unroll
      for (int k = 0; k < KMAX; ++k) {
        const int e4 = tid + k * MF_T;
        if (e4 < n4) {
          int f = (4 * e4) / C, c = 4 * e4 - f * C;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            Ws[slot(f / 4, (f % 4) * CW + c)] = f4_at(wl[k], q);
            if (++c == C) {
              c = 0;
              ++f;
            }
          }
        }
      }
    }
    if (RAG && tid < static_cast<int>(P & 3)) {
      const int e = 4 * n4 + tid, f = e / C;
      Ws[slot(f / 4, (f % 4) * CW + e - f * C)] = wrest;
    }
  }
  __syncthreads();

  f32x4 acc[U][4];
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[u][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  float loss_acc = 0.f;
  const float invB = 1.0f / static_cast<float>(a.B);
  const bool cls_ok = m < C;
  const int nch = (nrows + MF_ROWS - 1) / MF_ROWS;
  float rv[2];   // residuals of the chunk whose MFMAs run next

  // Partial logits of rows g, g + 4 over this lane's 4U features.  wl0 is
  // this lane's W run.  The W reads run one feature ahead of the FMAs, and
  // the empty asm statements pin every step in place: left alone, the
  // compiler would hoist all 4U x CW reads to the front and hold them in
  // registers that the row buffers need.
  auto logits = [&](const float4 (&x)[2][U], float (&z)[2][CW], const float* wl0) {
    float wc[CW], wn[CW];
    auto read_w = [&](int t, float (&wv)[CW]) {
      const float2* wp = reinterpret_cast<const float2*>(wl0 + t * CW);
#pragma unroll
      for (int c2 = 0; c2 < CW / 2; ++c2) {
        const float2 v = wp[c2];
        wv[2 * c2] = v.x;
        wv[2 * c2 + 1] = v.y;
      }
    };
    read_w(0, wc);
#pragma unroll
    for (int t = 0; t < 4 * U; ++t) {
      if (t + 1 < 4 * U) read_w(t + 1, wn);
      const float x0 = f4_at(x[0][t / 4], t % 4), x1 = f4_at(x[1][t / 4], t % 4);
#pragma unroll
      for (int c = 0; c < CW; ++c) {
        z[0][c] = fmaf(x0, wc[c], z[0][c]);
        z[1][c] = fmaf(x1, wc[c], z[1][c]);
      }
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int c = 0; c < CW; ++c) asm volatile("" : "+v"(z[e][c]));
      asm volatile("" ::: "memory");
#pragma unroll
      for (int c = 0; c < CW; ++c) wc[c] = wn[c];
    }
  };
  // Sum the partial logits over the 16-lane row group; lane m == 0 stores
  // the wave's partials for the block (zb[buf]).
  auto reduce_logits = [&](float (&z)[2][CW], int buf) {
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int c = 0; c < CW; ++c) z[e][c] += dpp<0xB1>(z[e][c]);
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int c = 0; c < CW; ++c) z[e][c] += dpp<0x4E>(z[e][c]);
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int c = 0; c < CW; ++c) z[e][c] += dpp<0x141>(z[e][c]);
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int c = 0; c < CW; ++c) z[e][c] += dpp<0x140>(z[e][c]);
    if (m == 0) {
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        float2* zp = reinterpret_cast<float2*>(&zb[buf][w][g + 4 * e][0]);
#pragma unroll
        for (int c2 = 0; c2 < CW / 2; ++c2) zp[c2] = make_float2(z[e][2 * c2], z[e][2 * c2 + 1]);
      }
    }
  };
  // After the barrier: the softmax of the chunk's rows from the eight waves'
  // partials, residuals into rv, cross entropy into the label's lane.
  auto softmax = [&](int cb, int buf) {
    // lane (m, g): rows g and g + 4 of the chunk, class m.  Every wave forms
    // the residuals it needs from the eight waves' partials (the same
    // arithmetic in every wave), so no second barrier; wave 0 keeps the
    // cross entropy.
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int r = cb + g + 4 * e;
      const bool row_ok = r < nrows;
      float zt = 0.f;
#pragma unroll
      for (int v = 0; v < MF_WAVES; ++v) zt += zb[buf][v][g + 4 * e][m];
      const float mx = row16_max(cls_ok ? zt : -INFINITY);
      const float ex = cls_ok ? __expf(zt - mx) : 0.f;
      const float se = row16_sum(ex);
      const int lab = sh_lab[row_ok ? r : 0];
      const bool hit = row_ok && m == lab;
      const float p = ex * __builtin_amdgcn_rcpf(se);
      rv[e] = row_ok && cls_ok ? (p - (hit ? 1.f : 0.f)) * invB : 0.f;
      if (w == 0) loss_acc += hit ? __logf(se) - (zt - mx) : 0.f;
    }
  };
  // One chunk: logits of chunk cb (rows in A) while chunk cb + 8 streams
  // into B, the block-wide softmax, then G += X^T R on the matrix cores.
  auto step = [&](float4 (&A)[2][U], float4 (&B)[2][U], int cb) {
    float z[2][CW];
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int c = 0; c < CW; ++c) z[e][c] = 0.f;
    {
      const uint32_t rn = row_off(cb + MF_ROWS, 0);
#pragma unroll
      for (int u = 0; u < U; ++u) B[0][u] = load_u(rn, u);
    }
    if (RAG) ragged(A);
    logits(A, z, &Ws[(w * 16 + m) * SL]);
    const int buf = (cb / MF_ROWS) & 1;
    reduce_logits(z, buf);
    {
      // rows g + 4 of the next chunk once the logit registers are released
      const uint32_t rn = row_off(cb + MF_ROWS, 1);
#pragma unroll
      for (int u = 0; u < U; ++u) B[1][u] = load_u(rn, u);
    }
    __syncthreads();
    softmax(cb, buf);
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[u][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(f4_at(A[e][u], j), rv[e], acc[u][j], 0, 0, 0);
  };
  int c = 0;
  for (; c + 1 < nch; c += 2) {
    step(xa, xb, c * MF_ROWS);
    step(xb, xa, (c + 1) * MF_ROWS);
  }
  if (c < nch) step(xa, xb, c * MF_ROWS);

  // lane (m, g) holds tile rows 4g + t (features w 64U + 64u + 16g + 4t + j)
  // of class m.
  if (slabs > 1) {
    // slab partial in tile order: float4 (t = 0..3) of (w, u, j, g, m) at
    // ((((w U + u) 4 + j) 4 + g) C + m) 4; k_slab_reduce_tiles sums the slabs
    // and restores the [d][C] order
    if (cls_ok) {
      float4* part = reinterpret_cast<float4*>(a.Gp + ((int64_t)i * slabs + q) * (int64_t)(MF_T * U * C));
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          part[(((w * U + u) * 4 + j) * 4 + g) * C + m] = make_float4(acc[u][j][0], acc[u][j][1], acc[u][j][2], acc[u][j][3]);
    }
  } else {
    // the worker's G ([d][C], P contiguous floats) is assembled in the LDS
    // that held W and written out in float4 pieces
    __syncthreads();
    if (cls_ok) {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const int f = w * 64 * U + 64 * u + 16 * g + 4 * t + j;
            if (f < d) Ws[f * C + m] = acc[u][j][t];
          }
    }
    __syncthreads();
    const float4* s4 = reinterpret_cast<const float4*>(Ws);
    float4* o4 = reinterpret_cast<float4*>(a.G + (int64_t)i * P);
    if (a.row_mask && !a.row_mask[i]) {
    } else if (RAG) {
      for (int k = tid; k < static_cast<int>(P); k += MF_T) a.G[(int64_t)i * P + k] = Ws[k];
    } else {
      for (int k = tid; k < static_cast<int>(P / 4); k += MF_T) o4[k] = s4[k];
    }
  }
  if (w == 0) {
    // the loss of every row sits in its label's lane of wave 0
    float l = loss_acc;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) l += __shfl_xor(l, o);
    if (lane == 0) {
      if (slabs == 1) a.loss[i] = l * invB;
      else a.lossp[(int64_t)i * slabs + q] = l;
    }
  }
}

// Sum of the tile-order slab partials of the matrix-core kernel, in slab
// order.  Block (x, i): features 64x .. 64x + 63 of worker i, whose 64C
// partial floats of one slab are contiguous (wave w' = x / U, group
// u = x % U).  Summed float4 pieces are put back in [d][C] order through LDS.
__global__ __launch_bounds__(256) void k_slab_reduce_tiles(SoftmaxArgs a, int slabs, int U) {
  __shared__ __attribute__((aligned(16))) float tile[64 * 16];
  const int i = blockIdx.y, x = blockIdx.x;
  const int C = a.C, d = a.d;
  const int64_t P = (int64_t)d * C;
  const int64_t part = (int64_t)MF_T * U * C;
  const int n4 = 16 * C;   // float4 pieces of the 64 features
  for (int k = threadIdx.x; k < n4; k += 256) {
    // piece k = ((j 4 + g) C + m): features 16g + 4t + j (t = 0..3), class m
    const int m = k % C, jg = k / C, g = jg % 4, j = jg / 4;
    const float* src = a.Gp + (int64_t)i * slabs * part + (int64_t)x * 64 * C + 4 * k;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int q0 = 0; q0 < slabs; q0 += 8) {
      // up to eight slabs' pieces in flight, then added in slab order (a
      // plain loop over a run-time slab count waits for each load in turn)
      float4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        v[u] = q0 + u < slabs ? *reinterpret_cast<const float4*>(src + (q0 + u) * part) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (q0 + u < slabs) {
          s.x += v[u].x; s.y += v[u].y; s.z += v[u].z; s.w += v[u].w;
        }
    }
    tile[(16 * g + 0 + j) * C + m] = s.x;
    tile[(16 * g + 4 + j) * C + m] = s.y;
    tile[(16 * g + 8 + j) * C + m] = s.z;
    tile[(16 * g + 12 + j) * C + m] = s.w;
  }
  __syncthreads();
  const int f0 = x * 64;
  const int nf = min(64, d - f0);   // features past d are not stored
  float* dst = a.G + (int64_t)i * P + (int64_t)f0 * C;
  if (a.row_mask && !a.row_mask[i]) {
  } else if (P % 4 == 0) {
    for (int k = threadIdx.x; k < nf * C / 4; k += 256)
      reinterpret_cast<float4*>(dst)[k] = reinterpret_cast<const float4*>(tile)[k];
  } else {
    for (int k = threadIdx.x; k < nf * C; k += 256) dst[k] = tile[k];
  }
  if (x == 0 && threadIdx.x == 0) {
    float l = 0.f;
    for (int q = 0; q < slabs; ++q) l += a.lossp[(int64_t)i * slabs + q];
    a.loss[i] = l / static_cast<float>(a.B);
  }
}

// ---------------------------------------------------------------------------
// GEMM path (any C, d, B): products on the bf16 matrix cores in three parts
// (split_gemm.h).  W is packed into fragments, the logits kernel leaves the
// residuals as fragments of the second product (from its registers when a
// wave holds all classes of its rows, C <= 16 SG_NARROW; else through Z and
// k_rows_pack), and the gradient kernel forms G_i = X_i^T R_i.
//
// The rows of the logits product are padded per worker to whole tiles of 16
// (tpw tiles), so that a tile's residuals belong to one worker's fragments.

// The residuals (at most 1) are packed 2^32 times as large: all their bits down
// to the least float then fit the three parts; the gradient's sums are brought
// back at the end, exactly.
constexpr float kResidualScale = 0x1p32f;
constexpr int SG_DIRECT = 4;   // up to so many column tiles a K-split wave always reads W itself

// Z[m][c] = sum_j X[row(m)][j] W[j][c] on MT x NT tiles of 16 x 16 per wave;
// blockIdx.x = NW MT row tiles, blockIdx.y = NT column tiles.  NARROW: all
// classes are in the wave: softmax, residuals (p - onehot(y)) / B as
// fragments and the rows' cross entropy.  Otherwise Z is stored.  KS: the
// block's waves share MT row tiles and split K (sg_loop_k).  PER_ROW: the rows
// are those of the dataset (n = 1, B = S), the residuals stay as rows in Z and
// the cross entropy in ce_row; labels are not reported here (a row may be in no
// minibatch).  256 x 512 x 3072 x
// 100: 430 - 475 us (fp32 matrix-core form 629), 1.6 GB of X at 3.4 - 3.7 TB/s
// and 1.1 - 1.3 PFLOP/s of issued bf16 products, both near what the chip holds.
// DIRECT (KS): W itself, not its fragments.
template <int MT, int NT, int NW, int OCC, bool KS, bool NARROW, bool TINY = false,
          bool PER_ROW = false, bool DIRECT = (NT <= SG_DIRECT)>
__global__ __launch_bounds__(64 * NW, OCC) void k_sg_logits(SoftmaxArgs a, int tiles, int tpw) {
  __shared__ std::conditional_t<KS, SgRed<MT, NT, NW>, SgLds<NT, NW>> L;
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, c = lane & 15;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int d = a.d, C = a.C, B = a.B;
  const int64_t xrows = a.rows ? a.S : (int64_t)a.n * B;
  const __amdgpu_buffer_rsrc_t xs = make_rsrc(a.X, static_cast<uint32_t>(xrows * d * 4));
  const int t0 = (KS ? static_cast<int>(blockIdx.x) : static_cast<int>(blockIdx.x) * NW + wv) * MT;
  const int nt0 = static_cast<int>(blockIdx.y) * NT;
  const bool report = !PER_ROW && blockIdx.y == 0 && g == 0 && (!KS || wv == 0);
  SgRows<MT, TINY> X(xs, d);
  int lab[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    const int i = (t0 + t) / tpw, b = (t0 + t) % tpw * 16 + c;
    X.roff[t] = kOutOfRange;
    lab[t] = 0;
    if (i < a.n && b < B) {
      const int64_t row = sample_row(a, i, b, report);
      if (NARROW) lab[t] = a.y[row];   // checked where it is used
      X.roff[t] = static_cast<uint32_t>(row * d * 4) + 32 * g;
    }
  }
  sg_f32x4 acc[NT][MT];
  sg_zero<MT, NT>(acc);
  {
    auto prep = [&](int kb, float (&x)[MT][8]) { X.prep(kb, x); };
    auto frag = [&](int kb) { return a.Wp + sg_frag(kb, tiles, nt0, 0) * 64; };
    if constexpr (KS && DIRECT)
      sg_loop_k<true, MT, NT, NW>(L, 0, X.slices(), X, prep, SgMatrix<NT>(make_rsrc(a.W, static_cast<uint32_t>((int64_t)d * C * 4)), C, nt0 * 16), acc);
    else if constexpr (KS)
      sg_loop_k<true, MT, NT, NW>(L, 0, X.slices(), X, prep, SgFrags<NT>{frag(0), (int64_t)tiles * 192}, acc);
    else
      sg_loop<(MT == 1 && NT <= 4), MT, NT, NW, MT == 1 ? 2 : 1>(L, 0, X.slices(), X, prep, frag, acc);
  }
  if (KS && wv > 0) return;
  sg_redo<MT, NT>(
      acc, d,
      [&](int t, int k) {
        const int i = (t0 + t) / tpw, b = (t0 + t) % tpw * 16 + c;
        const bool ok = i < a.n && b < B;
        const float v = a.X[sample_row(a, ok ? i : 0, ok ? b : 0, false) * d + k];
        return ok ? v : 0.f;
      },
      [&](int nt, int k) {
        const int cc = (nt0 + nt) * 16 + c;
        const float v = a.W[(int64_t)k * C + min(cc, C - 1)];
        return cc < C ? v : 0.f;
      });

  if (NARROW) {
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      if (PER_ROW) lab[t] = lab[t] < 0 || lab[t] >= C ? 0 : lab[t];
      else lab[t] = checked_label(a, lab[t]);
    }
  }
  const float invB = 1.0f / static_cast<float>(PER_ROW ? a.B_mean : B);
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    const int i = (t0 + t) / tpw, bt = (t0 + t) % tpw;
    if (i >= a.n) break;
    const int b0 = bt * 16 + 4 * g;   // this lane's rows b0 .. b0 + 3
    if constexpr (!NARROW) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (b0 + r < B)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) {
            const int cc = (nt0 + nt) * 16 + c;
            if (cc < C) a.Z[((int64_t)i * B + b0 + r) * C + cc] = acc[nt][t][r];
          }
    } else {
      // the row's classes are the 16 lanes of a DPP row
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float mx = -INFINITY;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
          if (nt * 16 + c < C) mx = fmaxf(mx, acc[nt][t][r]);
        mx = row16_max(mx);
        float ex[NT];
        float se = 0.f;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          ex[nt] = nt * 16 + c < C ? expf(acc[nt][t][r] - mx) : 0.f;
          se += ex[nt];
        }
        se = row16_sum(se);
        const int lr = __shfl(lab[t], 4 * g + r);
        const bool ok = b0 + r < B;
        const float inv = 1.0f / se;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const int cc = nt * 16 + c;
          if (ok && cc == lr) (PER_ROW ? a.ce_row : a.ce)[(int64_t)i * B + b0 + r] = (logf(se) + mx) - acc[nt][t][r];
          acc[nt][t][r] = ok && cc < C ? (ex[nt] * inv - (cc == lr ? 1.f : 0.f)) * invB : 0.f;
        }
      }
      if constexpr (PER_ROW) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (b0 + r < B)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
              if (nt * 16 + c < C) a.Z[(int64_t)(b0 + r) * C + nt * 16 + c] = acc[nt][t][r];
        continue;
      }
      sg_u32x4* rp = a.Rp + (int64_t)i * ((tpw + 1) / 2) * tiles * 3 * 64;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const float v[4] = {acc[nt][t][0] * kResidualScale, acc[nt][t][1] * kResidualScale, acc[nt][t][2] * kResidualScale,
                            acc[nt][t][3] * kResidualScale};
        sg_store4(rp, tiles, b0, nt * 16 + c, v);   // (rows past the last tile stay as they were created, zero)
      }
    }
  }
}

// Residuals as fragments and ce[m] = CE from rows in Z: logits of the
// minibatches' rows (ZROWS_BATCH) or of the dataset's rows (ZROWS_DATASET: the
// row of sample m is its dataset row), of which the row softmax is taken here,
// or the dataset rows' residuals (ZROWS_RESIDUAL, with ce_row).  Block (x, i):
// rows 8 x .. 8 x + 7 of worker i (fragments past the B rows, up to whole slices
// of 32, stay as they were created, zero), held in LDS;
// every wave runs two rows' statistics and leaves their exponentials, then
// packs a quarter of the columns.
enum ZRows { ZROWS_BATCH, ZROWS_DATASET, ZROWS_RESIDUAL };
template <int FROM>
__global__ __launch_bounds__(256) void k_rows_pack(SoftmaxArgs a, int tiles, int kblocks) {
  extern __shared__ float zrow[];   // [8][C]
  __shared__ float sh_inv[8];
  __shared__ int sh_lab[8], sh_row[8];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int i = blockIdx.y, b0 = static_cast<int>(blockIdx.x) * 8;
  const int C = a.C, B = a.B;
  const int nr = min(8, B - b0), nz = nr * C;
  if (FROM != ZROWS_BATCH) {
    if (tid < nr) {
      const int64_t row = sample_row(a, i, b0 + tid, true);
      sh_row[tid] = static_cast<int>(row);
      (void)sample_label(a, row, true);
      if (FROM == ZROWS_RESIDUAL) a.ce[(int64_t)i * B + b0 + tid] = a.ce_row[row];
    }
    __syncthreads();
    // a wave copies two rows
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int r = 2 * wv + q;
      if (r >= nr) break;
      const float* z = a.Z + (int64_t)sh_row[r] * C;
      for (int c = lane; c < C; c += WAVE) zrow[r * C + c] = z[c];
    }
  } else {
    const float* z0 = a.Z + ((int64_t)i * B + b0) * C;
    for (int e0 = 0; e0 < nz; e0 += 8 * 256) {
      float v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = e0 + q * 256 + tid < nz ? z0[e0 + q * 256 + tid] : 0.f;
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (e0 + q * 256 + tid < nz) zrow[e0 + q * 256 + tid] = v[q];
    }
  }
  __syncthreads();
  if (FROM != ZROWS_RESIDUAL) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int r = 2 * wv + q;
      if (r >= nr) break;
      float* z = zrow + r * C;
      const int lab = sample_label(a, sample_row(a, i, b0 + r, false), FROM == ZROWS_BATCH && lane == 0);
      float mx = -INFINITY;
      for (int c = lane; c < C; c += WAVE) mx = fmaxf(mx, z[c]);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, WAVE));
      const float zy = z[lab];
      float se = 0.f;
      for (int c = lane; c < C; c += WAVE) {
        const float ex = expf(z[c] - mx);
        z[c] = ex;
        se += ex;
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) se += __shfl_xor(se, o, WAVE);
      if (lane == 0) {
        sh_inv[r] = 1.0f / se;
        sh_lab[r] = lab;
        a.ce[(int64_t)i * B + b0 + r] = (logf(se) + mx) - zy;
      }
    }
    __syncthreads();
  }
  const float invB = 1.0f / static_cast<float>(B);
  sg_u32x4* rp = a.Rp + (int64_t)i * kblocks * tiles * 3 * 64;
  for (int c = tid; c < tiles * 16; c += 256) {
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      v[e] = 0.f;
      if (e < nr && c < C)
        v[e] = FROM == ZROWS_RESIDUAL ? zrow[e * C + c]
                                      : (zrow[e * C + c] * sh_inv[e] - (c == sh_lab[e] ? 1.f : 0.f)) * invB;
      v[e] *= kResidualScale;
    }
    sg_store8(rp, tiles, b0, c, v);
  }
}

// G_i[j][c] = sum_b X[row(i,b)][j] R_i[b][c] on MT x NT tiles per wave: lane
// (g, c) loads MT consecutive features (one per tile) of eight rows, which is
// the A operand.  A linear grid, dealt so that a worker's blocks share an XCD
// (its residual fragments meet in one L2); within a worker the column chunks
// of one feature block are neighbours (its rows of X are read once from HBM).
// The first block of a worker also writes its loss.  Bound by the matrix cores'
// bf16 rate at the clock they sustain (about 1.1 PFLOP/s of issued products at
// 256 x 512 x 3072 x 100: 460 us; the fp32 matrix-core form took 651).
template <int MT, int NT, int NW, int OCC, bool KS>
__global__ __launch_bounds__(64 * NW, OCC) void k_sg_grads(SoftmaxArgs a, int tiles, int kblocks, int fblocks,
                                                          int chunks, int64_t per_xcd) {
  __shared__ std::conditional_t<KS, SgRed<MT, NT, NW>, SgLds<NT, NW>> L;
  __shared__ __attribute__((aligned(16))) uint32_t srow[FUSED_MAX_ROWS];
  __shared__ float sh[NW];
  const int64_t logical = xcd_logical(blockIdx.x, per_xcd);
  if (logical >= (int64_t)a.n * fblocks * chunks) return;
  const int i = static_cast<int>(logical / (fblocks * chunks));
  const int rem = static_cast<int>(logical % (fblocks * chunks));
  const int fb = rem / chunks, nt0 = rem % chunks * NT;
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, c = lane & 15;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int d = a.d, C = a.C, B = a.B;
  const int64_t xrows = a.rows ? a.S : (int64_t)a.n * B;
  const __amdgpu_buffer_rsrc_t xs = make_rsrc(a.X, static_cast<uint32_t>(xrows * d * 4));
  const sg_u32x4* rp = a.Rp + (int64_t)i * kblocks * tiles * 3 * 64;
  const int f0 = (KS ? fb : fb * NW + wv) * 16 * MT;
  uint32_t foff;
  int shift;
  sg_feature<MT>(f0 + MT * c, d, foff, shift);
  const bool edge = f0 + 16 * MT > d;
  sg_f32x4 acc[NT][MT];
  sg_zero<MT, NT>(acc);
  for (int c0 = 0; c0 < B; c0 += FUSED_MAX_ROWS) {
    const int nr = min(B - c0, FUSED_MAX_ROWS), nb = (nr + SG_K - 1) / SG_K;
    __syncthreads();
    for (int b = tid; b < nb * SG_K; b += 64 * NW)
      srow[b] = b < nr ? static_cast<uint32_t>(sample_row(a, i, c0 + b, false) * d * 4) : kOutOfRange;
    __syncthreads();
    auto load = [&](int kb, float (&x)[MT][8], uint32_t dead = 0) { sg_load_cols<MT>(xs, srow + (kb * SG_K - c0) + 8 * g, foff, x, dead); };
    auto prep = [&](int, float (&x)[MT][8]) { sg_shift<MT>(shift, edge, x); };
    auto frag = [&](int kb) { return rp + sg_frag(kb, tiles, nt0, 0) * 64; };
    if constexpr (KS)
      sg_loop_k<(NT < 8), MT, NT, NW>(L, c0 / SG_K, c0 / SG_K + nb, load, prep, SgFrags<NT>{frag(0), (int64_t)tiles * 192}, acc);
    else
      sg_loop<MT == 1, MT, NT, NW, MT == 1 ? 2 : 1>(L, c0 / SG_K, c0 / SG_K + nb, load, prep, frag, acc);
  }
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[nt][t] *= 1.f / kResidualScale;
  sg_redo<MT, NT>(
      acc, B,
      [&](int t, int b) {
        const int j = f0 + MT * c + t;
        const float v = a.X[sample_row(a, i, b, false) * d + min(j, d - 1)];
        return j < d ? v : 0.f;
      },
      [&](int nt, int b) { return sg_unpack(rp, tiles, b, (nt0 + nt) * 16 + c) * (1.f / kResidualScale); });
  // the G rows of workers outside the row mask are computed but not stored
  if ((!KS || wv == 0) && (!a.row_mask || a.row_mask[i])) {
    float* Gi = a.G + (int64_t)i * d * C;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        const int j = f0 + MT * (4 * g + r) + t;
        if (j >= d) continue;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const int cc = (nt0 + nt) * 16 + c;
          if (cc < C) Gi[(int64_t)j * C + cc] = acc[nt][t][r];
        }
      }
  }
  if (rem == 0) {
    // loss_i = mean CE over the worker's rows (fixed order)
    float s = 0.f;
    for (int b = tid; b < B; b += 64 * NW) s += a.ce[(int64_t)i * B + b];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (lane == 0) sh[wv] = s;
    __syncthreads();
    if (tid == 0) {
      float l = 0.f;
      for (int q = 0; q < NW; ++q) l += sh[q];
      a.loss[i] = l / static_cast<float>(B);
    }
  }
}

// Whether the logits run over the dataset's rows (see launch_split_nt).  Below
// 1.5 samples a row the gather costs what the shared rows save.  Below 8192
// rows (two row tiles a CU) it depends on the work: us of the launch, per
// sample / per row, 256 x 512 x 3072 x 100 of 4096 rows 897 / 563, 128 x 300 x 256 x 300 of
// 4000 123 / 90, but 64 x 256 x 784 x 40 of 4000 36.9 / 40.3, 32 x 128 x 500 x 60 of 1500
// 16.2 / 27.3; those stay with the samples.
bool split_per_row(int n, int B, int d, int64_t S) {
  return S >= 8192 && d >= 8 && 2 * (int64_t)n * B >= 3 * S;
}

template <int NT>
hipError_t launch_split_nt(const SoftmaxPlan& p, const SoftmaxArgs& a, hipStream_t s) {
  const int tiles = p.tiles, tpw = (a.B + 15) / 16, kblocks = (a.B + SG_K - 1) / SG_K;
  const int chunks = tiles / NT;
  // With (well) more samples than dataset rows, the logits, residuals and cross
  // entropy of every dataset row are computed once and gathered by the
  // minibatches (they depend on the row and w alone): 256 x 512 samples of a
  // 50000 x 3072 dataset, 100 classes, 470 us of logits -> 216 and 38 of gathering;
  // 100 x 300 of 20000 x 500, 60 classes, 65 -> 51 the launch.
  const bool per_row = split_per_row(a.n, a.B, a.d, a.rows ? a.S : 0);
  SoftmaxArgs al = a;   // the rows of the logits product
  if (per_row) {
    al.rows = nullptr;
    al.n = 1;
    al.B = static_cast<int>(a.S);
    al.B_mean = a.B;
  }
  const int ltpw = per_row ? (al.B + 15) / 16 : tpw;
  const int64_t rt = (int64_t)al.n * ltpw;
  auto logits = [&](auto kernel, int per, int threads) {
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>((rt + per - 1) / per), chunks), dim3(threads), 0, s, al, tiles, ltpw);
  };
  auto pack = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((a.B + 7) / 8, a.n), dim3(256), 8 * sizeof(float) * a.C, s, a, tiles, kblocks);
  };
  // Waves per SIMD of the large logits blocks: as many as leave no spills.
  constexpr int OC8 = NT >= 4 ? 2 : 4;
  // Logits by the number of row tiles times column chunks: with few, a block's
  // eight waves split K of one row tile (kSplitK); then one row tile a wave,
  // four waves a block; from two full rounds of the chip on (or one of wide
  // tiles), 16 row tiles a block, which reads its fragments half as often.  us
  // of the launch, the large / middle / K-split form: 256 x 512 x 3072 x 100
  // (8192 tiles) 934 / 1028 / 1641; its logits over 50000 dataset rows (3125
  // tiles of 7 columns) 216 / 289 / -; 20000 x 500 x 60 (1250) 28 / 17 / -; of the whole
  // launch, 160 x 256 x 3072 x 100 (2560 of 7) 389 / 395, 170 x 256 x 500 x 112 (2720 of
  // 7) 84 / 76, 128 x 256 x 1000 x 100 (2048 of 7) 121 / 95; 128 x
  // 512 x 256 x 50 (4096) 51 / 49 / 81; 64 x 256 x 3072 x 100 (1024) 250 / 163 /
  // 209; 32 x 200 x 1024 x 64 (416) 73 / 40 / 36; 16 x 100 x 785 x 20 (112)
  // 40 / 25 / 17.
  enum { kLarge, kMiddle, kSplitK, kTiny };
  const int lv = a.d < 8 ? kTiny : rt * chunks >= 8192 || rt * chunks * NT >= 20000 ? kLarge
                 : rt * chunks > 512 || per_row ? kMiddle : kSplitK;
  // Wide K-split waves read W itself while the rows are few (row tiles times
  // slices): the packing launch is saved, the loads and splits of W are more.  us,
  // fragments / W: 15 x 29 x 204 x 308 (210) 22.4 / 20.4, 8 x 17 x 752 x 309 (384) 28.3 / 26.9,
  // 6 x 155 x 460 x 796 (900) 49.1 / 56.5, 10 x 91 x 2208 x 720 (4140) 95 / 124.
  const bool direct = lv == kSplitK && (NT <= SG_DIRECT || rt * ((a.d + SG_K - 1) / SG_K) <= 400);
  if (!direct) {
    const int64_t wtasks = (int64_t)((a.d + SG_K - 1) / SG_K) * tiles;
    hipLaunchKernelGGL(k_sg_pack, dim3(static_cast<unsigned>((wtasks + 3) / 4)), dim3(256), 0, s, a.W, (int64_t)a.C, int64_t{1}, a.d,
                       a.C, tiles, a.Wp);
  }
  if (chunks == 1 && per_row) {
    if (lv == kLarge) logits(k_sg_logits<2, NT, 8, OC8, false, true, false, true>, 16, 512);
    else logits(k_sg_logits<1, NT, 4, 2, false, true, false, true>, 4, 256);
    pack(k_rows_pack<ZROWS_RESIDUAL>);
  } else if (chunks == 1) {
    if (lv == kLarge) logits(k_sg_logits<2, NT, 8, OC8, false, true>, 16, 512);
    else if (lv == kMiddle) logits(k_sg_logits<1, NT, 4, 2, false, true>, 4, 256);
    else if (lv == kTiny) logits(k_sg_logits<1, NT, 4, 2, false, true, true>, 4, 256);
    else if (direct) logits(k_sg_logits<1, NT, 8, 2, true, true, false, false, true>, 1, 512);
    else logits(k_sg_logits<1, NT, 8, 2, true, true>, 1, 512);
  } else {
    if (lv == kLarge) logits(k_sg_logits<2, NT, 8, OC8, false, false>, 16, 512);
    else if (lv == kMiddle) logits(k_sg_logits<1, NT, 4, 2, false, false>, 4, 256);
    else if (lv == kTiny) logits(k_sg_logits<1, NT, 4, 2, false, false, true>, 4, 256);
    else if (direct) logits(k_sg_logits<1, NT, 8, 2, true, false, false, false, true>, 1, 512);
    else logits(k_sg_logits<1, NT, 8, 2, true, false>, 1, 512);
    if (per_row) pack(k_rows_pack<ZROWS_DATASET>);
    else pack(k_rows_pack<ZROWS_BATCH>);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  auto grads = [&](auto kernel, int feats, int threads) {
    const int fblocks = (a.d + feats - 1) / feats;
    const int64_t per_xcd = ((int64_t)a.n * fblocks * chunks + NXCD - 1) / NXCD;
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(per_xcd * NXCD)), dim3(threads), 0, s, a, tiles, kblocks, fblocks,
                       chunks, per_xcd);
  };
  // Gradients by the number of 16-feature tiles over all workers: four features
  // a lane (and half the residual reads) from 32768 tiles on, two from 4096,
  // else one; with so few that the chip stays idle and many rows, the block's
  // waves split the rows.  us of the launch, 4 / 2 / 1 features / split: 256 x
  // 512 x 3072 x 100 (49152 tiles) 1005 / 1021 / 1107 / 2157; 64 x 256 x 3072 x
  // 100 (12288) 182 / 163 / 165 / 366; 128 x 512 x 256 x 50 (2048) 65 / 49 / 46 /
  // 67; 4 x 512 x 2000 x 200 (1000) 123 / 97 / 85 / 98; the gradient kernel of 3 x
  // 1100 x 131 x 301 (81) 41 with one feature, 18 split.  (8 column tiles with
  // four features a lane spill.)
  const int64_t w16 = (int64_t)a.n * chunks * ((a.d + 15) / 16);
  if (w16 <= 256 && kblocks >= 8) grads(k_sg_grads<1, NT, 8, 2, true>, 16, 512);
  else if (w16 < 4096 || a.d < 4) grads(k_sg_grads<1, NT, 4, 2, false>, 64, 256);
  else if (w16 < 32768 || NT >= 8) grads(k_sg_grads<2, NT, 4, 3, false>, 128, 256);
  else grads(k_sg_grads<4, NT, 8, 2, false>, 512, 512);
  return hipGetLastError();
}

hipError_t launch_split(const SoftmaxPlan& p, const SoftmaxArgs& a, hipStream_t s) {
  switch (p.per_thread) {
    case 1: return launch_split_nt<1>(p, a, s);
    case 2: return launch_split_nt<2>(p, a, s);
    case 3: return launch_split_nt<3>(p, a, s);
    case 4: return launch_split_nt<4>(p, a, s);
    case 5: return launch_split_nt<5>(p, a, s);
    case 6: return launch_split_nt<6>(p, a, s);
    case 7: return launch_split_nt<7>(p, a, s);
    case 8: return launch_split_nt<8>(p, a, s);
  }
  return hipErrorInvalidValue;
}

template <int U, int CW>
hipError_t launch_mfma_t(const SoftmaxPlan& p, const SoftmaxArgs& a, hipStream_t s) {
  const int64_t nb = (int64_t)a.n * p.slabs;
  const int64_t per_xcd = (nb + NXCD - 1) / NXCD;
  auto pass = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(per_xcd * NXCD)), dim3(MF_T), 0, s, a, p.slabs, p.rows_per_slab, per_xcd);
  };
  if (a.d % 4 == 0) pass(k_softmax_mfma<U, CW, false>);
  else pass(k_softmax_mfma<U, CW, true>);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || p.slabs == 1 || a.keep_slabs) return e;
  const dim3 g2(static_cast<unsigned>((a.d + 63) / 64), static_cast<unsigned>(a.n));
  hipLaunchKernelGGL(k_slab_reduce_tiles, g2, dim3(256), 0, s, a, p.slabs, U);
  return hipGetLastError();
}

template <int CW>
hipError_t launch_mfma_c(const SoftmaxPlan& p, const SoftmaxArgs& a, hipStream_t s) {
  switch (p.per_thread) {
    case 1: return launch_mfma_t<1, CW>(p, a, s);
    case 2: return launch_mfma_t<2, CW>(p, a, s);
    case 3: return launch_mfma_t<3, CW>(p, a, s);
    case 4: return launch_mfma_t<4, CW>(p, a, s);
    case 5: if constexpr (CW <= 10) return launch_mfma_t<5, CW>(p, a, s); break;
    case 6: if constexpr (CW <= 10) return launch_mfma_t<6, CW>(p, a, s); break;
  }
  return hipErrorInvalidValue;
}

// GEMM path: column tiles of a wave (per_thread) and of all classes.  Up to
// SG_NARROW tiles a wave holds all of them; else chunks of equal width.
constexpr int SG_NARROW = 8;
SoftmaxPlan split_plan(int n, int B, int d, int C, int64_t S) {
  SoftmaxPlan p;
  const int need = (C + 15) / 16, chunks = (need + SG_NARROW - 1) / SG_NARROW;
  p.per_thread = (need + chunks - 1) / chunks;
  p.tiles = p.per_thread * chunks;
  p.w_bytes = sg_frag_bytes((d + SG_K - 1) / SG_K, p.tiles);
  p.r_bytes = sg_frag_bytes((int64_t)n * ((B + SG_K - 1) / SG_K), p.tiles);
  p.z_floats = chunks > 1 ? (int64_t)n * B * C : 0;
  if (split_per_row(n, B, d, S)) {
    p.z_floats = std::max(p.z_floats, S * C);
    p.row_floats = S;
  }
  return p;
}

}  // namespace

// Single pass or GEMM path for up to 16 classes.  The single pass reads X once,
// but a block is a chain: a prologue, then `chunks` chunks of 8 rows with a
// barrier each; it pads the features to 512 U and the classes to 4, 10 or 16, and
// several slabs a worker have to be summed (beyond 8 with a wait a slab in the
// PS kernel).  The GEMM path spreads a small problem over the chip, pads rows to
// 16 and 32, and reads X twice, from the caches while there is little of it.
// The estimate is the single pass's time less the GEMM path's (us), fitted to
// 2639 pairs of whole steps: n = 4 .. 256, B = 16 .. 512, d = 64 .. 3072, 2 .. 16 classes, all
// or none of G written (the bits must not depend on that).  The path it takes
// is 0.3% slower than the better one on average, more than 5% in 67 pairs, 12%
// at most.  us, single pass / GEMM path, C = 4: 256 x 16 x 1500 27.9 / 35.9, 64 x 64 x
// 1500 28.1 / 28.3, 16 x 64 x 3072 31.3 / 28.4; C = 10: 64 x 16 x 200 18.5 / 23.1, 16 x
// 64 x 1500 29.7 / 26.0, 128 x 200 x 200 42 / 33; C = 16: 16 x 16 x 200 18.9 / 22.0, 4 x 64 x
// 200 25.6 / 22.5, 16 x 256 x 1500 36.9 / 27.9.  From 8 million elements on (d >= 256)
// the one reading of X decides: 64 x 256 x 3072 x 10 65 / 110, 256 x 48 x 744 x 16
// 39.6 / 43.5.
bool single_pass_pays(int64_t elements, int d, int width, int U, int chunks, int slabs) {
  if (elements >= 8000000 && d >= 256) return true;
  struct Fit {
    double product, chunk, million, sum, many, gemm;
  };
  static constexpr Fit kFit[3] = {{0.40, 0.65, 1.20, 1.2, 1.6, 5.1}, {0.60, 0.60, 1.30, 4.8, 4.5, 4.3}, {0.90, 0.60, 0.75, 2.0, 5.0, 4.3}};
  const Fit& f = kFit[width == 4 ? 0 : width == 10 ? 1 : 2];
  return f.product * chunks * U + f.chunk * chunks - f.million * 1e-6 * elements + (slabs > 1 ? f.sum : 0.0) +
             (slabs > 8 ? f.many : 0.0) < f.gemm;
}

SoftmaxPlan softmax_plan(int n, int B, int d, int C, int64_t S) {
  SoftmaxPlan p;
  const int cw = C <= 4 ? 4 : C <= 10 ? 10 : C <= 16 ? 16 : 0;
  const int U = (d + MF_T - 1) / MF_T;
  const bool fits = cw == 16 ? U <= 4 : U <= 6;
  if (!cw || !fits || d < 4) return split_plan(n, B, d, C, S);
  // about 256 blocks, at least four 8-row chunks per slab
  int slabs = 256 / n, max_slabs = B / (4 * MF_ROWS);
  slabs = slabs < 1 ? 1 : slabs;
  max_slabs = max_slabs < 1 ? 1 : max_slabs;
  slabs = slabs > max_slabs ? max_slabs : slabs;
  int rps = (B + slabs - 1) / slabs;
  rps = (rps + MF_ROWS - 1) / MF_ROWS * MF_ROWS;
  if (rps > FUSED_MAX_ROWS) rps = FUSED_MAX_ROWS;
  slabs = (B + rps - 1) / rps;
  if (!single_pass_pays((int64_t)n * B * d, d, cw, U, rps / MF_ROWS, slabs)) return split_plan(n, B, d, C, S);
  // 8 waves x 64U features, W staged in LDS
  p.fused = 1;
  p.per_thread = U;
  p.cpad = cw;
  p.rows_per_slab = rps;
  p.slabs = slabs;
  p.part = (int64_t)MF_T * U * C;   // tile-order partial
  // one worker's partials are read through one buffer resource
  return (int64_t)p.slabs * p.part * 4 <= kMaxBufferBytes ? p : split_plan(n, B, d, C, S);
}

hipError_t launch_softmax_grads(const SoftmaxPlan& p, const SoftmaxArgs& a, hipStream_t s) {
  if (p.fused) {
    switch (p.cpad) {
      case 4: return launch_mfma_c<4>(p, a, s);
      case 10: return launch_mfma_c<10>(p, a, s);
      case 16: return launch_mfma_c<16>(p, a, s);
    }
    return hipErrorInvalidValue;
  }
  return launch_split(p, a, s);
}

}  // namespace dbw
