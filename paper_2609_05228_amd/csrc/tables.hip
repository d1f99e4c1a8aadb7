// Offline per-expert amplification tables on the device, in fp64:
//   GSP (Alg. 2): with G = W_gate diag(gamma), U = W_up diag(gamma) ([m, d],
//     nn.Linear layout) and W_down [d, m],
//       a_up = ||U||_F ||W_down G||_F, a_gate = ||G||_F ||W_down U||_F
//       (Eqs. gsp_up_path, gsp_gate_path), a~ = sqrt(a_up a_gate)
//       (Eq. gsp_geometric_mean), A = a~ / (mean a~ + eps) (Eq. gsp_layer_normalization).
//     The two [d, d] products are never formed: ||W_down G||_F^2 =
//     <W_down^T W_down, G G^T>_F, an inner product of two m x m Gram matrices
//     (about 1.8x fewer flops than the products).  gsp_tile_kernel computes,
//     per expert and per 64 x 64 tile pair (bi <= bj) of the m x m space, the
//     tiles of W_down^T W_down, G G^T and U U^T on fp64 MFMA
//     (v_mfma_f64_16x16x4f64) and reduces sum(D o G) and sum(D o U) over the
//     tile; the Gram matrices are symmetric, so an off-diagonal pair counts
//     twice.
//   RCR (Alg. 3): w~_e = w_e - mean_j w_j (Eq. rcr_centered_router),
//     q_e = rho w~_e / (RMS(w~_e) + eps) with rho = 1 (Eq. rcr_direction_prototype),
//     a~ = ||f_e(q_e)|| / (||q_e|| + eps) with f_e the SwiGLU expert applied to
//     q_e as its input (Eq. rcr_raw_amplification), A = a~ / (mean a~ + eps)
//     (Eq. rcr_layer_normalization).  fp64 VALU (about 3 m d multiply-adds per
//     expert), rows spread over the chip: h, then W_down h.  The pass over W_gate
//     and W_up also gives each row's share of ||G||_F^2 and ||U||_F^2 for GSP.
// Every reduction has a fixed order, so the tables are deterministic; fp64
// throughout, they agree with an fp64 evaluation to ~1e-15 relative.
#include "lds_dma.h"

namespace ace {

namespace {

typedef double f64x4_t __attribute__((ext_vector_type(4)));

// 16 bytes of consecutive elements as raw storage; element i as a double
template <typename T> struct Vec;
template <> struct Vec<bf16_t> {
  static constexpr int n = 8;
  uint4 v;
  __device__ __forceinline__ void load(const bf16_t *p) { v = *reinterpret_cast<const uint4 *>(p); }
  __device__ __forceinline__ double at(int i) const {
    const uint32_t w = i < 2 ? v.x : i < 4 ? v.y : i < 6 ? v.z : v.w;
    return static_cast<double>(__uint_as_float((i & 1) ? (w & 0xFFFF0000u) : (w << 16)));
  }
};
template <> struct Vec<float> {
  static constexpr int n = 4;
  float4 v;
  __device__ __forceinline__ void load(const float *p) { v = *reinterpret_cast<const float4 *>(p); }
  __device__ __forceinline__ double at(int i) const {
    return static_cast<double>(i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w);
  }
};

// two consecutive elements
template <typename T> struct Pair;
template <> struct Pair<bf16_t> {
  uint32_t v;
  __device__ __forceinline__ void load(const bf16_t *p) { v = *reinterpret_cast<const uint32_t *>(p); }
  __device__ __forceinline__ double at(int i) const {
    return static_cast<double>(__uint_as_float(i ? (v & 0xFFFF0000u) : (v << 16)));
  }
};
template <> struct Pair<float> {
  float2 v;
  __device__ __forceinline__ void load(const float *p) { v = *reinterpret_cast<const float2 *>(p); }
  __device__ __forceinline__ double at(int i) const { return static_cast<double>(i ? v.y : v.x); }
};

__device__ __forceinline__ double to_f64(bf16_t v) { return static_cast<double>(bf16_to_f32(v)); }
__device__ __forceinline__ double to_f64(float v) { return static_cast<double>(v); }

struct TabArgs {
  const void *gamma, *w_router, *w_gate, *w_up, *w_down;
  int N, d, m, mt, n_pairs;
  double eps, rho;
  double *pair_part;  // [N][n_pairs][2]: sum(D o G), sum(D o U) of each tile pair
  double *wbar;       // [d] mean router row
  double *h;          // [N][m] SwiGLU activation of the prototype
  double *row_norm2;  // [N][m][2]: squared norms of row i of G and of U
  double *f_part;     // [N][d / 32]: sums of f_e(q_e)^2 over 32 outputs
  double *q_norm;     // [N] ||q_e||
  double *gsp_raw, *rcr_raw;  // [N]
  float *a_gsp, *a_rcr;
  double *a_gsp64, *a_rcr64;
};

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// Sums of D o G and D o U over one 64 x 64 tile pair of one expert, 4 waves;
// wave (wr, wc) owns a 32 x 32 sub-tile.  Bound by the fp64 matrix cores (a wave
// issues 12 MFMAs of 64 cycles per 4 k) and by the conversions to fp64, which hold
// them up: of 8.1 ms for 128 experts of 768 x 2048 (60 TFLOP/s of the MFMAs issued; a
// 4096^3 library product reaches 74) the conversions take 0.95 and the products with
// gamma^2 0.3.  Operands come through two LDS stages, one copied while the other is
// multiplied; read straight from L2 at every K block the kernel took 9.2 ms, and with
// the next block's loads in registers they spill (15 ms).  Two waves per SIMD; three
// measured the same.
// gamma enters one operand of each product as gamma^2, which halves the fp64
// multiplies.  gamma^2 is exact in fp64 (16 bits of bf16, 48 of fp32), and so is its
// product with a bf16 weight (24 bits); with an fp32 weight (72 bits) that is rounded
// once.  The fp32 tables do not show it: their experts spread 1.0-1.5e-16 (rms, relative)
// around sums with a 64-bit mantissa, as with gamma on both operands (six shapes of
// 128-2048 hidden, 64-256 experts of 64-192).  Row r of a
// sub-tile's 16-row block u is row 2 r + u, so W_down is read in adjacent column
// pairs.  In a diagonal tile the sub-tile below the diagonal mirrors the one above
// it: its wave does nothing and the other counts twice.
template <typename T>
__global__ __launch_bounds__(256, 2) void gsp_tile_kernel(TabArgs a) {
  constexpr int KL = Vec<T>::n;  // consecutive k of a lane
  // experts dealt to the 8 XCDs, so the tile pairs of one expert share its weights in one L2
  const int e = (blockIdx.x & 7) + 8 * blockIdx.y;
  if (e >= a.N) return;
  int p = blockIdx.x >> 3, bi = 0;
  const int pair = p;
  while (p >= a.mt - bi) {
    p -= a.mt - bi;
    ++bi;
  }
  const int bj = bi + p;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, g = lane >> 4;
  const int wr = wave >> 1, wc = wave & 1;
  const int d = a.d, m = a.m;
  const size_t eo = static_cast<size_t>(e) * m * d;
  const double mult = bi != bj || wr < wc ? 2.0 : wr == wc ? 1.0 : 0.0;
  // A stage holds 4 KL k of six operands, 4 KB each: 64 rows (bi, then bj) of W_gate
  // and of W_up, 64 bytes a row, and 64 columns (bi, bj) of W_down; then gamma's 64
  // bytes.  Wave w copies a quarter of each.  Slot 32 s + 16 u + r of a row operand
  // holds row 2 r + u of sub-tile s, so a fragment read is 1 KB in one piece.
  constexpr int KB = 4 * KL, kOp = 4096, kStage = 6 * kOp + 64;
  constexpr int kDRow = 64 * static_cast<int>(sizeof(T));  // bytes of 64 columns
  __shared__ __align__(16) uint8_t ring[2][kStage];
  const int srow = 32 * (wave >> 1) + 2 * (lane >> 2) + (wave & 1), schunk = KL * (lane & 3);
  const T *wg = static_cast<const T *>(a.w_gate) + eo, *wu = static_cast<const T *>(a.w_up) + eo;
  const size_t ra = static_cast<size_t>(bi * 64 + srow) * d + schunk, rb = static_cast<size_t>(bj * 64 + srow) * d + schunk;
  constexpr int kPerRow = kDRow / 16;  // DMA lanes of one k of W_down
  const T *wd = static_cast<const T *>(a.w_down) + eo +
                static_cast<size_t>(wave * (64 / kPerRow) + lane / kPerRow) * m + KL * (lane % kPerRow);
  const T *gam = static_cast<const T *>(a.gamma) + KL * lane;
  auto issue = [&](int slot, int k0) {
    const uint32_t base = lds_addr(ring[slot]) + wave * kUnitBytes;
    dma16(wg + ra + k0, base);
    dma16(wg + rb + k0, base + kOp);
    dma16(wu + ra + k0, base + 2 * kOp);
    dma16(wu + rb + k0, base + 3 * kOp);
    dma16(wd + static_cast<size_t>(k0) * m + bi * 64, base + 4 * kOp);
    dma16(wd + static_cast<size_t>(k0) * m + bj * 64, base + 5 * kOp);
    if (wave == 0 && lane < 4) dma16(gam + k0, lds_addr(ring[slot]) + 6 * kOp);
  };
  double sg = 0.0, su = 0.0;
  {
    f64x4_t accD[2][2], accG[2][2], accU[2][2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int v = 0; v < 2; ++v) accD[u][v] = accG[u][v] = accU[u][v] = f64x4_t{0.0, 0.0, 0.0, 0.0};

    // lane group g holds k = k0 + KL g + j and MFMA j takes element j
    const int fr = r16 * 64 + g * 16;                     // fragment offset in 16 slots
    const int dr = KL * g * kDRow + 2 * r16 * static_cast<int>(sizeof(T));
    issue(0, 0);
#pragma unroll 1
    for (int k0 = 0, slot = 0; k0 < d; k0 += KB, slot ^= 1) {
      // this stage landed for every wave, and every wave has read the other slot
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
      if (k0 + KB < d) issue(slot ^ 1, k0 + KB);
      if (mult == 0.0) continue;  // wave-uniform
      const uint8_t *st = ring[slot];
      Vec<T> gm, ga[2], gb[2], ua[2], ub[2];
      gm.load(reinterpret_cast<const T *>(st + 6 * kOp) + KL * g);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        ga[u].load(reinterpret_cast<const T *>(st + (2 * wr + u) * kUnitBytes + fr));
        gb[u].load(reinterpret_cast<const T *>(st + kOp + (2 * wc + u) * kUnitBytes + fr));
        ua[u].load(reinterpret_cast<const T *>(st + 2 * kOp + (2 * wr + u) * kUnitBytes + fr));
        ub[u].load(reinterpret_cast<const T *>(st + 3 * kOp + (2 * wc + u) * kUnitBytes + fr));
      }
#pragma unroll
      for (int j = 0; j < KL; ++j) {
        Pair<T> da, db;  // W_down[k][col], col = the pair of columns of this lane's two blocks
        da.load(reinterpret_cast<const T *>(st + 4 * kOp + dr + j * kDRow + wr * (kDRow / 2)));
        db.load(reinterpret_cast<const T *>(st + 5 * kOp + dr + j * kDRow + wc * (kDRow / 2)));
        const double gj = gm.at(j), g2 = gj * gj;
        double xa[2], xb[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          xa[u] = ga[u].at(j) * g2;
          xb[u] = gb[u].at(j);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int v = 0; v < 2; ++v)
            accG[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(xa[u], xb[v], accG[u][v], 0, 0, 0);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          xa[u] = ua[u].at(j) * g2;
          xb[u] = ub[u].at(j);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int v = 0; v < 2; ++v)
            accU[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(xa[u], xb[v], accU[u][v], 0, 0, 0);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          xa[u] = da.at(u);
          xb[u] = db.at(u);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int v = 0; v < 2; ++v)
            accD[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(xa[u], xb[v], accD[u][v], 0, 0, 0);
      }
    }
    // this wave's sub-tile (the three tiles share one layout)
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          sg = fma(accD[u][v][i], accG[u][v][i], sg);
          su = fma(accD[u][v][i], accU[u][v][i], su);
        }
    sg = wave_sum(sg) * mult;
    su = wave_sum(su) * mult;
  }
  __shared__ double part[4][2];
  if (lane == 0) {
    part[wave][0] = sg;
    part[wave][1] = su;
  }
  __syncthreads();
  if (tid == 0) {
    double *o = a.pair_part + (static_cast<size_t>(e) * a.n_pairs + pair) * 2;
    o[0] = ((part[0][0] + part[1][0]) + part[2][0]) + part[3][0];
    o[1] = ((part[0][1] + part[1][1]) + part[2][1]) + part[3][1];
  }
}

// mean router row: a workgroup takes 64 columns, wave w the experts w, w + 4, ...
template <typename T>
__global__ __launch_bounds__(256) void rcr_mean_kernel(TabArgs a) {
  __shared__ double part[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int k = blockIdx.x * 64 + lane;
  const T *W = static_cast<const T *>(a.w_router);
  double s = 0.0;
  if (k < a.d) {
#pragma unroll 8
    for (int e = wave; e < a.N; e += 4) s += to_f64(W[static_cast<size_t>(e) * a.d + k]);
  }
  part[wave][lane] = s;
  __syncthreads();
  if (wave == 0 && k < a.d)
    a.wbar[k] = (((part[0][lane] + part[1][lane]) + part[2][lane]) + part[3][lane]) / a.N;
}

// block-wide sum in a fixed order (wave butterflies, then waves in order)
__device__ __forceinline__ double block_sum4(double v, double *scratch) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) scratch[wave] = v;
  __syncthreads();
  return ((scratch[0] + scratch[1]) + scratch[2]) + scratch[3];
}

// h = SiLU(W_gate q) * (W_up q) for 16 rows of one expert (wave w: rows 4 w .. 4 w + 3),
// and the rows' shares of ||G||^2, ||U||^2.  Bound by reading the weights once, so
// the rows are spread over N m / 16 workgroups (one workgroup per expert left half
// the chip idle behind a serial chain of rows: 9.3 ms for 128 experts of 768 x 2048,
// now 0.18 ms here and 0.076 ms in rcr_out_kernel).
constexpr int kHRows = 4;  // rows of one wave
template <typename T>
__global__ __launch_bounds__(256) void rcr_hidden_kernel(TabArgs a) {
  constexpr int KL = Vec<T>::n;
  __shared__ double red[4];
  const int e = blockIdx.y, blk = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int d = a.d, m = a.m;
  const T *wr = static_cast<const T *>(a.w_router) + static_cast<size_t>(e) * d;
  const T *gam = static_cast<const T *>(a.gamma);
  // RMS of the centred router row, and ||q|| (block 0)
  double s2 = 0.0;
  for (int k = tid; k < d; k += 256) {
    const double w = to_f64(wr[k]) - a.wbar[k];
    s2 = fma(w, w, s2);
  }
  const double r = sqrt(block_sum4(s2, red) / d);
  const double inv = a.rho / (r + a.eps);
  if (blk == 0) {  // uniform over the workgroup
    double q2 = 0.0;
    for (int k = tid; k < d; k += 256) {
      const double q = (to_f64(wr[k]) - a.wbar[k]) * inv;
      q2 = fma(q, q, q2);
    }
    q2 = block_sum4(q2, red);
    if (tid == 0) a.q_norm[e] = sqrt(q2);
  }
  const int i0 = blk * 4 * kHRows + wave * kHRows;
  const size_t ro = (static_cast<size_t>(e) * m + i0) * d;
  const T *Wg = static_cast<const T *>(a.w_gate) + ro;
  const T *Wu = static_cast<const T *>(a.w_up) + ro;
  double sg[kHRows], su[kHRows], ng[kHRows], nu[kHRows];
#pragma unroll
  for (int i = 0; i < kHRows; ++i) sg[i] = su[i] = ng[i] = nu[i] = 0.0;
  for (int k = KL * lane; k < d; k += KL * 64) {
    Vec<T> wv, gv, g[kHRows], u[kHRows];
    wv.load(wr + k);
    gv.load(gam + k);
#pragma unroll
    for (int i = 0; i < kHRows; ++i) {
      g[i].load(Wg + static_cast<size_t>(i) * d + k);
      u[i].load(Wu + static_cast<size_t>(i) * d + k);
    }
#pragma unroll
    for (int j = 0; j < KL; ++j) {
      const double q = (wv.at(j) - a.wbar[k + j]) * inv, gk = gv.at(j);
#pragma unroll
      for (int i = 0; i < kHRows; ++i) {
        const double wg = g[i].at(j), wu = u[i].at(j);
        sg[i] = fma(wg, q, sg[i]);
        su[i] = fma(wu, q, su[i]);
        const double G = wg * gk, U = wu * gk;
        ng[i] = fma(G, G, ng[i]);
        nu[i] = fma(U, U, nu[i]);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < kHRows; ++i) {
    const double sgi = wave_sum(sg[i]), sui = wave_sum(su[i]);
    const double ngi = wave_sum(ng[i]), nui = wave_sum(nu[i]);
    if (lane == 0) {
      const size_t o = static_cast<size_t>(e) * m + i0 + i;
      a.h[o] = sgi / (1.0 + exp(-sgi)) * sui;
      a.row_norm2[2 * o] = ngi;
      a.row_norm2[2 * o + 1] = nui;
    }
  }
}

// sum of squares of 32 outputs f = W_down h of one expert (wave w: outputs 8 w .. 8 w + 7)
constexpr int kFRows = 8;  // outputs of one wave
template <typename T>
__global__ __launch_bounds__(256) void rcr_out_kernel(TabArgs a) {
  constexpr int KL = Vec<T>::n;
  __shared__ double red[4];
  const int nb = a.d / (4 * kFRows);
  const int e = blockIdx.y, blk = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int d = a.d, m = a.m;
  const T *Wd = static_cast<const T *>(a.w_down) +
                (static_cast<size_t>(e) * d + blk * 4 * kFRows + wave * kFRows) * static_cast<size_t>(m);
  const double *h = a.h + static_cast<size_t>(e) * m;
  double s[kFRows];
#pragma unroll
  for (int i = 0; i < kFRows; ++i) s[i] = 0.0;
  for (int k = KL * lane; k < m; k += KL * 64) {
    Vec<T> w[kFRows];
#pragma unroll
    for (int i = 0; i < kFRows; ++i) w[i].load(Wd + static_cast<size_t>(i) * m + k);
#pragma unroll
    for (int j = 0; j < KL; ++j) {
      const double hj = h[k + j];
#pragma unroll
      for (int i = 0; i < kFRows; ++i) s[i] = fma(w[i].at(j), hj, s[i]);
    }
  }
  double f2 = 0.0;  // identical in every lane of the wave
#pragma unroll
  for (int i = 0; i < kFRows; ++i) {
    const double f = wave_sum(s[i]);
    f2 = fma(f, f, f2);
  }
  if (lane == 0) red[wave] = f2;
  __syncthreads();
  if (threadIdx.x == 0) a.f_part[static_cast<size_t>(e) * nb + blk] = ((red[0] + red[1]) + red[2]) + red[3];
}

// raw GSP and RCR values of one expert: every partial sum added in a fixed order
__global__ __launch_bounds__(256) void tables_expert_kernel(TabArgs a) {
  __shared__ double red[4];
  const int e = blockIdx.x, tid = threadIdx.x;
  double dg = 0.0, du = 0.0, ng = 0.0, nu = 0.0, f2 = 0.0;
  const double *pp = a.pair_part + static_cast<size_t>(e) * a.n_pairs * 2;
  for (int p = tid; p < a.n_pairs; p += 256) {
    dg += pp[2 * p];
    du += pp[2 * p + 1];
  }
  const double *rn = a.row_norm2 + static_cast<size_t>(e) * a.m * 2;
  for (int i = tid; i < a.m; i += 256) {
    ng += rn[2 * i];
    nu += rn[2 * i + 1];
  }
  const int nb = a.d / (4 * kFRows);
  for (int i = tid; i < nb; i += 256) f2 += a.f_part[static_cast<size_t>(e) * nb + i];
  dg = block_sum4(dg, red);
  du = block_sum4(du, red);
  ng = block_sum4(ng, red);
  nu = block_sum4(nu, red);
  f2 = block_sum4(f2, red);
  if (tid == 0) {
    const double a_up = sqrt(nu) * sqrt(dg);    // ||U|| ||W_d G||
    const double a_gate = sqrt(ng) * sqrt(du);  // ||G|| ||W_d U||
    a.gsp_raw[e] = sqrt(a_up * a_gate);
    a.rcr_raw[e] = sqrt(f2) / (a.q_norm[e] + a.eps);
  }
}

// both layer normalisations
__global__ __launch_bounds__(256) void tables_finalize_kernel(TabArgs a) {
  __shared__ double red[4];
  const int tid = threadIdx.x;
  double sg_all = 0.0, sr_all = 0.0;
  for (int e = tid; e < a.N; e += 256) {
    sg_all += a.gsp_raw[e];
    sr_all += a.rcr_raw[e];
  }
  const double mg = block_sum4(sg_all, red) / a.N;
  const double mr = block_sum4(sr_all, red) / a.N;
  for (int e = tid; e < a.N; e += 256) {
    const double ag = a.gsp_raw[e] / (mg + a.eps);
    const double ar = a.rcr_raw[e] / (mr + a.eps);
    a.a_gsp[e] = static_cast<float>(ag);
    a.a_rcr[e] = static_cast<float>(ar);
    if (a.a_gsp64) a.a_gsp64[e] = ag;
    if (a.a_rcr64) a.a_rcr64[e] = ar;
  }
}

// Experts lie in the grids' y: a launch takes fewer than 2^32 threads in x (512 experts of
// 16384 have 2^24 tile pairs).
template <typename T>
void launch_tables_t(const TabArgs &a, hipStream_t stream) {
  gsp_tile_kernel<T><<<dim3(8 * a.n_pairs, (a.N + 7) / 8), 256, 0, stream>>>(a);
  rcr_mean_kernel<T><<<dim3((a.d + 63) / 64), 256, 0, stream>>>(a);
  rcr_hidden_kernel<T><<<dim3(a.m / (4 * kHRows), a.N), 256, 0, stream>>>(a);
  rcr_out_kernel<T><<<dim3(a.d / (4 * kFRows), a.N), 256, 0, stream>>>(a);
  tables_expert_kernel<<<dim3(a.N), 256, 0, stream>>>(a);
  tables_finalize_kernel<<<1, 256, 0, stream>>>(a);
}

size_t al(size_t v) { return (v + 255) / 256 * 256; }

// workspace regions of TabArgs, in order; returns the bytes used
size_t carve(TabArgs &a, char *ws) {
  size_t off = 0;
  auto take = [&](size_t n) {
    double *p = reinterpret_cast<double *>(ws + off);
    off += al(n * sizeof(double));
    return p;
  };
  const size_t N = a.N, d = a.d, m = a.m;
  a.pair_part = take(N * a.n_pairs * 2);
  a.wbar = take(d);
  a.h = take(N * m);
  a.row_norm2 = take(N * m * 2);
  a.f_part = take(N * (d / (4 * kFRows)));
  a.q_norm = take(N);
  a.gsp_raw = take(N);
  a.rcr_raw = take(N);
  return off;
}

void set_shape(TabArgs &a, int N, int d, int m) {
  a.N = N;
  a.d = d;
  a.m = m;
  a.mt = m / 64;
  a.n_pairs = a.mt * (a.mt + 1) / 2;
}

}  // namespace

size_t tables_workspace_bytes(int N, int d, int m) {
  TabArgs a{};
  set_shape(a, N, d, m);
  return carve(a, nullptr);
}

hipError_t launch_tables(const TablesCall &c, hipStream_t stream) {
  TabArgs a{};
  set_shape(a, c.N, c.d, c.m);
  carve(a, static_cast<char *>(c.workspace));
  a.gamma = c.gamma;
  a.w_router = c.w_router;
  a.w_gate = c.w_gate;
  a.w_up = c.w_up;
  a.w_down = c.w_down;
  a.eps = c.eps;
  a.rho = 1.0;
  a.a_gsp = c.a_gsp;
  a.a_rcr = c.a_rcr;
  a.a_gsp64 = c.a_gsp64;
  a.a_rcr64 = c.a_rcr64;
  if (c.bf16)
    launch_tables_t<bf16_t>(a, stream);
  else
    launch_tables_t<float>(a, stream);
  return hipGetLastError();
}

}  // namespace ace
