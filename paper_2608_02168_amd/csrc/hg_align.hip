// hg_align_loss_fwd_bwd: CCA consistency-alignment loss on the overlap batch
// (Section "Cross-Subgraph Consistency Alignment": standardisation,
// invariance, decorrelation and CCA-loss equations) and its gradient, in
// three passes over the two views X = H[overlap] and Y = H_ref:
//
//   (d1) k_align_stats: per-column float64 sums of x and x^2 of both views,
//        one partial row set per chunk of rows; k_align_mean: mean, 1/sigma
//        and standardisation scale of every column from them;
//   (d2) k_align_gram: over its chunk of rows a block forms the Gram matrices
//        Xh^T Xh and Yh^T Yh on the split-fp16 MFMA (only the blocks on and
//        above the diagonal) and, in float64, the column sums the gradient
//        and the loss need:
//          v = sum Xh, w = sum Yh, u = sum o (Xh - Yh),
//          p = sum o (Xh - Yh) Xh, q = sum o (Yh - Xh) Yh, l = sum o (Xh - Yh)^2
//        (o the row weight); k_align_reduce sums the chunks, mirrors the Grams
//        and writes C' = Xh^T Xh - I (and of Y);
//   (d3) the gradient row GEMM Xh C' on the split-fp16 MFMA.  Its blocks form
//        the two column vectors of the standardisation backward from C' and
//        the sums: with G = 2 o (Xh - Yh) + 4 lambda Xh C' and g' = G / sqrt(M),
//          S1 = sum_b g'_b = (2 u + 4 lambda v C') / sqrt(M),
//          S2 = sum_b g'_b xt_b = 2 p + 4 lambda diag(C C')
//        (xt = (x - mu) / sigma = Xh sqrt(M)), so G never reaches memory; the
//        first block writes the loss.  The epilogue forms G, the
//        standardisation backward
//          dX = (1/sigma) (g' - S1 / M - xt S2 / (M - ddof))
//        and writes dH[overlap] = base + scale * dX (rows are distinct: no
//        atomics); the same for Y into dH_ref when it is requested.
//
// Every reduction has a fixed order: results are bitwise reproducible.
#include <mutex>

#include "hg_internal.h"
#include "hg_mfma.h"

namespace hg {

namespace {

constexpr int kStatChunksMax = 128;   // chunks per view of (d1)
constexpr float kGramScale = 16384.f;                      // 2^14
constexpr float kGramUnscale = 1.0f / (16384.f * 16384.f);  // 2^-28

// |Xh| <= 1 for every element: (x - mu)^2 is one term of the column's sum of
// squares, which is (M - ddof) var <= M (var + eps) = M sigma^2.  Scaled by
// 2^14 every value is below 2^15, so the split-fp16 parts cannot overflow.

template <int D>
struct AShape {
  static constexpr int QN = D / 64;                  // 64-feature quadrants per side
  static constexpr int NQ = QN * (QN + 1) / 2;       // quadrants with qi <= qj
  // a block takes both views, at d = 256 one (two blocks per chunk): a thread
  // stages 4 rows x 4 columns of each view it holds
  static constexpr int VB = D == 256 ? 1 : 2;
  static constexpr int BPC = 2 / VB;
  static constexpr int kThreads = 2 * D;
  static constexpr int NW = kThreads / 64;
  static constexpr int TASKS = 2 * VB * NQ;          // half quadrants (32 x 64) of a block
  static constexpr int TPW = (TASKS + NW - 1) / NW;  // of a wave: 2, 3 and 3
  // two blocks per compute unit (one at d = 256) within the static scratch
  // of the no-allocation entry point
  static constexpr int kChunkCap = D == 64 ? 512 : (D == 128 ? 448 : 128);
  static constexpr int kGramFloats = 2 * NQ * 64 * 64;  // one chunk's partial Grams, both views
  static constexpr int kRedGram = kGramFloats / 64;     // blocks of the reduction: Gram elements,
  static constexpr int kRedSums = 6 * D / 16;           // column sums
};

struct AlignPlan {
  int64_t m, nch1, rpc1, nchg, rpc2, grid2;
};

constexpr int kGramStep = 32;  // rows of a step

template <int D>
AlignPlan align_plan(int64_t m) {
  AlignPlan p{};
  p.m = m;
  p.nch1 = m > 0 ? (cdiv(m, 512) < kStatChunksMax ? cdiv(m, 512) : kStatChunksMax) : 1;
  p.rpc1 = m > 0 ? cdiv(m, p.nch1) : 1;
  int64_t n = m > 0 ? cdiv(m, 2 * kGramStep) : 1;
  n = n < AShape<D>::kChunkCap ? n : AShape<D>::kChunkCap;
  p.rpc2 = cdiv(cdiv(m > 0 ? m : 1, n), kGramStep) * kGramStep;
  p.nchg = m > 0 ? cdiv(m, p.rpc2) : 1;
  p.grid2 = AShape<D>::BPC == 1 ? p.nchg : 16 * cdiv(p.nchg, 8);
  return p;
}

// finals: C' of both views, then per view mu, 1/sigma and the standardisation
// scale 1/(sigma sqrt(M)) ([2][D] each)
template <int D>
struct AlignFin {
  float* base;
  __host__ __device__ float* cp(int v) const { return base + (int64_t)v * D * D; }
  __host__ __device__ float* mu(int v) const { return base + 2 * D * D + v * D; }
  __host__ __device__ float* is(int v) const { return base + 2 * D * D + 2 * D + v * D; }
  __host__ __device__ float* sh(int v) const { return base + 2 * D * D + 4 * D + v * D; }
  static constexpr int64_t kFloats = 2 * D * D + 6 * D;
};

template <int D>
struct AlignWs {
  double* stat;   // [nch1][2 views][2][D]
  float* gpart;   // [nchg][2 views][NQ][64 x 64]
  double* spart;  // [nchg][6][D]
  double* sums;   // [6][D]
  double* lpart;  // [kRedGram] parts of L_dec
  float* fin;     // AlignFin
  template <class A>
  void layout(A& a, const AlignPlan& p) {
    stat = a.template take<double>(p.nch1 * 4 * D);
    gpart = a.template take<float>(p.nchg * (int64_t)AShape<D>::kGramFloats);
    spart = a.template take<double>(p.nchg * 6 * D);
    sums = a.template take<double>(6 * D);
    lpart = a.template take<double>(AShape<D>::kRedGram);
    fin = a.template take<float>(AlignFin<D>::kFloats);
  }
};

// ---- (d1) column sums of x and x^2 ----------------------------------------------
// grid (chunks, 2 views), 16 waves; a row is D/4 lanes reading 16 bytes
// (columns c..c+3), four rows per lane in flight (their overlap entries first).
// Lanes of one column are combined by xor shuffles inside the wave, then the
// waves in order.
constexpr int kStatThreads = 1024;
template <int D, class T>
__global__ void __launch_bounds__(kStatThreads) k_align_stats(int64_t m, int64_t rpc, const T* __restrict__ H,
                                                              const int32_t* __restrict__ ov,
                                                              const T* __restrict__ Href, double* __restrict__ stat) {
  constexpr int TPR = D / 4, RPI = kStatThreads / TPR, U = 4, NW = kStatThreads / 64;
  __shared__ double red[NW][8][TPR < 64 ? TPR : 64];
  const int t = threadIdx.x;
  const int view = blockIdx.y;
  const int c = (t % TPR) * 4, ph = t / TPR;
  const int64_t b0 = (int64_t)blockIdx.x * rpc;
  const int64_t b1 = (b0 + rpc < m) ? b0 + rpc : m;
  const T* base = view ? Href : H;
  double s[4] = {0.0, 0.0, 0.0, 0.0}, q[4] = {0.0, 0.0, 0.0, 0.0};
  auto add = [&](const f32x4& v) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double x = (double)v[k];
      s[k] += x;
      q[k] += x * x;
    }
  };
  int64_t b = b0 + ph;
  for (; b + (U - 1) * RPI < b1; b += U * RPI) {
    int64_t r[U];
#pragma unroll
    for (int u = 0; u < U; ++u) r[u] = view ? b + u * RPI : (int64_t)ov[b + u * RPI];
    f32x4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = Elt<T>::load4(base + r[u] * D + c);
#pragma unroll
    for (int u = 0; u < U; ++u) add(v[u]);
  }
  for (; b < b1; b += RPI) add(Elt<T>::load4(base + (view ? b : (int64_t)ov[b]) * D + c));
  // lanes of the same columns inside the wave (rows ph differ in the lane bits above TPR)
#pragma unroll
  for (int o = TPR; o < 64; o <<= 1)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      s[k] += __shfl_xor(s[k], o, 64);
      q[k] += __shfl_xor(q[k], o, 64);
    }
  const int wv = t >> 6, l = t & 63;
  constexpr int LW = TPR < 64 ? TPR : 64;  // distinct column groups per wave
  if (l < LW)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      red[wv][k][l] = s[k];
      red[wv][4 + k][l] = q[k];
    }
  __syncthreads();
  // column group cg is held by lane cg % 64 of the waves whose lanes cover it
  if (t < TPR) {
    double* out = stat + ((int64_t)blockIdx.x * 2 + view) * 2 * D;
    constexpr int WPR = TPR / LW;  // waves per row (D = 256: a row spans one wave)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      double ts = 0.0, tq = 0.0;
      for (int ww = t / LW; ww < NW; ww += WPR) {
        ts += red[ww][k][t % LW];
        tq += red[ww][4 + k][t % LW];
      }
      out[c + k] = ts;
      out[D + c + k] = tq;
    }
  }
}

// Fixed-order sum over the threads of a block (NT <= 1024).
template <int NT>
__device__ double block_sum_d(double v, double* red) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int o = 512; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o && (int)threadIdx.x + o < NT) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  const double r = red[0];
  __syncthreads();
  return r;
}

// quadrant index q (qi <= qj, row-major over the upper triangle) -> (qi, qj)
template <int QN>
__device__ __forceinline__ void quad_of(int q, int& qi, int& qj) {
  qi = 0;
  qj = 0;
#pragma unroll
  for (int i = 0; i < QN; ++i) {
    if (q >= 0 && q < QN - i) {
      qi = i;
      qj = i + q;
    }
    q -= QN - i;
  }
}

// Mean, 1/sigma and scale of both views from the chunks' sums: 16 columns x 16
// runs of chunks per block, each run in order, then the runs in order.
template <int D>
__global__ void __launch_bounds__(256) k_align_mean(int64_t m, int64_t nch1, int32_t ddof, float eps,
                                                    const double* __restrict__ stat, float* __restrict__ finp) {
  __shared__ double rs[16][16], rq[16][16];
  const int e = threadIdx.x & 15, grp = threadIdx.x >> 4;
  const int vc = blockIdx.x * 16 + e, v = vc / D, c = vc % D;
  const int64_t per = (nch1 + 15) / 16;
  double s = 0.0, q = 0.0;
  for (int64_t k = grp * per; k < (grp + 1) * per && k < nch1; ++k) {
    s += stat[(k * 2 + v) * 2 * D + c];
    q += stat[(k * 2 + v) * 2 * D + D + c];
  }
  rs[grp][e] = s;
  rq[grp][e] = q;
  __syncthreads();
  if (grp) return;
  for (int g = 1; g < 16; ++g) {
    s += rs[g][e];
    q += rq[g][e];
  }
  const double mean = s / (double)m;
  double var = (q - s * mean) / (double)(m - ddof);
  var = var > 0.0 ? var : 0.0;
  const float sig = sqrtf((float)var + eps);
  const AlignFin<D> fin{finp};
  fin.mu(v)[c] = (float)mean;
  fin.is(v)[c] = 1.0f / sig;
  fin.sh(v)[c] = 1.0f / (sig * sqrtf((float)m));
}

// ---- (d2) Grams and column sums ------------------------------------------------
// A step is 32 rows of the block's views.  Thread (row quarter of 8, 4 columns)
// loads 4 rows x 4 columns of each view, standardises them, adds its share of
// the float64 column sums and writes the values' two fp16 parts into LDS in the
// MFMA's order (8 rows of one feature per 16 bytes), once per element; the next
// step's rows are loaded while the waves multiply, and two LDS buffers leave one
// barrier per step.  A wave owns TPW half quadrants of the upper triangles, so a
// step's products are spread evenly over the waves.  Feature f sits at f ^ ((f /
// 16) mod 4), which spreads the staging stores over the banks.
// With the rows parked as stored, every wave that used an element standardised
// and split it again, two waves summed the columns (a serial float64 chain per
// step) and each block reduced the statistics first: 184 us at 100k rows, d =
// 128, of which the last-block reductions took about 50, and 526 us at 800k. Now
// 41 and 238 us, with the statistics (6) and the reduction (12) as launches of
// their own; d = 256 in bf16 at 800k rows 1610 -> 666 us.
template <int D, class T>
struct GramLds {
  static constexpr size_t kFrag = sizeof(uint4) * 2 * AShape<D>::VB * 4 * D;  // one buffer
  static constexpr size_t kTail = sizeof(double) * AShape<D>::kThreads * 25;  // the column sums after the walk
  static constexpr size_t kBytes = 2 * kFrag > kTail ? 2 * kFrag : kTail;
};

template <int D, class T>
__global__ void __launch_bounds__(AShape<D>::kThreads, 2) k_align_gram(
    int64_t m, int64_t rpc, int64_t nchg, const T* __restrict__ H, const int32_t* __restrict__ ov,
    const T* __restrict__ Href, const float* __restrict__ w, const float* __restrict__ finp,
    float* __restrict__ gpart, double* __restrict__ spart) {
  typedef AShape<D> S;
  constexpr int NQ = S::NQ, QN = S::QN, VB = S::VB, TPW = S::TPW, C4 = D / 4;
  constexpr bool kPad = S::TASKS != S::NW * TPW;
  typedef typename Elt<T>::raw4_t Raw;
  extern __shared__ __align__(16) unsigned char lds[];
  uint4* frag = reinterpret_cast<uint4*>(lds);  // [2 buffers][hi, lo][VB][4 K groups][D]
  auto slot = [](int buf, int part, int v) { return ((buf * 2 + part) * VB + v) * 4 * D; };
  const int tid = threadIdx.x;
  int64_t chunk;
  int y;
  if (S::BPC == 1) {
    chunk = blockIdx.x;
    y = 0;
  } else {
    // the two blocks of a chunk are 8 apart: same XCD, so the second read of a row hits its L2
    y = (blockIdx.x >> 3) & 1;
    chunk = (int64_t)(((blockIdx.x >> 4) << 3) | (blockIdx.x & 7));
  }
  if (chunk >= nchg) return;  // a padding block
  const int64_t r_beg = chunk * rpc, r_end = (r_beg + rpc < m) ? r_beg + rpc : m;
  const AlignFin<D> fin{const_cast<float*>(finp)};
  // staging role
  const int rq = tid / C4, col = 4 * (tid % C4);  // rows 4 rq .. + 3 of a step
  const bool useX = VB == 2 || y == 0, csum = y == 0;
  // mean and scale of the thread's columns, read from LDS where they are used
  __shared__ float k_st[4][D];  // mu, scale of X, then of Y
  for (int e = tid; e < 4 * D; e += S::kThreads)
    k_st[e / D][e % D] = (e / D) & 1 ? fin.sh(e / (2 * D))[e % D] : fin.mu(e / (2 * D))[e % D];
  __syncthreads();
  int32_t id[4];
  Raw xr[4], yr[4];
  float om[4];
  // rows past the end are read from the last one and zeroed before use
  auto row_at = [&](int64_t r0, int e) -> int64_t {
    const int64_t r = r0 + 4 * rq + e;
    return r < r_end ? r : r_end - 1;
  };
  auto ids = [&](int64_t r0) {
#pragma unroll
    for (int e = 0; e < 4; ++e) id[e] = VB == 2 || useX ? ov[row_at(r0, e)] : 0;
  };
  auto fetch = [&](int64_t r0) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (VB == 2 || useX) xr[e] = Elt<T>::raw4(H + (int64_t)id[e] * D + col);
      yr[e] = Elt<T>::raw4(Href + row_at(r0, e) * D + col);
      om[e] = w ? w[row_at(r0, e)] : 1.f;
    }
  };
  double cs[6][4];
#pragma unroll
  for (int k = 0; k < 6; ++k)
#pragma unroll
    for (int q = 0; q < 4; ++q) cs[k][q] = 0.0;
  // fp16 parts of 4 rows of one column: pairs of words
  auto put = [&](int buf, int v, int q, const float (&x)[4]) {
    uint2 h, lo;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const float a = x[2 * p] * kGramScale, b = x[2 * p + 1] * kGramScale;
      const auto hp = __builtin_amdgcn_cvt_pkrtz(a, b);
      const auto lp = __builtin_amdgcn_cvt_pkrtz(a - (float)hp[0], b - (float)hp[1]);
      (p ? h.y : h.x) = __builtin_bit_cast(uint32_t, hp);
      (p ? lo.y : lo.x) = __builtin_bit_cast(uint32_t, lp);
    }
    const int f = (rq >> 1) * D + col + (q ^ ((col >> 4) & 3));
    reinterpret_cast<uint2*>(frag + slot(buf, 0, v) + f)[rq & 1] = h;
    reinterpret_cast<uint2*>(frag + slot(buf, 1, v) + f)[rq & 1] = lo;
  };
  // one column at a time (the barriers and the constants in LDS keep the
  // compiler from holding all four columns' values at once, which spilled 55
  // registers at d = 128 and doubled the pass's time)
  auto park = [&](int buf, int64_t r0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float mx = k_st[0][col + q], sx = k_st[1][col + q], my = k_st[2][col + q], sy = k_st[3][col + q];
      float xh[4], yh[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool ok = r0 + 4 * rq + e < r_end;
        xh[e] = (VB == 2 || useX) && ok ? (Elt<T>::cook4(xr[e])[q] - mx) * sx : 0.f;
        yh[e] = ok ? (Elt<T>::cook4(yr[e])[q] - my) * sy : 0.f;
      }
      if (VB == 2 || csum) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const double xv = (double)xh[e], yv = (double)yh[e], dl = xv - yv, od = (double)om[e] * dl;
          cs[0][q] += xv;
          cs[1][q] += yv;
          cs[2][q] += od;
          cs[3][q] += od * xv;
          cs[4][q] -= od * yv;
          cs[5][q] += od * dl;
        }
      }
      if constexpr (VB == 2) {
        put(buf, 0, q, xh);
        put(buf, 1, q, yh);
      } else {
        if (y == 0) put(buf, 0, q, xh); else put(buf, 0, q, yh);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // the wave's tasks, in scalar registers
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), l = lane64();
  const int g = l >> 4, c = l & 15;
  f32x4 acc[TPW][2][4];
  int tv[TPW], tq[TPW], fa[TPW], fb[TPW];  // view slot, quadrant, first feature of the two sides
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int tk = wv * TPW + t;
    tv[t] = tk < S::TASKS ? tk / (2 * NQ) : -1;
    tq[t] = (tk >> 1) % NQ;
    int qi, qj;
    quad_of<QN>(tq[t], qi, qj);
    fa[t] = 64 * qi + 32 * (tk & 1);
    fb[t] = 64 * qj;
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
      for (int bj = 0; bj < 4; ++bj) acc[t][bi][bj] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  ids(r_beg);
  fetch(r_beg);
  ids(r_beg + kGramStep);
  int buf = 0;
  for (int64_t r0 = r_beg; r0 < r_end; r0 += kGramStep, buf ^= 1) {
    park(buf, r0);
    lds_barrier();
    if (r0 + kGramStep < r_end) {
      fetch(r0 + kGramStep);
      ids(r0 + 2 * kGramStep);
    }
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
      if (kPad && tv[t] < 0) continue;
      uint4 ha[2], la[2];
#pragma unroll
      for (int bi = 0; bi < 2; ++bi) {
        // (f / 16) mod 4 of the feature: 2 (half) + bi on this side, bj on the other
        const int f = fa[t] + 16 * bi + (c ^ (((fa[t] >> 4) & 2) + bi));
        ha[bi] = frag[slot(buf, 0, tv[t]) + g * D + f];
        la[bi] = frag[slot(buf, 1, tv[t]) + g * D + f];
      }
#pragma unroll
      for (int bj = 0; bj < 4; ++bj) {
        const int f = fb[t] + 16 * bj + (c ^ bj);
        const uint4 hb = frag[slot(buf, 0, tv[t]) + g * D + f];
        const uint4 lb = frag[slot(buf, 1, tv[t]) + g * D + f];
#pragma unroll
        for (int bi = 0; bi < 2; ++bi) {
          acc[t][bi][bj] = mfma_f16(ha[bi], hb, acc[t][bi][bj]);
          acc[t][bi][bj] = mfma_f16(ha[bi], lb, acc[t][bi][bj]);
          acc[t][bi][bj] = mfma_f16(la[bi], hb, acc[t][bi][bj]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);  // one task's fragments at a time
    }
  }
  // partial Grams of this chunk: register v of block (bi, bj) is element
  // [16 bi + 4 g + v][16 bj + c] of the half quadrant
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    if (kPad && tv[t] < 0) continue;
    const int view = VB == 2 ? tv[t] : y;
    float* out = gpart + chunk * (int64_t)S::kGramFloats + (int64_t)(view * NQ + tq[t]) * 4096 + (fa[t] & 32) * 64;
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int bj = 0; bj < 4; ++bj)
          out[(16 * bi + 4 * g + v) * 64 + 16 * bj + c] = acc[t][bi][bj][v] * kGramUnscale;
  }
  if (!csum) return;  // the whole block
  __syncthreads();    // the last step's fragments have been read
  double* sred = reinterpret_cast<double*>(lds);  // [threads][25]
#pragma unroll
  for (int k = 0; k < 6; ++k)
#pragma unroll
    for (int q = 0; q < 4; ++q) sred[tid * 25 + 4 * k + q] = cs[k][q];
  __syncthreads();
  for (int e = tid; e < 6 * D; e += S::kThreads) {
    const int k = e / D, cc = e % D;
    double t = 0.0;
#pragma unroll
    for (int p = 0; p < 8; ++p) t += sred[(p * C4 + cc / 4) * 25 + 4 * k + cc % 4];
    spart[chunk * 6 * D + e] = t;
  }
}

// Reduction of the chunks: 16 elements (4 floats each, or one double) x 16 runs
// of chunks per block, each run in order, then the runs in order.  Blocks below
// kRedGram form C' = sum - I (both triangles) and their part of L_dec, the rest
// the column sums.
template <int D>
__global__ void __launch_bounds__(256) k_align_reduce(int64_t nchg, const float* __restrict__ gpart,
                                                      const double* __restrict__ spart, double* __restrict__ sums,
                                                      double* __restrict__ lpart, float* __restrict__ finp) {
  typedef AShape<D> S;
  __shared__ f32x4 rf[16][16];
  __shared__ double rd[16][16];
  const int e = threadIdx.x & 15, grp = threadIdx.x >> 4;
  const int64_t per = (nchg + 15) / 16, c0 = grp * per, c1 = c0 + per < nchg ? c0 + per : nchg;
  if ((int)blockIdx.x >= S::kRedGram) {
    const int el = (blockIdx.x - S::kRedGram) * 16 + e;
    double t = 0.0;
#pragma unroll 8
    for (int64_t k = c0; k < c1; ++k) t += spart[k * 6 * D + el];
    rd[grp][e] = t;
    __syncthreads();
    if (grp) return;
    for (int g = 1; g < 16; ++g) t += rd[g][e];
    sums[el] = t;
    return;
  }
  const int e4 = blockIdx.x * 16 + e;
  f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
  for (int64_t k = c0; k < c1; ++k) t += *reinterpret_cast<const f32x4*>(gpart + k * S::kGramFloats + 4 * e4);
  rf[grp][e] = t;
  __syncthreads();
  if (grp) return;
  for (int g = 1; g < 16; ++g) t += rf[g][e];
  const AlignFin<D> fin{finp};
  const int el = 4 * e4;
  const int vw = el / (S::NQ * 4096), q = (el / 4096) % S::NQ, i = (el % 4096) / 64, j0 = el % 64;
  int a, b;
  quad_of<S::QN>(q, a, b);
  const int gi = 64 * a + i;
  double ldec = 0.0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int gj = 64 * b + j0 + k;
    const float cp = t[k] - (gi == gj ? 1.f : 0.f);
    fin.cp(vw)[gi * D + gj] = cp;
    if (a != b) fin.cp(vw)[gj * D + gi] = cp;
    ldec += (a != b ? 2.0 : 1.0) * (double)cp * (double)cp;
  }
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) ldec += __shfl_xor(ldec, o, 64);
  if (e == 0) lpart[blockIdx.x] = ldec;
}

// ---- (d3) the gradient pass ---------------------------------------------------
// Row GEMM acc = Xh C' on the split-fp16 MFMA (C' staged once per block in
// LDS in fragment order, as in k_gemm_rows: the W fragments are the A
// operand, the rows the B operand, so lane (c, g) of wave w ends with row
// 16 w + c of a 128-row tile, columns col0 + 16 nb + 4 g .. + 3), with the
// standardisation backward in the epilogue:
//   out = base + o kx (Xh - Yh) - kc - ke (x - mu) + ka acc,
//   kx = scale (1/sigma) 2 / sqrt(M),  kc = scale (1/sigma) S1 / M,
//   ke = scale (1/sigma)^2 S2 / (M - ddof),  ka = scale (1/sigma) 4 lambda / sqrt(M)
// (the file comment's dX times scale).  The lane's x columns of every output
// block are among the A-operand columns it holds, so only the other view's
// row and the base row are read in the epilogue.  blockIdx.y picks the
// 128-column slice at d = 256.
template <int D, class T>
__global__ void __launch_bounds__(kGemmThreads) k_align_grad(int64_t m, const T* __restrict__ self, RowMap smap,
                                                             const T* __restrict__ other, RowMap omap,
                                                             const float* __restrict__ finp, int view,
                                                             const float* __restrict__ w, const T* base, T* out,
                                                             float scale, float lambda_n, int32_t ddof,
                                                             const double* __restrict__ sums,
                                                             const double* __restrict__ lpart,
                                                             float* __restrict__ loss3) {
  constexpr int DN = F32Slice<D>::DN;
  constexpr int KB = D / 16, KB2 = D / 32, NB = DN / 16;
  constexpr int kWaves = kGemmThreads / 64;
  constexpr int kRowsPerTile = 16 * kWaves;
  constexpr int kFrag = KB2 * NB * 64;
  extern __shared__ uint4 wsl[];  // [kFrag] high parts, then [kFrag] remainders
  __shared__ float wmax[kWaves + 1];
  __shared__ float k_mu[D], k_sh[D], k_muo[D], k_sho[D], k_x[D], k_c[D], k_e[D], k_a[D];
  const AlignFin<D> fin{const_cast<float*>(finp)};
  const float* W = fin.cp(view);
  const int tid = threadIdx.x;
  const int col0 = DN * blockIdx.y;
  {
    // S1 and S2 of every column: a column of C' by kPer threads (C' is
    // symmetric, so (C' C')_cc is the column's sum of squares)
    constexpr int kPer = kGemmThreads / D, kRows = D / kPer;
    __shared__ double r1[kPer][D], r2[kPer][D];
    {
      const int c = tid % D, part = tid / D;
      double t1 = 0.0, t2 = 0.0;
#pragma unroll 16
      for (int k = part * kRows; k < (part + 1) * kRows; ++k) {
        const double pk = (double)W[(int64_t)k * D + c];
        t1 += sums[view * D + k] * pk;  // v C' (view X) or w C' (view Y)
        t2 += pk * pk;
      }
      r1[part][c] = t1;
      r2[part][c] = t2;
    }
    __syncthreads();
    const float rs = 1.0f / sqrtf((float)m);
    const double inv_sqrt_m = 1.0 / sqrt((double)m);
    for (int c = tid; c < D; c += kGemmThreads) {
      double t1 = 0.0, t2 = 0.0;
#pragma unroll
      for (int p = 0; p < kPer; ++p) {
        t1 += r1[p][c];
        t2 += r2[p][c];
      }
      const double u = view == 0 ? sums[2 * D + c] : -sums[2 * D + c];
      const double pq = view == 0 ? sums[3 * D + c] : sums[4 * D + c];
      const float S1 = (float)((2.0 * u + 4.0 * (double)lambda_n * t1) * inv_sqrt_m);
      const float S2 = (float)(2.0 * pq + 4.0 * (double)lambda_n * (t2 + (double)W[(int64_t)c * D + c]));
      const float isg = fin.is(view)[c];
      k_mu[c] = fin.mu(view)[c];
      k_sh[c] = fin.sh(view)[c];
      k_muo[c] = fin.mu(1 - view)[c];
      k_sho[c] = fin.sh(1 - view)[c];
      k_x[c] = scale * isg * 2.0f * rs;
      k_c[c] = scale * isg * S1 / (float)m;
      k_e[c] = scale * isg * isg * S2 / (float)(m - ddof);
      k_a[c] = scale * isg * 4.0f * lambda_n * rs;
    }
    if (loss3 && blockIdx.x == 0 && blockIdx.y == 0) {  // the losses (the whole block)
      double* lred = &r1[0][0];  // kPer * D = kGemmThreads words, read above
      __syncthreads();
      double ld = 0.0, li = 0.0;
      for (int e = tid; e < AShape<D>::kRedGram; e += kGemmThreads) ld += lpart[e];
      for (int e = tid; e < D; e += kGemmThreads) li += sums[5 * D + e];
      const double L_dec = block_sum_d<kGemmThreads>(ld, lred), L_inv = block_sum_d<kGemmThreads>(li, lred);
      if (tid == 0) {
        loss3[0] = (float)L_inv;
        loss3[1] = (float)L_dec;
        loss3[2] = (float)(L_inv + (double)lambda_n * L_dec);
      }
    }
    float mx = 0.f;
    for (int e = tid; e < D * D / 4; e += kGemmThreads) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(W + 4 * e);
      mx = fmaxf(mx, fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3]))));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    if ((tid & 63) == 0) wmax[tid >> 6] = mx;
    __syncthreads();
    mx = wmax[0];
#pragma unroll
    for (int q = 1; q < kWaves; ++q) mx = fmaxf(mx, wmax[q]);
    const uint32_t ew = split_exp(mx);
    const float sw = split_scale(ew);
    for (int e = tid; e < kFrag; e += kGemmThreads) {
      const int l = e & 63;
      const int nb = (e >> 6) % NB;
      const int kb2 = (e >> 6) / NB;
      const int j = col0 + 16 * nb + (l & 15);
      float v[8];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int k0 = 16 * (2 * kb2 + h) + 4 * (l >> 4);
#pragma unroll
        for (int q = 0; q < 4; ++q) v[4 * h + q] = W[(int64_t)(k0 + q) * D + j] * sw;
      }
      split8(v, wsl[e], wsl[kFrag + e]);
    }
    if (tid == 0) wmax[kWaves] = split_unscale(ew);
    __syncthreads();
  }
  const float uw = wmax[kWaves];
  const int wv = tid >> 6;
  const int l = lane64();
  const int g = l >> 4, c = l & 15;
  const int64_t ntiles = (m + kRowsPerTile - 1) / kRowsPerTile;
  for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const int64_t i = t * kRowsPerTile + 16 * wv + c;
    const bool live = i < m;
    const int64_t rs_ = live ? smap(i) : 0;
    typename Elt<T>::raw4_t xr[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) xr[kb] = Elt<T>::raw4(self + rs_ * D + 16 * kb + 4 * g);
    uint4 xh[KB2], xlo[KB2];
    float ux;
    {
      auto xhat = [&](int kb) -> f32x4 {
        const int col = 16 * kb + 4 * g;
        const f32x4 x = Elt<T>::cook4(xr[kb]);
        f32x4 r;
#pragma unroll
        for (int q = 0; q < 4; ++q) r[q] = live ? (x[q] - k_mu[col + q]) * k_sh[col + q] : 0.f;
        return r;
      };
      float mx = 0.f;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const f32x4 a = xhat(kb);
        mx = fmaxf(mx, fmaxf(fmaxf(fabsf(a[0]), fabsf(a[1])), fmaxf(fabsf(a[2]), fabsf(a[3]))));
      }
      mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const uint32_t ex = split_exp(mx);
      const float sx = split_scale(ex);
      ux = split_unscale(ex);
#pragma unroll
      for (int kb2 = 0; kb2 < KB2; ++kb2) {
        const f32x4 a0 = xhat(2 * kb2), a1 = xhat(2 * kb2 + 1);
        float v[8];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          v[q] = a0[q] * sx;
          v[4 + q] = a1[q] * sx;
        }
        split8(v, xh[kb2], xlo[kb2]);
      }
    }
    f32x4 acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb2 = 0; kb2 < KB2; ++kb2) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const int e = (kb2 * NB + nb) * 64 + l;
        const uint4 bh = wsl[e], bl = wsl[kFrag + e];
        acc[nb] = mfma_f16(bh, xh[kb2], acc[nb]);
        acc[nb] = mfma_f16(bh, xlo[kb2], acc[nb]);
        acc[nb] = mfma_f16(bl, xh[kb2], acc[nb]);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (live) {
      const int64_t ro = omap(i);
      const float om = w ? w[i] : 1.f;
      f32x4 yv[NB], bv[NB];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const int col = col0 + 16 * nb + 4 * g;
        yv[nb] = Elt<T>::load4(other + ro * D + col);
        bv[nb] = base ? Elt<T>::load4(base + rs_ * D + col) : f32x4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const int col = col0 + 16 * nb + 4 * g;
        // the lane's A chunk of these columns (both candidates named at
        // compile time: a run-time index would put the row in scratch)
        f32x4 x;
        if constexpr (D == DN) {
          x = Elt<T>::cook4(xr[nb]);
        } else {
          x = blockIdx.y == 0 ? Elt<T>::cook4(xr[nb]) : Elt<T>::cook4(xr[NB + nb]);
        }
        const f32x4 a = split_unscale4(acc[nb], ux, uw);
        f32x4 r;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int cc = col + q;
          const float dxm = x[q] - k_mu[cc];
          const float xhv = dxm * k_sh[cc];
          const float yhv = (yv[nb][q] - k_muo[cc]) * k_sho[cc];
          r[q] = bv[nb][q] + om * k_x[cc] * (xhv - yhv) - k_c[cc] - k_e[cc] * dxm + k_a[cc] * a[q];
        }
        if constexpr (sizeof(T) == 4) {
          *reinterpret_cast<f32x4*>(out + rs_ * D + col) = r;
        } else {
          *reinterpret_cast<uint2*>(out + rs_ * D + col) = uint2{pack2bf(r[0], r[1]), pack2bf(r[2], r[3])};
        }
      }
    }
  }
}

template <int D, class T>
int launch_align_grad(int64_t m, const T* self, RowMap smap, const T* other, RowMap omap, const float* fin,
                      int view, const float* w, const T* base, T* out, float scale, float lambda_n, int32_t ddof,
                      const double* sums, const double* lpart, float* loss3, hipStream_t s) {
  constexpr int DN = F32Slice<D>::DN;
  const int64_t tiles = cdiv(m, 16 * (kGemmThreads / 64));
  const int64_t cap = (int64_t)num_cus() * (D > 128 ? 1 : 2);
  const int64_t grid = tiles < cap ? tiles : cap;
  const size_t lds = sizeof(float) * D * DN;
  auto kern = k_align_grad<D, T>;
  if (lds > 65536) {
    static bool attr_set = false;
    if (!attr_set) {
      HG_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds));
      attr_set = true;
    }
  }
  HG_LAUNCH("align_grad", kern, dim3((unsigned)grid, D / DN), dim3(kGemmThreads), lds, s, m, self, smap, other,
            omap, fin, view, w, base, out, scale, lambda_n, ddof, sums, lpart, loss3);
  return HG_OK;
}

template <int D, class T>
int align_impl(int64_t m, const T* H, const int32_t* overlap, const T* Href, const float* w, float lambda_n,
               float scale, float eps, int32_t ddof, float* loss3, T* dH, const T* dHbase, T* dHref, void* ws,
               size_t ws_bytes, hipStream_t s) {
  const AlignPlan p = align_plan<D>(m);
  Arena a(ws, ws_bytes);
  AlignWs<D> q;
  q.layout(a, p);
  if (!a.ok()) return fail(HG_ERR_CAPACITY, "alignment workspace needs %zu bytes, got %zu", a.used, ws_bytes);
  // (d1)
  HG_LAUNCH("align_stats", (k_align_stats<D, T>), dim3((unsigned)p.nch1, 2), dim3(kStatThreads), 0, s, m, p.rpc1, H,
            overlap, Href, q.stat);
  HG_LAUNCH("align_mean", (k_align_mean<D>), dim3(2 * D / 16), dim3(256), 0, s, m, p.nch1, ddof, eps,
            (const double*)q.stat, q.fin);
  // (d2)
  {
    auto kern = k_align_gram<D, T>;
    const size_t lds = GramLds<D, T>::kBytes;
    if (lds > 65536) {
      static bool attr_set = false;
      if (!attr_set) {
        HG_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        attr_set = true;
      }
    }
    HG_LAUNCH("align_gram", kern, dim3((unsigned)p.grid2), dim3(AShape<D>::kThreads), lds, s, m, p.rpc2, p.nchg, H,
              overlap, Href, w, (const float*)q.fin, q.gpart, q.spart);
  }
  HG_LAUNCH("align_reduce", (k_align_reduce<D>), dim3(AShape<D>::kRedGram + AShape<D>::kRedSums), dim3(256), 0, s,
            p.nchg, (const float*)q.gpart, (const double*)q.spart, q.sums, q.lpart, q.fin);
  // (d3)
  HG_TRY((launch_align_grad<D, T>(m, H, rows_list(overlap), Href, rows_contig(0), q.fin, 0, w,
                                  dHbase ? dHbase : (const T*)dH, dH, scale, lambda_n, ddof, q.sums,
                                  q.lpart, loss3, s)));
  if (dHref)
    HG_TRY((launch_align_grad<D, T>(m, Href, rows_contig(0), H, rows_list(overlap), q.fin, 1, w, nullptr, dHref,
                                    scale, lambda_n, ddof, q.sums, q.lpart, nullptr, s)));
  return HG_OK;
}

template <int D>
size_t align_ws_bytes(int64_t m) {
  Sizer z;
  AlignWs<D> w;
  w.layout(z, align_plan<D>(m));
  return z.used + 256;
}

}  // namespace

}  // namespace hg

using namespace hg;

extern "C" size_t hg_align_workspace_size(int64_t M, int32_t d) {
  if (M < 0) return 0;
  if (d == 64) return align_ws_bytes<64>(M);
  if (d == 128) return align_ws_bytes<128>(M);
  if (d == 256) return align_ws_bytes<256>(M);
  return 0;
}

extern "C" int hg_align_loss_fwd_bwd(int64_t M, int32_t d, int32_t dtype, int64_t n_rows, const void* H,
                                     const int32_t* overlap, const void* H_ref, const float* w,
                                     float lambda_n, float scale, float eps, int32_t ddof, float* loss3,
                                     void* dH, const void* dH_base, void* dH_ref, void* ws, size_t ws_bytes,
                                     void* stream) {
  if (M < 0 || n_rows < 0) return fail(HG_ERR_ARG, "negative size");
  if (!loss3) return fail(HG_ERR_ARG, "null loss3");
  if (dtype != HG_DTYPE_F32 && dtype != HG_DTYPE_BF16) return fail(HG_ERR_ARG, "dtype %d", dtype);
  if (d != 64 && d != 128 && d != 256)
    return fail(HG_ERR_UNSUPPORTED, "alignment supports d in {64, 128, 256}, got %d", d);
  if (ddof < 0) return fail(HG_ERR_ARG, "ddof < 0");
  if (!(eps >= 0.f)) return fail(HG_ERR_ARG, "eps must be >= 0");
  if (M > n_rows) return fail(HG_ERR_ARG, "M %lld > n_rows %lld", (long long)M, (long long)n_rows);
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (M == 0) return fill_f32(loss3, 0.f, 3, s);
  if (M <= ddof) return fail(HG_ERR_ARG, "M %lld <= ddof %d", (long long)M, ddof);
  if (!H || !overlap || !H_ref || !dH) return fail(HG_ERR_ARG, "null alignment argument");
  if (dtype == HG_DTYPE_BF16) {
    const bf16_t *h = (const bf16_t*)H, *r = (const bf16_t*)H_ref;
    bf16_t *dh = (bf16_t*)dH, *dr = (bf16_t*)dH_ref;
    const bf16_t* db = (const bf16_t*)dH_base;
    if (d == 64) return align_impl<64, bf16_t>(M, h, overlap, r, w, lambda_n, scale, eps, ddof, loss3, dh, db, dr, ws, ws_bytes, s);
    if (d == 128) return align_impl<128, bf16_t>(M, h, overlap, r, w, lambda_n, scale, eps, ddof, loss3, dh, db, dr, ws, ws_bytes, s);
    return align_impl<256, bf16_t>(M, h, overlap, r, w, lambda_n, scale, eps, ddof, loss3, dh, db, dr, ws, ws_bytes, s);
  }
  const float *h = (const float*)H, *r = (const float*)H_ref;
  float *dh = (float*)dH, *dr = (float*)dH_ref;
  const float* db = (const float*)dH_base;
  if (d == 64) return align_impl<64, float>(M, h, overlap, r, w, lambda_n, scale, eps, ddof, loss3, dh, db, dr, ws, ws_bytes, s);
  if (d == 128) return align_impl<128, float>(M, h, overlap, r, w, lambda_n, scale, eps, ddof, loss3, dh, db, dr, ws, ws_bytes, s);
  return align_impl<256, float>(M, h, overlap, r, w, lambda_n, scale, eps, ddof, loss3, dh, db, dr, ws, ws_bytes, s);
}

// ---- no-allocation variant -------------------------------------------------------
// The same passes with the workspace in a file-scope device array.  In host
// code `scratch` names a host-side stand-in, not device memory: its device
// address is taken with hipGetSymbolAddress once per device (each device
// holds its own copy) and only that address is passed to the kernels.  Nothing
// has to be cleared between calls.
namespace hg {
namespace {
constexpr size_t kAlignScratchBytes = size_t(48) << 20;
constexpr int kMaxDevices = 64;
__device__ __align__(256) unsigned char scratch[kAlignScratchBytes];
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

int scratch_address(void** out) {
  int dev = 0;
  HG_HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(HG_ERR_UNSUPPORTED, "device %d beyond %d", dev, kMaxDevices);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      return fail(HG_ERR_HIP, "hipGetSymbolAddress(scratch) on device %d failed: %s", dev, hipGetErrorString(e));
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return HG_OK;
}
}  // namespace
}  // namespace hg

extern "C" size_t hg_align_noalloc_scratch_size(void) { return kAlignScratchBytes; }

extern "C" int hg_align_loss_fwd_bwd_noalloc(int64_t M, int32_t d, int32_t dtype, int64_t n_rows, const void* H,
                                             const int32_t* overlap, const void* H_ref, const float* w,
                                             float lambda_n, float scale, float eps, int32_t ddof, float* loss3,
                                             void* dH, const void* dH_base, void* dH_ref, void* stream) {
  if (d != 64 && d != 128 && d != 256)
    return fail(HG_ERR_UNSUPPORTED, "alignment supports d in {64, 128, 256}, got %d", d);
  const size_t need = hg_align_workspace_size(M, d);
  if (need > kAlignScratchBytes)
    return fail(HG_ERR_CAPACITY, "alignment needs %zu bytes of scratch, the static scratch holds %zu", need,
                kAlignScratchBytes);
  void* ws = nullptr;
  HG_TRY(scratch_address(&ws));
  return hg_align_loss_fwd_bwd(M, d, dtype, n_rows, H, overlap, H_ref, w, lambda_n, scale, eps, ddof, loss3, dH,
                               dH_base, dH_ref, ws, kAlignScratchBytes, stream);
}
