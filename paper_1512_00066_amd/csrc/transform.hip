// Elementwise transforms and the Jacobi iteration (Section 4.1).
//
// Transforms (Section 3.4's user-defined transforms, here a fixed set of
// functor templates chosen by an enum): every element c of C is updated
// from the elements of A and B at the same letters; a letter of C missing
// from A or B broadcasts that operand along it (stride 0), which covers the
// listing's D["abij"] += Ei["i"] and the nested-loop example
// C["ij"] = C["ij"] / (A["i"] + B["j"]).
//
// Jacobi: x^{l+1}_i = (b_i - sum_{j != i} A_ij x^l_j) / A_ii until the
// residual b - A x is small.  One fused kernel per step forms the row sum
// once and gives both the update and the residual of the incoming iterate
// (r_i = b_i - sum_{j != i} A_ij x_j - A_ii x_i), so a step reads A once.
#include <algorithm>

#include "internal.hpp"

namespace srtc {

namespace {

struct BcastArgs {
  int64_t ext[SRTC_MAX_ORDER];  // C's extents
  int64_t sa[SRTC_MAX_ORDER];   // A's stride along C's mode q (0: broadcast)
  int64_t sb[SRTC_MAX_ORDER];
  int order;
  int64_t total;
};

template <class T, int OP>
__device__ __forceinline__ T apply(T a, T b, T c, T alpha) {
  if constexpr (OP == SRTC_TF_RECIP) return alpha / c;
  else if constexpr (OP == SRTC_TF_SCALE) return alpha * c;
  else if constexpr (OP == SRTC_TF_ADD) return c + alpha * a;
  else if constexpr (OP == SRTC_TF_FMA) return c + alpha * a * b;
  else return c / (a + b);  // SRTC_TF_DIV_SUM
}

template <class T, int OP>
__global__ void transform_dense(const T *__restrict__ A, const T *__restrict__ B, T *__restrict__ C, BcastArgs g,
                                T alpha) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < g.total; e += (int64_t)gridDim.x * blockDim.x) {
    int64_t rem = e, oa = 0, ob = 0;
    for (int q = g.order - 1; q >= 0; q--) {
      const int64_t i = rem % g.ext[q];
      rem /= g.ext[q];
      oa += i * g.sa[q];
      ob += i * g.sb[q];
    }
    const T a = A ? A[oa] : (T)0, b = B ? B[ob] : (T)0;
    C[e] = apply<T, OP>(a, b, C[e], alpha);
  }
}

template <class T, int OP>
void launch_transform(const void *A, const void *B, void *C, const BcastArgs &g, double alpha, hipStream_t s) {
  const unsigned grid = (unsigned)std::min<int64_t>((g.total + 255) / 256, 65536);
  transform_dense<T, OP><<<grid, 256, 0, s>>>((const T *)A, (const T *)B, (T *)C, g, (T)alpha);
  SRTC_LAUNCH_CHECK("transform_dense");
}

template <class T>
void transform_typed(int op, const void *A, const void *B, void *C, const BcastArgs &g, double alpha, hipStream_t s) {
  switch (op) {
    case SRTC_TF_RECIP: launch_transform<T, SRTC_TF_RECIP>(A, B, C, g, alpha, s); break;
    case SRTC_TF_SCALE: launch_transform<T, SRTC_TF_SCALE>(A, B, C, g, alpha, s); break;
    case SRTC_TF_ADD: launch_transform<T, SRTC_TF_ADD>(A, B, C, g, alpha, s); break;
    case SRTC_TF_FMA: launch_transform<T, SRTC_TF_FMA>(A, B, C, g, alpha, s); break;
    case SRTC_TF_DIV_SUM: launch_transform<T, SRTC_TF_DIV_SUM>(A, B, C, g, alpha, s); break;
    default: fail(SRTC_ERR_ARG, "unknown transform");
  }
}

// ------------------------------------------------------------- Jacobi --

// The diagonal of each row (0 where missing), eight lanes per row; flags[0]
// set if any is 0, flags[1] if some entry lies 2^15 or more columns from its
// row.
template <class T>
__global__ void __launch_bounds__(256) jacobi_diag(const int64_t *__restrict__ rp, const int32_t *__restrict__ col,
                                                   const T *__restrict__ val, int64_t n, T *__restrict__ d,
                                                   int64_t *flags) {
  constexpr int G = 8;
  const int sub = lane_id() % G;
  const int64_t ngrp = (int64_t)gridDim.x * blockDim.x / G;
  bool zero = false, far = false;
  for (int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / G; i < n; i += ngrp) {
    T dii = 0;
    for (int64_t p = rp[i] + sub; p < rp[i + 1]; p += G) {
      const int64_t o = col[p] - i;
      if (o == 0) dii += val[p];
      far |= o < -32768 || o > 32767;
    }
#pragma unroll
    for (int w = G / 2; w >= 1; w >>= 1) dii += __shfl_xor(dii, w, G);
    if (sub == 0) d[i] = dii;
    zero |= dii == (T)0;
  }
  if (__any(zero) && lane_id() == 0) atomicOr((unsigned long long *)&flags[0], 1ull);
  if (__any(far) && lane_id() == 0) atomicOr((unsigned long long *)&flags[1], 1ull);
}

// Slices of 64 rows, one per lane of a wave, stored entry by entry: entry k of
// the slice's rows at (start + k) 64 .. + 63, start = the scan of the slices'
// longest rows.
__global__ void __launch_bounds__(256) slice_widths(const int64_t *__restrict__ rp, int64_t n, int64_t slices,
                                                    int64_t *__restrict__ width) {
  const int64_t nw = (int64_t)gridDim.x * blockDim.x / WAVE;
  for (int64_t q = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / WAVE; q < slices; q += nw) {
    const int64_t i = q * WAVE + lane_id();
    int64_t len = i < n ? rp[i + 1] - rp[i] : 0;
#pragma unroll
    for (int w = WAVE / 2; w >= 1; w >>= 1) len = max(len, (int64_t)__shfl_xor((long long)len, w, WAVE));
    if (lane_id() == 0) width[q] = len;
  }
}

// Columns as offsets from the row in C; rows shorter than their slice are
// filled up with value 0 at offset 0 (the diagonal, which steps skip).  A wave
// reads 16 consecutive entries of four rows at a time and turns them over
// through LDS, so that reads and writes are whole lines.  Bound by its bytes:
// stencil 100^3, fp64, 0.58 GB in 131 us (4.4 TB/s); with each lane reading a row of
// its own 897 us, as much as the steps gain by the copy in 20 updates.
template <class T, class C>
__global__ void __launch_bounds__(256) slice_fill(const int64_t *__restrict__ rp, const int32_t *__restrict__ col,
                                                  const T *__restrict__ val, int64_t n, int64_t slices,
                                                  const int64_t *__restrict__ start, C *__restrict__ off,
                                                  T *__restrict__ sval) {
  constexpr int KT = 16, RPL = WAVE / KT, WPB = 256 / WAVE;
  __shared__ T tv[WPB][WAVE][KT + 1];
  __shared__ C to[WPB][WAVE][KT + 1];
  const int l = lane_id(), wv = threadIdx.x / WAVE, kl = l % KT, rl = l / KT;
  const int64_t nw = (int64_t)gridDim.x * WPB;
  for (int64_t q = (int64_t)blockIdx.x * WPB + wv; q < slices; q += nw) {
    const int64_t i0 = q * WAVE, i = i0 + l;
    const int64_t a = i < n ? rp[i] : 0, len = i < n ? rp[i + 1] - a : 0;
    const int64_t s0 = start[q], w = start[q + 1] - s0;
    for (int64_t k0 = 0; k0 < w; k0 += KT) {
      T v[KT];
      int32_t c[KT];
#pragma unroll
      for (int u = 0; u < KT; u++) {
        const int r = u * RPL + rl;
        const int64_t p = __shfl((long long)a, r, WAVE) + k0 + kl;
        const bool in = k0 + kl < __shfl((long long)len, r, WAVE);
        v[u] = in ? val[p] : (T)0;
        c[u] = in ? col[p] : (int32_t)(i0 + r);
      }
#pragma unroll
      for (int u = 0; u < KT; u++) {
        const int r = u * RPL + rl;
        tv[wv][r][kl] = v[u];
        to[wv][r][kl] = (C)(c[u] - (i0 + r));
      }
      wave_sync();
      const int kn = (int)min((int64_t)KT, w - k0);
      for (int k = 0; k < kn; k++) {
        off[(s0 + k0 + k) * WAVE + l] = to[wv][l][k];
        sval[(s0 + k0 + k) * WAVE + l] = tv[wv][l][k];
      }
      wave_sync();
    }
  }
}

// Sum of part[0..nb) in a fixed order by a block of BS threads (every thread
// gets it).
template <int BS> __device__ __forceinline__ double sum_parts(const double *__restrict__ part, int64_t nb) {
  __shared__ double red[BS / WAVE];
  double t = 0.0;
  for (int64_t q = threadIdx.x; q < nb; q += BS) t += part[q];
  t = wave_sum(t);
  if (lane_id() == 0) red[threadIdx.x / WAVE] = t;
  __syncthreads();
  double u = 0.0;
#pragma unroll
  for (int w = 0; w < BS / WAVE; w++) u += red[w];
  return u;
}

// Whether step j of a run of steps stops before it starts: for j > 0 every
// block adds up the partial sums of step j - 1 itself (8 KB from L2, the same
// order everywhere) and stops if that iterate, l = st->base + j - 1, meets
// the tolerance; block 0 records it.  (A kernel of its own for that sum took
// one block 17 us and a launch per step.)  Later steps see st->done.
// Block 0 may set st->done while other blocks read it, so a block reads it
// once, in thread 0, and all its waves take that value from LDS, after a
// barrier that none of them can leave before.  Waves reading it for themselves
// could disagree: one that saw the flag would leave, and the others would add
// up a sum without its part and might run the step, over the iterate that is
// the answer.  As it is, a block that reads the flag early and one that reads
// it late both stop, the first by its sum.
template <int BS>
__device__ __forceinline__ bool step_stops(const double *__restrict__ part_in, int j, JacobiState *st, double tol2) {
  __shared__ int32_t stopped;
  if (threadIdx.x == 0) stopped = st->done;
  const double u = sum_parts<BS>(part_in, j > 0 ? gridDim.x : 0);  // its barrier publishes `stopped`
  if (stopped) return true;
  const int64_t l = st->base + j - 1;
  if (j == 0 || l < 1 || u > tol2 || u != u) return false;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->rsq = u;
    st->iter = l;
    st->done = 1;
  }
  return true;
}

// The block's sum of rr to part_out[blockIdx.x].
template <int BS> __device__ __forceinline__ void put_part(double rr, double *part_out) {
  __shared__ double red[BS / WAVE];
  rr = wave_sum(rr);
  if (lane_id() == 0) red[threadIdx.x / WAVE] = rr;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < BS / WAVE; w++) t += red[w];
    part_out[blockIdx.x] = t;
  }
}

// Block id renumbered so that blocks of one XCD (id mod 8) are neighbours.
__device__ __forceinline__ int xcd_block() {
  const int nb = gridDim.x;
  return nb % 8 == 0 ? (int)(blockIdx.x % 8) * (nb / 8) + (int)(blockIdx.x / 8) : (int)blockIdx.x;
}

// Step j of a run of steps (a replayed graph): x_out = (b - R x_in) / d and
// the block's partial sum of r_i^2 for r = b - A x_in (fp64).  G lanes per
// row on the CSR itself; for small systems and uneven rows.
constexpr int JAC_BS = 512;
template <class T, int G>
__global__ void __launch_bounds__(JAC_BS) jacobi_step(const int64_t *__restrict__ rp, const int32_t *__restrict__ col,
                                                      const T *__restrict__ val, const T *__restrict__ d,
                                                      const T *__restrict__ b, const T *__restrict__ x_in,
                                                      T *__restrict__ x_out, int64_t n, double *__restrict__ part_out,
                                                      const double *__restrict__ part_in, int j, JacobiState *st,
                                                      double tol2) {
  if (step_stops<JAC_BS>(part_in, j, st, tol2)) return;
  const int sub = lane_id() % G;
  const int64_t grp = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / G;
  const int64_t ngrp = ((int64_t)gridDim.x * blockDim.x) / G;
  double rr = 0.0;
  // the G lanes of a row are one aligned lane group, so the shuffles below
  // stay inside lanes that take the same trips
  for (int64_t i = grp; i < n; i += ngrp) {
    // the row's own terms first, so their loads overlap the row sum
    const double bi = sub == 0 ? (double)b[i] : 0.0, di = sub == 0 ? (double)d[i] : 0.0;
    const double xi = sub == 0 ? (double)x_in[i] : 0.0;
    const int64_t p1 = rp[i + 1];
    double s = 0.0;
    // four entries per lane per pass, all loads issued before the sums;
    // padding uses column i, which the diagonal test skips
    for (int64_t p = rp[i] + sub; p < p1; p += 4 * G) {
      int32_t c[4];
      T v[4];
#pragma unroll
      for (int u = 0; u < 4; u++) {
        const bool ok = p + u * G < p1;
        c[u] = ok ? col[p + u * G] : (int32_t)i;
        v[u] = ok ? val[p + u * G] : (T)0;
      }
      double xv[4];
#pragma unroll
      for (int u = 0; u < 4; u++) xv[u] = c[u] != i ? (double)x_in[c[u]] : 0.0;
#pragma unroll
      for (int u = 0; u < 4; u++) s += (double)v[u] * xv[u];
    }
#pragma unroll
    for (int w = G / 2; w >= 1; w >>= 1) s += __shfl_xor(s, w, G);
    if (sub == 0) {
      x_out[i] = (T)((bi - s) / di);
      const double r = bi - s - di * xi;
      rr += r * r;
    }
  }
  put_part<JAC_BS>(rr, part_out);
}

// The same step on the slices: one row per lane, so every load of A is one
// contiguous run per wave and the row sum needs no shuffles.  Bound by the
// stream of A (10 bytes per fp64 entry with 16-bit offsets, 12 with 32-bit
// ones); on the CSR, eight lanes per row, about 25 vector instructions per
// entry bound it instead.  Blocks of one XCD take neighbouring slices, so its
// L2 holds its part of x_in.  Stencil 100^3 (26.5 M nonzeros), per update:
// fp64 103 us before (83 the step, 17 the separate sum), 61.6 now (100 on the
// CSR); fp32 45.9 (69 on the CSR); stencil 50^3 fp64 14.9 (16.7).
template <class T, class C>
__global__ void __launch_bounds__(JAC_BS, 8) jacobi_slices(const int64_t *__restrict__ start, const C *__restrict__ off,
                                                        const T *__restrict__ sval, const T *__restrict__ d,
                                                        const T *__restrict__ b, const T *__restrict__ x_in,
                                                        T *__restrict__ x_out, int64_t n, int64_t slices,
                                                        double *__restrict__ part_out,
                                                        const double *__restrict__ part_in, int j, JacobiState *st,
                                                        double tol2) {
  constexpr int U = 7;  // entries in flight per lane: 64 registers, eight waves per SIMD
  if (step_stops<JAC_BS>(part_in, j, st, tol2)) return;
  const int l = lane_id();
  const int64_t nw = (int64_t)gridDim.x * (JAC_BS / WAVE);
  const int64_t w0 = (int64_t)xcd_block() * (JAC_BS / WAVE) + threadIdx.x / WAVE;
  double rr = 0.0;
  for (int64_t q = w0; q < slices; q += nw) {
    const int64_t i = q * WAVE + l;
    const int64_t s0 = start[q];
    const int w = (int)(start[q + 1] - s0);
    const bool in = i < n;
    const double bi = in ? (double)b[i] : 0.0, di = in ? (double)d[i] : 1.0, xi = in ? (double)x_in[i] : 0.0;
    const C *po = off + s0 * WAVE + l;
    const T *pv = sval + s0 * WAVE + l;
    const T *px = x_in + i;
    double s = 0.0;
    for (int k = 0; k < w; k += U) {
      C o[U];
      T v[U];
#pragma unroll
      for (int u = 0; u < U; u++) {
        o[u] = k + u < w ? po[u * WAVE] : (C)0;
        v[u] = k + u < w ? pv[u * WAVE] : (T)0;
      }
      po += U * WAVE;
      pv += U * WAVE;
      double xv[U];
#pragma unroll
      for (int u = 0; u < U; u++) xv[u] = o[u] != 0 ? (double)px[o[u]] : 0.0;
#pragma unroll
      for (int u = 0; u < U; u++) s += (double)v[u] * xv[u];
    }
    if (in) {
      x_out[i] = (T)((bi - s) / di);
      const double r = bi - s - di * xi;
      rr += r * r;
    }
  }
  put_part<JAC_BS>(rr, part_out);
}

// The end of a run of k steps: the residual of the last step's incoming
// iterate x^l, l = st->base + k - 1 (one block of 256 threads).  Stops the
// iteration when l >= 1 and |r|^2 <= tol2, else moves on to x^{base + k}.
__global__ void __launch_bounds__(256) jacobi_reduce(const double *__restrict__ part, int64_t nb, int k,
                                                     JacobiState *__restrict__ st, double tol2) {
  if (st->done) return;  // uniform over the block
  const double u = sum_parts<256>(part, nb);
  if (threadIdx.x == 0) {
    const int64_t l = st->base + k - 1;
    st->rsq = u;
    if (l >= 1 && u <= tol2) {
      st->iter = l;
      st->done = 1;
    } else {
      st->base += k;
      st->iter = st->base;
    }
  }
}

}  // namespace

void transform_dense_call(int op, int dt, double alpha, const int64_t *cext, int order, const void *A,
                          const int64_t *sa, const void *B, const int64_t *sb, void *C, hipStream_t s) {
  BcastArgs g{};
  g.order = order;
  g.total = 1;
  for (int q = 0; q < order; q++) {
    g.ext[q] = cext[q];
    g.sa[q] = sa[q];
    g.sb[q] = sb[q];
    g.total *= cext[q];
  }
  if (g.total == 0) return;
  if (dt == SRTC_F64) transform_typed<double>(op, A, B, C, g, alpha, s);
  else if (dt == SRTC_F32) transform_typed<float>(op, A, B, C, g, alpha, s);
  else fail(SRTC_ERR_DTYPE, "transforms are defined for F64 and F32");
}

// Fewest slices of 64 rows that the steps take one row per lane: fewer leave
// CUs without a wave (stencil 25^3, 244 slices: 15.3 us per update against
// 8.9 with eight lanes per row; 50^3, 1,954: 14.8 against 16.7).  The copy is
// made before the number of updates is known: it costs one update at this size
// and two at 100^3 (131 us), where it pays from the fourth on.
constexpr int64_t JAC_SLICES_MIN = 1024;

void JacobiPlan::build(Ctx *c, int dt_, const CsrView &A_, hipStream_t s) {
  ctx = c;
  dt = dt_;
  A = A_;
  const int64_t n = A.m;
  const double avg = n > 0 ? (double)A.nnz / (double)n : 1.0;
  // about four nonzeros per lane: more rows in flight per wave hides the
  // dependent loads of a row (row pointer, then columns, then x)
  G = 4;
  while (G < 64 && 4 * G < avg) G <<= 1;
  const size_t es = dtype_size(dt);
  dbuf = Buf(c, es * (size_t)std::max<int64_t>(n, 1));
  // the slices' starts, their end, and the two flags: one read has the last three
  const int64_t slices_ = (n + WAVE - 1) / WAVE;
  start = Buf(c, sizeof(int64_t) * (size_t)(slices_ + 3));
  int64_t *flags = start.as<int64_t>() + slices_ + 1;
  fill_i64(flags - 1, 3, 0, s);
  // slices for systems that fill the chip with one row per lane
  const bool want = slices_ >= JAC_SLICES_MIN;
  int64_t h[3] = {0, 0, 0};
  if (n > 0) {
    const unsigned g = (unsigned)std::max<int64_t>(1, std::min<int64_t>((n * 8 + 255) / 256, 8192));
    if (dt == SRTC_F64)
      jacobi_diag<double><<<g, 256, 0, s>>>(A.rowptr, A.col, (const double *)A.val, n, dbuf.as<double>(), flags);
    else
      jacobi_diag<float><<<g, 256, 0, s>>>(A.rowptr, A.col, (const float *)A.val, n, dbuf.as<float>(), flags);
    SRTC_LAUNCH_CHECK("jacobi_diag");
    if (want) {
      Buf width(c, sizeof(int64_t) * (size_t)slices_);
      slice_widths<<<(unsigned)std::min<int64_t>((slices_ + 3) / 4, 8192), 256, 0, s>>>(A.rowptr, n, slices_,
                                                                                       width.as<int64_t>());
      SRTC_LAUNCH_CHECK("slice_widths");
      excl_scan_i64(c, width.as<int64_t>(), start.as<int64_t>(), slices_, s);
    }
    read_to_host(c, h, flags - 1, sizeof(h), s);
    if (h[1]) fail(SRTC_ERR_ARG, "Jacobi needs a nonzero diagonal entry in every row");
  }
  // rows of much the same length: at most a quarter of padding; and room for
  // the copy
  const int64_t cells = h[0] * WAVE;
  if (want && 4 * cells <= 5 * A.nnz) {
    wide = h[2] != 0;
    try {
      off = Buf(c, (wide ? sizeof(int32_t) : sizeof(int16_t)) * (size_t)cells);
      sval = Buf(c, es * (size_t)cells);
      slices = slices_;
    } catch (const Error &e) {
      if (e.st != SRTC_ERR_OOM) throw;
      off = Buf();
      sval = Buf();
    }
  }
  if (slices > 0) {
    ProfScope ps(c, "jacobi.slice_copy", (4.0 + es) * (double)A.nnz + ((wide ? 4.0 : 2.0) + es) * (double)cells, s);
    const unsigned g = (unsigned)std::min<int64_t>((slices + 3) / 4, 16384);
    if (dt == SRTC_F64 && wide)
      slice_fill<double, int32_t><<<g, 256, 0, s>>>(A.rowptr, A.col, (const double *)A.val, n, slices,
                                                    start.as<int64_t>(), off.as<int32_t>(), sval.as<double>());
    else if (dt == SRTC_F64)
      slice_fill<double, int16_t><<<g, 256, 0, s>>>(A.rowptr, A.col, (const double *)A.val, n, slices,
                                                    start.as<int64_t>(), off.as<int16_t>(), sval.as<double>());
    else if (wide)
      slice_fill<float, int32_t><<<g, 256, 0, s>>>(A.rowptr, A.col, (const float *)A.val, n, slices,
                                                   start.as<int64_t>(), off.as<int32_t>(), sval.as<float>());
    else
      slice_fill<float, int16_t><<<g, 256, 0, s>>>(A.rowptr, A.col, (const float *)A.val, n, slices,
                                                   start.as<int64_t>(), off.as<int16_t>(), sval.as<float>());
    SRTC_LAUNCH_CHECK("slice_fill");
  }
  // all blocks resident at once, a multiple of the eight XCDs where there are
  // that many
  const int64_t threads = slices > 0 ? slices * WAVE : n * G;
  grid = (int)std::max<int64_t>(1, std::min<int64_t>((threads + JAC_BS - 1) / JAC_BS,
                                                     (int64_t)c->num_cus * (2048 / JAC_BS)));
  if (grid > 8) grid -= grid % 8;
  part = Buf(c, sizeof(double) * (size_t)(2 * grid));
}

struct StepCall {
  const JacobiPlan &pl;
  const void *b, *x_in;
  void *x_out;
  JacobiState *st;
  double tol2;
  int j;
  hipStream_t s;
};

template <class T, int G> static void step_typed(const StepCall &q) {
  const JacobiPlan &pl = q.pl;
  double *out = pl.part.as<double>() + (int64_t)(q.j & 1) * pl.grid;
  const double *in = pl.part.as<double>() + (int64_t)((q.j & 1) ^ 1) * pl.grid;
  if (pl.slices > 0 && pl.wide)
    jacobi_slices<T, int32_t><<<pl.grid, JAC_BS, 0, q.s>>>(pl.start.as<int64_t>(), pl.off.as<int32_t>(),
                                                           pl.sval.as<T>(), pl.dbuf.as<T>(), (const T *)q.b,
                                                           (const T *)q.x_in, (T *)q.x_out, pl.A.m, pl.slices, out,
                                                           in, q.j, q.st, q.tol2);
  else if (pl.slices > 0)
    jacobi_slices<T, int16_t><<<pl.grid, JAC_BS, 0, q.s>>>(pl.start.as<int64_t>(), pl.off.as<int16_t>(),
                                                           pl.sval.as<T>(), pl.dbuf.as<T>(), (const T *)q.b,
                                                           (const T *)q.x_in, (T *)q.x_out, pl.A.m, pl.slices, out,
                                                           in, q.j, q.st, q.tol2);
  else
    jacobi_step<T, G><<<pl.grid, JAC_BS, 0, q.s>>>(pl.A.rowptr, pl.A.col, (const T *)pl.A.val, pl.dbuf.as<T>(),
                                                   (const T *)q.b, (const T *)q.x_in, (T *)q.x_out, pl.A.m, out, in,
                                                   q.j, q.st, q.tol2);
  SRTC_LAUNCH_CHECK("jacobi_step");
}

template <class T> static void step_width(const StepCall &q) {
  switch (q.pl.G) {
    case 4: step_typed<T, 4>(q); break;
    case 8: step_typed<T, 8>(q); break;
    case 16: step_typed<T, 16>(q); break;
    case 32: step_typed<T, 32>(q); break;
    default: step_typed<T, 64>(q); break;
  }
}

void jacobi_step_call(const JacobiPlan &pl, const void *b, const void *x_in, void *x_out, JacobiState *st,
                      double tol2, int j, bool last, hipStream_t s) {
  ProfScope ps(pl.ctx, "jacobi.step",
               (4.0 + (double)dtype_size(pl.dt)) * (double)pl.A.nnz + 8.0 * (double)(pl.A.m + 1) +
                   4.0 * (double)dtype_size(pl.dt) * (double)pl.A.m,
               s);
  const StepCall q{pl, b, x_in, x_out, st, tol2, j, s};
  if (pl.dt == SRTC_F64) step_width<double>(q);
  else step_width<float>(q);
  if (last) {
    jacobi_reduce<<<1, 256, 0, s>>>(pl.part.as<double>() + (int64_t)(j & 1) * pl.grid, pl.grid, j + 1, st, tol2);
    SRTC_LAUNCH_CHECK("jacobi_reduce");
  }
}

}  // namespace srtc
