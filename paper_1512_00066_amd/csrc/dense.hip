// Dense (+,x) tiles on the matrix cores, and dense mode permutation.
//
// Dense operands appear where a contraction has no sparsity to exploit; the
// paper's dense baseline runs such products as BLAS GEMM and notes that small
// dense blocks inside sparse data are worth exploiting (Section 6).  Only the
// (+,x) semiring maps onto MFMA; tropical, boolean and (max,x) products have
// no matrix-core form.
//
//   fp64: V_MFMA_F64_16X16X4_F64, fp64 accumulation.
//   fp32: V_MFMA_F32_16X16X4_F32, with the fp32 accumulators added into fp64
//         registers every 128 k-terms, so a dot product of any length keeps
//         the relative error of an fp32 sum of at most 128 terms.
#include <algorithm>
#include <type_traits>

#include "internal.hpp"

namespace srtc {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

// One tile of C per block: WM x WN waves, each forming NTM x NTN MFMA 16x16
// tiles, k taken 128 bytes of A's row (16 fp64 or 32 fp32 terms) at a time
// through two LDS buffers, one barrier per k-tile.  Bound by the matrix
// cores: fp64 8192^3 47 -> 72 TFLOP/s of 78.6, fp32 8192^3 76 -> 130 of 157
// (single-entry loads and LDS accesses, one tile of 128 x 128 per block and
// accumulators spilled before).  The 16-byte global loads run two k-tiles
// ahead in registers: with one tile of distance the matrix cores waited for
// them (67 and 117 TFLOP/s; a lone block per CU 48 and 86).
// Which k a lane group multiplies in a step, and which column a lane of a
// 16x16 tile stands for, are free as long as both operands (and the stores)
// agree: lane group g takes k = g VEC .. g VEC + VEC - 1 of a 4 VEC deep step,
// so a fragment of A is one 16-byte LDS read, and a lane's tiles are adjacent
// columns, so fragments of B and C's stores are 16 bytes too.  A's LDS rows
// are 144 bytes apart (8 lanes of a read touch 64 different banks).
// Global loads need only their element's alignment, whatever the row length.
// The main loop has no branch (the compiler copied every accumulator at each
// join): rows past M and vectors past N are clamped into the matrix (their
// results are not stored; a vector that crosses N, possible when N is no
// multiple of VEC, is shifted into place), loads past the last whole k-tile
// repeat it, and the k remainder follows the loop, entry by entry.
// Batch z of a strided batch (grid z, grid-stride over batches) multiplies
// A + z M K by B + z K N into C + z M N.  With W given, block row y handles
// the k range [y kchunk, (y + 1) kchunk) and stores its fp64 partial sums to
// W + (z gridDim.y + y) M N; gemm_combine adds them in order.
template <class T> struct GemmVec {
  static constexpr int N = 16 / (int)sizeof(T);
  typedef T lds __attribute__((ext_vector_type(16 / sizeof(T))));
  typedef T glb __attribute__((ext_vector_type(16 / sizeof(T)), aligned(sizeof(T))));
};
template <class T, int NTM, int NTN, int WM, int WN> struct GemmTile {
  static constexpr int VEC = GemmVec<T>::N;
  static constexpr int BK = 128 / (int)sizeof(T);
  static constexpr int TM = NTM * 16 * WM, TN = NTN * 16 * WN;
  static constexpr int THREADS = WAVE * WM * WN;
  static constexpr int SA = BK + VEC, SB = TN + VEC;
};

// Off: 32-bit byte offsets into a row tile where they suffice (one register
// per address, the row and k advance in scalar registers), else 64-bit.
// SHIFT: N is no multiple of VEC.  N is at least VEC.
template <class T, int NTM, int NTN, int WM, int WN, class Off, bool SHIFT>
__global__ void __launch_bounds__(WAVE *WM *WN, 2) gemm_mfma(const T *__restrict__ A0, const T *__restrict__ B0,
                                                    T *__restrict__ C0, double *__restrict__ W, int64_t M, int64_t N,
                                                    int64_t K, int64_t kchunk, int accumulate, int64_t batch) {
  using G = GemmTile<T, NTM, NTN, WM, WN>;
  constexpr int THREADS = G::THREADS;
  constexpr int VEC = G::VEC, BK = G::BK, TM = G::TM, TN = G::TN, SA = G::SA, SB = G::SB;
  constexpr int CV = NTN < VEC ? NTN : VEC;        // adjacent columns of a lane
  constexpr int RA = THREADS / 8, LA = TM / RA;    // A rows per round of loads, rounds
  constexpr int VB = TN / VEC, RB = THREADS / VB, LB = BK / RB;  // the same for B (VB vectors per row)
  static_assert(TM % RA == 0 && THREADS % VB == 0 && BK % RB == 0, "whole rounds of loads");
  using VL = typename GemmVec<T>::lds;
  using VG = typename GemmVec<T>::glb;
  typedef T VC __attribute__((ext_vector_type(CV)));
  typedef T VCG __attribute__((ext_vector_type(CV), aligned(sizeof(T))));
  using Acc = std::conditional_t<sizeof(T) == 8, v4d, v4f>;
  __shared__ __align__(16) T As[2][TM * SA];
  __shared__ __align__(16) T Bs[2][BK * SB];
  const int t = threadIdx.x, w = t / WAVE, l = lane_id();
  const int wm = (w / WN) * NTM * 16, wn = (w % WN) * NTN * 16;
  const int lr = l % 16, lg = l / 16;
  const int64_t tm = (M + TM - 1) / TM;
  const int64_t m0 = blockIdx.x % tm * TM, n0 = blockIdx.x / tm * TN;
  const int64_t kb = (int64_t)blockIdx.y * kchunk, ke = min(K, kb + kchunk);
  for (int64_t z = blockIdx.z; z < batch; z += gridDim.z) {
    const T *__restrict__ A = A0 + z * M * K;
    const T *__restrict__ B = B0 + z * K * N;
    // a thread's bytes from the tile's first row of A, and from B's row k0
    const T *__restrict__ Am = A + m0 * K;
    Off oa[LA];
#pragma unroll
    for (int i = 0; i < LA; i++)
      oa[i] = (Off)(((Off)min((int64_t)(t / 8 + RA * i), M - 1 - m0) * (Off)K + (t % 8) * VEC) * sizeof(T));
    const int64_t bn = n0 + (t % VB) * VEC, bc = min(bn, N - VEC);
    const int sh = (int)min(bn - bc, (int64_t)VEC);  // VEC: past the matrix, never stored
    const Off ob = (Off)(((Off)(t / VB) * (Off)N + (Off)bc) * sizeof(T));
    auto at_a = [&](int i, int64_t k0) { return (const T *)((const char *)(Am + k0) + oa[i]); };
    auto at_b = [&](int64_t k) { return (const T *)((const char *)(B + k * N) + ob); };
    struct Regs {
      VL a[LA], b[LB];
    };
    const int64_t nt = (ke - kb) / BK;  // whole k-tiles
    auto fetch = [&](Regs &r, int64_t tile) {
      const int64_t k0 = kb + min(tile, nt - 1) * BK;
#pragma unroll
      for (int i = 0; i < LA; i++) r.a[i] = *(const VG *)at_a(i, k0);
#pragma unroll
      for (int i = 0; i < LB; i++) r.b[i] = *(const VG *)at_b(k0 + i * RB);
    };
    // the terms from k0 on, fewer than a tile; zero beyond
    auto fetch_rest = [&](Regs &r, int64_t k0) {
      const int64_t ka = k0 + (t % 8) * VEC;
#pragma unroll
      for (int i = 0; i < LA; i++) {
        r.a[i] = VL{};
        if (ka + VEC <= ke) {
          r.a[i] = *(const VG *)at_a(i, k0);
        } else {
#pragma unroll
          for (int e = 0; e < VEC - 1; e++)
            if (ka + e < ke) r.a[i][e] = at_a(i, k0)[e];
        }
      }
#pragma unroll
      for (int i = 0; i < LB; i++) {
        r.b[i] = VL{};
        if (k0 + t / VB + i * RB < ke) r.b[i] = *(const VG *)at_b(k0 + i * RB);
      }
    };
    auto stage = [&](const Regs &r, int buf) {
#pragma unroll
      for (int i = 0; i < LA; i++) *(VL *)&As[buf][(t / 8 + RA * i) * SA + (t % 8) * VEC] = r.a[i];
#pragma unroll
      for (int i = 0; i < LB; i++) {
        VL v = r.b[i];
        if constexpr (SHIFT) {
#pragma unroll
          for (int e = 0; e < VEC; e++)
#pragma unroll
            for (int d = 1; e + d < VEC; d++) v[e] = sh == d ? r.b[i][e + d] : v[e];
        }
        *(VL *)&Bs[buf][(t / VB + i * RB) * SB + (t % VB) * VEC] = v;
      }
    };
    Acc acc[NTM][NTN];
    double acc64[sizeof(T) == 4 ? NTM : 1][NTN][4];
#pragma unroll
    for (int a = 0; a < NTM; a++)
#pragma unroll
      for (int b = 0; b < NTN; b++)
#pragma unroll
        for (int q = 0; q < 4; q++) {
          acc[a][b][q] = 0;
          if constexpr (sizeof(T) == 4) acc64[a][b][q] = 0.0;
        }
    auto multiply = [&](int buf) {
#pragma unroll
      for (int s = 0; s < BK / (4 * VEC); s++) {
        VL av[NTM];
#pragma unroll
        for (int a = 0; a < NTM; a++)
          av[a] = *(const VL *)&As[buf][(wm + a * 16 + lr) * SA + s * 4 * VEC + lg * VEC];
#pragma unroll
        for (int e = 0; e < VEC; e++) {
          VC bv[NTN / CV];
#pragma unroll
          for (int h = 0; h < NTN / CV; h++)
            bv[h] = *(const VC *)&Bs[buf][(s * 4 * VEC + lg * VEC + e) * SB + wn + h * 16 * CV + lr * CV];
#pragma unroll
          for (int a = 0; a < NTM; a++)
#pragma unroll
            for (int b = 0; b < NTN; b++) {
              if constexpr (sizeof(T) == 8)
                acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a][e], bv[b / CV][b % CV], acc[a][b], 0, 0, 0);
              else
                acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[a][e], bv[b / CV][b % CV], acc[a][b], 0, 0, 0);
            }
        }
      }
    };
    auto flush = [&]() {
      if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int a = 0; a < NTM; a++)
#pragma unroll
          for (int b = 0; b < NTN; b++)
#pragma unroll
            for (int q = 0; q < 4; q++) {
              acc64[a][b][q] += (double)acc[a][b][q];
              acc[a][b][q] = 0.f;
            }
      }
    };
    // UN tiles per round (128 k-terms for fp32, then the flush).  At its head
    // tile i is in buffer 0, i + 1 in r1 and i + 2 in r0; a buffer is refilled
    // one barrier after its last read.
    constexpr int UN = sizeof(T) == 4 ? 128 / BK : 2;
    Regs r0, r1;
    if (nt > 0) {
      fetch(r0, 0);
      if (TM > 64 || nt > 1) fetch(r1, 1);  // (the small tile's products may be short)
      stage(r0, 0);
      if (TM > 64 || nt > 2) fetch(r0, 2);
    }
    __syncthreads();
    int64_t i = 0;
    for (; i + UN <= nt; i += UN) {
#pragma unroll
      for (int u = 0; u < UN; u += 2) {
        multiply(0);
        stage(r1, 1);
        fetch(r1, i + u + 3);
        __syncthreads();
        multiply(1);
        stage(r0, 0);
        fetch(r0, i + u + 4);
        __syncthreads();
      }
      flush();
    }
    // up to UN - 1 more tiles and the rest: fewer than 128 terms in fp32
    if (i < nt) {
      multiply(0);
      if (i + 1 < nt) {
        stage(r1, 1);
        __syncthreads();
        multiply(1);
        if (i + 2 < nt) {
          stage(r0, 0);
          __syncthreads();
          multiply(0);
        }
      }
    }
    if (kb + nt * BK < ke) {
      fetch_rest(r0, kb + nt * BK);
      __syncthreads();
      stage(r0, 0);
      __syncthreads();
      multiply(0);
    }
    // output layout of a 16x16 MFMA tile, lane l, accumulator q:
    //   fp32 (16x16x4 f32): row 4*(l/16) + q
    //   fp64 (16x16x4 f64): row 4*q + l/16
    // and tile h CV + e, lane column l % 16 holds column h 16 CV + (l % 16) CV + e
    T *__restrict__ C = C0 + z * M * N;
    double *__restrict__ P = W ? W + (z * gridDim.y + blockIdx.y) * M * N : nullptr;
#pragma unroll
    for (int a = 0; a < NTM; a++)
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const int64_t gm = m0 + wm + a * 16 + (sizeof(T) == 8 ? 4 * q + lg : 4 * lg + q);
        if (gm >= M) continue;
#pragma unroll
        for (int h = 0; h < NTN / CV; h++) {
          const int64_t gn = n0 + wn + h * 16 * CV + lr * CV;
          double v[CV];
#pragma unroll
          for (int e = 0; e < CV; e++) {
            v[e] = (double)acc[a][h * CV + e][q];
            if constexpr (sizeof(T) == 4) v[e] += acc64[a][h * CV + e][q];
          }
          if (P) {
#pragma unroll
            for (int e = 0; e < CV; e++)
              if (gn + e < N) P[gm * N + gn + e] = v[e];
          } else if (!accumulate && gn + CV <= N) {
            VCG o;
#pragma unroll
            for (int e = 0; e < CV; e++) o[e] = (T)v[e];
            *(VCG *)(C + gm * N + gn) = o;
          } else {
#pragma unroll
            for (int e = 0; e < CV; e++)
              if (gn + e < N) C[gm * N + gn + e] = (T)(accumulate ? v[e] + (double)C[gm * N + gn + e] : v[e]);
          }
        }
      }
    __syncthreads();  // the next batch restages As and Bs
  }
}

// Products with fewer columns than a vector: one wave per row of C, exact
// products summed in fp64.
template <class T>
__global__ void __launch_bounds__(256) gemm_narrow(const T *__restrict__ A, const T *__restrict__ B,
                                                   T *__restrict__ C, int64_t M, int N, int64_t K, int accumulate,
                                                   int64_t batch) {
  constexpr int MAXN = GemmVec<T>::N - 1;
  const int64_t wid = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / WAVE;
  const int64_t nw = ((int64_t)gridDim.x * blockDim.x) / WAVE;
  for (int64_t r = wid; r < batch * M; r += nw) {
    const T *a = A + r * K, *b = B + r / M * K * N;
    double acc[MAXN] = {};
    for (int64_t k = lane_id(); k < K; k += WAVE)
#pragma unroll
      for (int n = 0; n < MAXN; n++)
        if (n < N) acc[n] += (double)a[k] * (double)b[k * N + n];
#pragma unroll
    for (int n = 0; n < MAXN; n++) {
      const double v = wave_sum(acc[n]);
      if (n < N && lane_id() == 0) C[r * N + n] = (T)(accumulate ? v + (double)C[r * N + n] : v);
    }
  }
}

// Many small products: one thread per entry of C, products summed in fp64 in
// order (fp32: exact ones).  Bound by its loads from L1; a 64 x 64 tile per
// product stages and stores mostly padding (10,000 of 8 x 8 x 8: fp64 85 us,
// 12.9 so, fp32 96 and 12.0; 16 x 16 x 16 84 and 32, 97 and 16).
template <class T>
__global__ void __launch_bounds__(256) gemm_tiny(const T *__restrict__ A, const T *__restrict__ B, T *__restrict__ C,
                                                 int M, int N, int K, int accumulate, int64_t total) {
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; o < total; o += step) {
    const int64_t r = o / N, z = r / M;
    const T *a = A + r * K, *b = B + z * K * N + (o - r * N);
    double v = 0.0;
#pragma unroll 4
    for (int k = 0; k < K; k++) v += (double)a[k] * (double)b[(int64_t)k * N];
    C[o] = (T)(accumulate ? v + (double)C[o] : v);
  }
}

// C (+)= the S partial products of each batch, added in order in fp64.
template <class T>
__global__ void gemm_combine(const double *__restrict__ W, T *__restrict__ C, int64_t mn, int S, int64_t total,
                             int accumulate) {
  for (int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; o < total; o += (int64_t)gridDim.x * blockDim.x) {
    const int64_t z = o / mn, e = o - z * mn;
    const double *p = W + z * S * mn + e;
    double v = 0.0;
    for (int y = 0; y < S; y++) v += p[(int64_t)y * mn];
    if (accumulate) v += (double)C[o];
    C[o] = (T)v;
  }
}

template <class T, int NTM, int NTN, int WM, int WN, class Off = uint32_t>
void gemm_launch(Ctx *c, const T *A, const T *B, T *C, int64_t M, int64_t N, int64_t K, int accumulate,
                 int64_t batch, int S, hipStream_t s) {
  using G = GemmTile<T, NTM, NTN, WM, WN>;
  const int64_t tiles = ((M + G::TM - 1) / G::TM) * ((N + G::TN - 1) / G::TN);
  const int64_t kt = (K + G::BK - 1) / G::BK;
  int64_t kchunk = std::max<int64_t>(K, 1);
  Buf ws;
  if (S > 1) {
    kchunk = (kt + S - 1) / S * G::BK;
    S = (int)((K + kchunk - 1) / kchunk);
  }
  if (S > 1) {
    try {
      ws = Buf(c, sizeof(double) * (size_t)(S * batch) * (size_t)(M * N));
    } catch (const Error &e) {  // no room for the partial sums: one pass over k
      if (e.st != SRTC_ERR_OOM) throw;
      S = 1;
      kchunk = K;
    }
  }
  const dim3 grid((unsigned)tiles, (unsigned)std::max(S, 1), (unsigned)std::min<int64_t>(batch, 65535));
  if (N % G::VEC == 0)
    gemm_mfma<T, NTM, NTN, WM, WN, Off, false><<<grid, G::THREADS, 0, s>>>(A, B, C, ws.as<double>(), M, N, K, kchunk,
                                                                          accumulate, batch);
  else
    gemm_mfma<T, NTM, NTN, WM, WN, Off, true><<<grid, G::THREADS, 0, s>>>(A, B, C, ws.as<double>(), M, N, K, kchunk,
                                                                         accumulate, batch);
  SRTC_LAUNCH_CHECK("gemm_mfma");
  if (S > 1) {
    const int64_t total = batch * M * N;
    gemm_combine<T><<<(unsigned)std::min<int64_t>((total + 255) / 256, 65536), 256, 0, s>>>(ws.as<double>(), C, M * N,
                                                                                         S, total, accumulate);
    SRTC_LAUNCH_CHECK("gemm_combine");
  }
}

struct PermArgs {
  int64_t sdims[SRTC_MAX_ORDER];   // source extents
  int64_t sstride[SRTC_MAX_ORDER]; // source strides
  int64_t odims[SRTC_MAX_ORDER];   // output extents (source mode perm[q])
  int perm[SRTC_MAX_ORDER];
  int order;
  int64_t total;
};

template <class E>
__global__ void permute_kernel(const E *__restrict__ src, E *__restrict__ dst, PermArgs a) {
  for (int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; o < a.total;
       o += (int64_t)gridDim.x * blockDim.x) {
    int64_t rem = o, si = 0;
    for (int q = a.order - 1; q >= 0; q--) {
      const int64_t idx = rem % a.odims[q];
      rem /= a.odims[q];
      si += idx * a.sstride[a.perm[q]];
    }
    dst[o] = src[si];
  }
}

// dst (in its own mode order) = src permuted, combined with dst's previous
// value by the semiring's (+); entries equal to the identity are absent.
template <class SR>
__global__ void permute_combine_kernel(const typename SR::val_t *__restrict__ src, typename SR::val_t *__restrict__ dst,
                                       PermArgs a, typename SR::acc_t id) {
  using A = typename SR::acc_t;
  for (int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; o < a.total;
       o += (int64_t)gridDim.x * blockDim.x) {
    int64_t rem = o, si = 0;
    for (int q = a.order - 1; q >= 0; q--) {
      const int64_t idx = rem % a.odims[q];
      rem /= a.odims[q];
      si += idx * a.sstride[a.perm[q]];
    }
    A acc = id;
    const auto x = src[si], y = dst[o];
    if (!SR::absent(x, id)) acc = SR::add(acc, (A)x);
    if (!SR::absent(y, id)) acc = SR::add(acc, (A)y);
    dst[o] = out_clamped<SR>(acc, id);
  }
}

PermArgs perm_args(int order, const int64_t *dims, const int *perm) {
  PermArgs a{};
  a.order = order;
  a.total = 1;
  int64_t st = 1;
  for (int q = order - 1; q >= 0; q--) {
    a.sdims[q] = dims[q];
    a.sstride[q] = st;
    st *= dims[q];
  }
  for (int q = 0; q < order; q++) {
    a.perm[q] = perm[q];
    a.odims[q] = dims[perm[q]];
    a.total *= dims[q];
  }
  return a;
}

struct CombineCall {
  IdVal id;
  const void *src;
  void *dst;
  PermArgs a;
  hipStream_t s;
};

template <class SR> void permute_combine_typed(const CombineCall &q) {
  using V = typename SR::val_t;
  const unsigned grid = (unsigned)std::min<int64_t>((q.a.total + 255) / 256, 65536);
  permute_combine_kernel<SR><<<grid, 256, 0, q.s>>>((const V *)q.src, (V *)q.dst, q.a, id_as<SR>(q.id));
  SRTC_LAUNCH_CHECK("permute_combine_kernel");
}

// C = A (x) B elementwise, combined with C's previous value by (+) when
// accumulating; identity operands give the identity.
template <class SR>
__global__ void hadamard_kernel(const typename SR::val_t *__restrict__ A, const typename SR::val_t *__restrict__ B,
                                typename SR::val_t *__restrict__ C, int64_t n, int accumulate,
                                typename SR::acc_t id) {
  using Acc = typename SR::acc_t;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
    const auto a = A[e], b = B[e];
    Acc acc = id;
    if (!SR::absent(a, id) && !SR::absent(b, id)) acc = SR::mul(a, b);
    if (accumulate) {
      const auto y = C[e];
      if (!SR::absent(y, id)) acc = SR::add(acc, (Acc)y);
    }
    C[e] = out_clamped<SR>(acc, id);
  }
}

struct HadamardCall {
  IdVal id;
  const void *A, *B;
  void *C;
  int64_t n;
  int accumulate;
  hipStream_t s;
};

template <class SR> void hadamard_typed(const HadamardCall &q) {
  using V = typename SR::val_t;
  const unsigned grid = (unsigned)std::min<int64_t>((q.n + 255) / 256, 65536);
  hadamard_kernel<SR><<<grid, 256, 0, q.s>>>((const V *)q.A, (const V *)q.B, (V *)q.C, q.n, q.accumulate,
                                             id_as<SR>(q.id));
  SRTC_LAUNCH_CHECK("hadamard_kernel");
}

}  // namespace

void dense_hadamard(int sr, int dt, IdVal id, const void *A, const void *B, void *C, int64_t n, int accumulate,
                    hipStream_t s) {
  if (n <= 0) return;
  HadamardCall q{id, A, B, C, n, accumulate, s};
  SRTC_DISPATCH_SR(sr, dt, hadamard_typed, q);
}

void dense_permute_combine(int sr, int dt, IdVal id, const void *src, void *dst, int order, const int64_t *dims,
                           const int *perm, hipStream_t s) {
  CombineCall q{id, src, dst, perm_args(order, dims, perm), s};
  if (q.a.total == 0) return;
  SRTC_DISPATCH_SR(sr, dt, permute_combine_typed, q);
}

namespace {
// Tile and split of a product.  64 x 64 tiles, four blocks per CU, are the
// general shape: fp64 8192^3 15.1 ms (72.8 TFLOP/s) and 2560^3 0.53 ms,
// against 15.3 and 0.62 ms with 128 x 128 tiles, whose last round of blocks
// leaves more of the chip idle.  128 x 64 tiles read A's and B's entries less
// often and gain 1 to 5% (fp64 4096^3 1.99 -> 1.92 ms, fp32 2048^3 0.149 ->
// 0.142 ms) where their blocks fill the last round of two per CU to at
// least nine tenths (2560^3, filled to 0.78: 0.53 -> 0.61 ms) and cover at most
// 15% more than the small ones (192 x 16,384 x 2,000 fp64 243 us, 202 with the
// small tiles; 448 x 8,192 x 2,000 fp32, 14% more, 140 and 145; 2,000 products
// of 64 x 64 x 64 fp32 in one call 33 and 23).
// Otherwise k may be split over S blocks.  The time of S parts follows the
// blocks per CU: one alone takes c1 ns per k-term (it waits on memory), b
// together c2 b; a split adds a launch (6 us) and its fp64 partial sums
// written and read at about 4 TB/s.  At c1, c2 as measured (64 x 64 x 5000:
// 190 us fp64, 108 us fp32; 2000^3: 246 and 148 us) S = 1 stays for 1000^3
// (46 against 48 us at S = 2), 500 x 500 x 3000 fp64 goes from 118 to 40 us
// and 800 x 2500 x 6000 from 555 to 411 us.  Partial sums take at most 64 MB;
// nothing is split while the stream is captured, where nothing is allocated.
template <class T, int LM, int LN, int WM, int WN>
void gemm_shape(Ctx *c, const T *A, const T *B, T *C, int64_t M, int64_t N, int64_t K, int accumulate,
                int64_t batch, hipStream_t s) {
  // Small products in a batch that gives every CU one and more: a thread per
  // entry takes 0.75 (fp64) or 0.3 (fp32) ns per 1,000 terms, a 64 x 64 tile,
  // whatever part of it is used, 3.2 + K / 10 or 4.6 + K / 22 ns.  (Long dot
  // products stay with the tiles, which split them.)
  const double each = sizeof(T) == 8 ? 0.75e-3 : 0.3e-3;
  const double tile = sizeof(T) == 8 ? 3.2 + 0.105 * (double)K : 4.6 + 0.045 * (double)K;
  if (batch > c->num_cus && K <= 256 && M <= 64 && N <= 64 && each * (double)(M * N * K) <= tile) {
    const int64_t total = M * N * batch;
    gemm_tiny<T><<<(unsigned)std::min<int64_t>((total + 255) / 256, 65536), 256, 0, s>>>(A, B, C, (int)M, (int)N, (int)K,
                                                                                       accumulate, total);
    SRTC_LAUNCH_CHECK("gemm_tiny");
    return;
  }
  if (N < GemmVec<T>::N) {
    gemm_narrow<T><<<(unsigned)std::min<int64_t>((M * batch + 3) / 4, 16384), 256, 0, s>>>(A, B, C, M, (int)N, K,
                                                                                         accumulate, batch);
    SRTC_LAUNCH_CHECK("gemm_narrow");
    return;
  }
  auto blocks = [&](int tm, int tn) { return ((M + tm - 1) / tm) * ((N + tn - 1) / tn) * batch; };
  const int64_t cus = c->num_cus;
  // byte offsets of a row tile past 32 bits: 64-bit ones
  if (std::max(K, N) >= (int64_t(1) << 32) / (128 * (int64_t)sizeof(T))) {
    gemm_launch<T, 2, 2, 2, 2, uint64_t>(c, A, B, C, M, N, K, accumulate, batch, 1, s);
    return;
  }
  const int64_t big = blocks(LM * 16 * WM, LN * 16 * WN), small = blocks(64, 64);
  const int64_t round = 2 * cus;
  if (40 * big <= 23 * small && 10 * big >= 9 * ((big + round - 1) / round * round)) {
    gemm_launch<T, LM, LN, WM, WN>(c, A, B, C, M, N, K, accumulate, batch, 1, s);
    return;
  }
  const double c1 = sizeof(T) == 8 ? 38e-3 : 21.6e-3, c2 = sizeof(T) == 8 ? 31e-3 : 18.5e-3;  // us
  const double mn = (double)M * (double)N * (double)batch;
  int best = 1;
  double t_best = 0;
  for (int S = 1; S <= 32 && (S == 1 || (K / S >= 64 && 8.0 * S * mn <= (double)(64 << 20))); S++) {
    const double b = (double)((small * S + cus - 1) / cus);
    const double t = (double)K / S * std::max(c1, c2 * b) + (S > 1 ? 6.0 + S * mn * 16.0 / 4e6 : 0.0);
    if (S == 1 || t < t_best) {
      best = S;
      t_best = t;
    }
  }
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (best > 1 && (hipStreamIsCapturing(s, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone)) best = 1;
  gemm_launch<T, 2, 2, 2, 2>(c, A, B, C, M, N, K, accumulate, batch, best, s);
}
}  // namespace

void dense_gemm_plus_times(Ctx *c, int dt, const void *A, const void *B, void *C, int64_t M, int64_t N, int64_t K,
                           int accumulate, hipStream_t s, int64_t batch) {
  if (M == 0 || N == 0 || batch <= 0) return;
  const int64_t side = M >= 128 && N >= 128 ? 128 : 64;
  if ((M + side - 1) / side > 65535) fail(SRTC_ERR_UNSUPPORTED, "dense gemm: too many row tiles");
  if (dt == SRTC_F64)
    gemm_shape<double, 2, 2, 4, 2>(c, (const double *)A, (const double *)B, (double *)C, M, N, K, accumulate, batch, s);
  else if (dt == SRTC_F32)
    gemm_shape<float, 4, 2, 2, 2>(c, (const float *)A, (const float *)B, (float *)C, M, N, K, accumulate, batch, s);
  else
    fail(SRTC_ERR_DTYPE, "dense (+,x) needs F64 or F32");
}

void dense_permute(const void *src, void *dst, int esize, int order, const int64_t *dims, const int *perm,
                   hipStream_t s) {
  const PermArgs a = perm_args(order, dims, perm);
  if (a.total == 0) return;
  const unsigned grid = (unsigned)std::min<int64_t>((a.total + 255) / 256, 65536);
  switch (esize) {
    case 8: permute_kernel<uint64_t><<<grid, 256, 0, s>>>((const uint64_t *)src, (uint64_t *)dst, a); break;
    case 4: permute_kernel<uint32_t><<<grid, 256, 0, s>>>((const uint32_t *)src, (uint32_t *)dst, a); break;
    default: permute_kernel<uint8_t><<<grid, 256, 0, s>>>((const uint8_t *)src, (uint8_t *)dst, a); break;
  }
  SRTC_LAUNCH_CHECK("permute_kernel");
}

}  // namespace srtc
