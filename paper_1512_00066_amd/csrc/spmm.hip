// Sparse x dense semiring products and the fixpoint steps built on them.
//
//   Y[i, c] = (+)_{k in A_i} A_ik (x) X[k, c]               (SpMM)
//   Y[i, c] = X[i, c] (+) (+)_{k in A_i} A_ik (x) X[k, c]   (Bellman-Ford step)
//
// The paper's measured kernel is exactly this sparse x dense product (MKL
// CSRMM for (+,x), a COO kernel for the tropical semiring; Section 6), and
// Bellman-Ford is P <- P (+) A (x) P on the tropical semiring (Section 4.2).
//
// Work is cut into items of at most T nonzeros of one row, so a row of any
// length costs at most T sequential gathers per lane.  Up to 32 dense columns,
// G lanes (G = a power of two >= the width) share an item, one lane per
// column; above, a wave takes a unit of consecutive nonzeros, of however many
// items, times a chunk of 64 columns.  A row split into several items writes
// partial sums that a second kernel combines in item order, which keeps every
// semiring, including fp (+), deterministic.
#include <algorithm>
#include <mutex>
#include <string>

#include "internal.hpp"
#include "spmm_plan.hpp"

// The one device buffer of the product that allocates nothing: its work-item
// plan and the partial results of split rows.  Each device holds its own copy
// from the first look-up until the process ends.  Host code never passes this
// name to a kernel (on the host it is a stand-in, not a device address): it
// uses the address hipGetSymbolAddress returns for the current device.
static constexpr size_t kFixedScratchBytes = size_t(64) << 20;
static __device__ __align__(256) unsigned char scratch[kFixedScratchBytes];

namespace srtc {

namespace {

inline unsigned gridn(int64_t n, int bs = 256, int64_t cap = 65536) {
  int64_t g = (n + bs - 1) / bs;
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>(g, cap));
}

__global__ void items_count(const int64_t *rp, int64_t m, int64_t T, int64_t *cnt, int64_t *pcnt) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t nz = rp[i + 1] - rp[i];
    const int64_t c = nz <= T ? 1 : (nz + T - 1) / T;
    cnt[i] = c;
    pcnt[i] = c > 1 ? c : 0;
  }
}

__global__ void items_fill(const int64_t *rp, int64_t m, int64_t T, const int64_t *ioff, const int64_t *poff,
                           int32_t *irow, int64_t *ibeg, int64_t *ipidx) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t a = rp[i];
    const int64_t c = ioff[i + 1] - ioff[i];
    if (i == m - 1) ibeg[ioff[m]] = rp[m];  // items are consecutive: item it ends where it + 1 begins
    for (int64_t t = 0; t < c; t++) {
      const int64_t it = ioff[i] + t;
      irow[it] = (int32_t)i;
      ibeg[it] = a + t * T;
      ipidx[it] = c > 1 ? poff[i] + t : -1;
    }
  }
}

// First item of every unit: items are cut into units of about `cost` work,
// an item counting its nonzeros plus UNIT_ITEM.  Unit w starts at the first
// item whose preceding work reaches w cost; ufirst[nunits] = nitems.  With
// cost <= T + UNIT_ITEM and T <= 256 a unit has at most 53 items, one per lane.
constexpr int64_t UNIT_ITEM = 5;
constexpr int T_MAX = 256;  // most nonzeros of an item (a grain as long is never reached)
__global__ void units_fill(const int64_t *__restrict__ ibeg, const int64_t *__restrict__ nitems_p, int64_t cost,
                           int64_t max_units, int64_t *__restrict__ ufirst) {
  const int64_t nitems = *nitems_p;
  const int64_t z0 = nitems > 0 ? ibeg[0] : 0;
  for (int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; w <= max_units;
       w += (int64_t)gridDim.x * blockDim.x) {
    int64_t lo = 0, hi = nitems;
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      if (ibeg[mid] - z0 + mid * UNIT_ITEM < w * cost) lo = mid + 1; else hi = mid;
    }
    ufirst[w] = lo;
  }
}

// A lane's value as a scalar (the same on every lane of the wave).
template <class T> __device__ __forceinline__ T lane_value(T v, int lane) {
  if constexpr (sizeof(T) == 8) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint64_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
    const uint64_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
    return __builtin_bit_cast(T, (hi << 32) | lo);
  } else if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
  } else {
    return (T)__builtin_amdgcn_readlane((int)v, lane);
  }
}

// The products wider than 32 columns: one wave per (unit, chunk of 64
// columns), one lane per column.  A unit's nonzeros are consecutive whatever
// rows they belong to, so the wave reads 64 of A's entries at a time (one
// load, the next 64 in flight) and takes each as a scalar, U rows of X in
// flight; an item's sum is written when its last nonzero has been added.
// (One wave per item kept at most four rows in flight and waited for the
// item's bounds, its entries and X one after the other: R-MAT 18, 64 int32
// sources, 311 us per step; 140 now.)
// Sums run over `grain` nonzeros of an item in order, and those sums are added
// in order.  (Reading the next U rows during the additions of these gained
// nothing: eight waves per SIMD cover the wait.)
// With at least eight chunks, XCD x (block id mod 8) takes chunks x, x + 8,
// ...: its L2 then holds one 64-column slice of X at a time, not all of X
// (16,384 x 16,384 at 1% times 1,024 fp64 columns: 2.96 -> 2.17 ms).
// DELTA (rin given): only nonzeros of rows that changed in the previous step
// count: an unchanged row's term is already part of the row's value.
// Eight waves per SIMD (64 registers): the grid's blocks are then all resident.
template <class SR, int MODE, bool ACC, bool DELTA>
__global__ void __launch_bounds__(256, 8) spmm_units(const int64_t *__restrict__ ufirst, int32_t nunits,
                                                  const int32_t *__restrict__ irow, const int64_t *__restrict__ ibeg,
                                                  const int64_t *__restrict__ ipidx, const int32_t *__restrict__ cA,
                                                  const typename SR::val_t *__restrict__ vA,
                                                  const typename SR::val_t *__restrict__ X, int64_t s, int grain,
                                                  void *__restrict__ Yv, typename SR::acc_t *__restrict__ P,
                                                  typename SR::acc_t id, int32_t *changed,
                                                  const uint8_t *__restrict__ rin, uint8_t *__restrict__ rout) {
  using V = typename SR::val_t;
  using A = typename SR::acc_t;
  constexpr int U = 8, WPB = 256 / WAVE;
  static_assert(MODE == 0 || !ACC, "one old value per entry");
  constexpr bool OLD = MODE == 1 || ACC;
  V *Y = reinterpret_cast<V *>(Yv);
  const int lane = lane_id();
  const int32_t wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
  UnitTurns turns(nunits, (int32_t)((s + WAVE - 1) / WAVE), gridDim.x, WPB, blockIdx.x, wv, s * sizeof(V) % 128 != 0);
  int32_t un, c;
  while (turns.next(&un, &c)) {
    const int64_t i0 = ufirst[un];
    const int n = (int)(ufirst[un + 1] - i0);
    if (n == 0) continue;
    const int64_t col = (int64_t)c * WAVE + lane;
    const bool on = col < s;
    const uint32_t lo = (uint32_t)((on ? lane : 0) * sizeof(V));  // a lane's bytes into the chunk
    const char *Xc = reinterpret_cast<const char *>(X + (int64_t)c * WAVE);
    const uint32_t rb = (uint32_t)(s * sizeof(V));  // bytes per row (the host checks that they fit)
    auto row_of = [&](const char *base, int32_t r) { return base + (uint64_t)(uint32_t)r * rb; };
    // lane j: item j's row, partial slot and end
    int32_t mrow = 0;
    int64_t mpi = -1, mend = 0;
    const int64_t b = ibeg[i0], e = ibeg[i0 + n];
    if (lane < n) {
      mrow = irow[i0 + lane];
      mpi = ipidx[i0 + lane];
      mend = ibeg[i0 + lane + 1] - b;
    }
    const int32_t len = (int32_t)(e - b);
    const int32_t mend32 = (int32_t)mend;
    // item `it` ends at iend; its running sum `acc` stops at ie, there or at
    // the next multiple of grain
    int it = 0;
    int32_t iend = lane_value(mend32, 0), ie = min(iend, grain);
    const char *Oc = MODE == 1 ? Xc : reinterpret_cast<const char *>(Y + (int64_t)c * WAVE);
    V old{};
    if (OLD) old = *(const V *)(row_of(Oc, lane_value(mrow, 0)) + lo);
    A acc = id, tot = id;
    // the running sum is complete; if item `it` is too, its total goes out and
    // the next one's old value comes in
    auto put = [&]() {
      if (ie < iend) {
        tot = SR::add(tot, acc);
        acc = id;
        ie = min(iend, ie + grain);
        return;
      }
      if (grain < T_MAX) acc = SR::add(tot, acc);
      const int32_t row = lane_value(mrow, it);
      const int64_t pi = lane_value(mpi, it);
      bool diff = false;
      if (pi >= 0) {
        if (on) P[pi * s + col] = acc;
      } else {
        if (OLD && !SR::absent(old, id)) acc = SR::add(acc, (A)old);
        const V o = out_clamped<SR>(acc, id);
        if (on) Y[(int64_t)row * s + col] = o;
        if (MODE == 1) diff = on && o != old;
      }
      if (MODE == 1 && __any(diff) && lane == 0) {
        *changed = 1;
        if (rout) rout[row] = 1;
      }
      acc = id;
      tot = id;
      it++;
      if (it < n) {
        const int32_t ib = iend;
        iend = lane_value(mend32, it);
        ie = min(iend, ib + grain);
        if (OLD) old = *(const V *)(row_of(Oc, lane_value(mrow, it)) + lo);
      }
    };
    const int32_t *cb = cA + b;
    const V *vb = vA + b;
    int32_t kk = 0, kn = 0;
    V vv{}, vn{};
    if (lane < len) {
      kn = cb[lane];
      vn = vb[lane];
    }
    for (int32_t p = 0; p < len; p += WAVE) {
      kk = kn;
      vv = vn;
      const int cnt = min(WAVE, len - p);
      if (p + WAVE + lane < len) {
        kn = cb[p + WAVE + lane];
        vn = vb[p + WAVE + lane];
      }
      bool good = lane < cnt && !SR::absent(vv, id);
      if (DELTA && good) good = rin[kk] != 0;
      const uint64_t use = __ballot(good);
      for (int q = 0; q < cnt; q += U) {
        const uint32_t m = (uint32_t)(use >> q) & ((1u << U) - 1u);
        // every load is issued (past the last nonzero, of a row read before):
        // a branch around each would wait for all of them
        V x[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
          x[u] = V{};
          if (!DELTA || ((m >> u) & 1u)) x[u] = *(const V *)(row_of(Xc, lane_value(kk, q + u)) + lo);
        }
        if (m == (1u << U) - 1u && ie >= p + q + U) {
#pragma unroll
          for (int u = 0; u < U; u++) {
            const A y = SR::mul(lane_value(vv, q + u), x[u]);
            if (!SR::absent(x[u], id)) acc = SR::add(acc, y);
          }
        } else {
#pragma unroll
          for (int u = 0; u < U; u++) {
            if (q + u < cnt)
              while (ie <= p + q + u) put();
            const A y = SR::mul(lane_value(vv, q + u), x[u]);
            if (((m >> u) & 1u) && !SR::absent(x[u], id)) acc = SR::add(acc, y);
          }
        }
      }
    }
    while (it < n) put();
  }
}

// MODE: 0 = plain product (Y = A X, or Y (+)= A X with ACC), 1 = fixpoint
// step (self term, change flag, optional per-instance bookkeeping).
template <class SR, int G, int MODE, bool ACC>
__global__ void __launch_bounds__(256) spmm_items(const int32_t *__restrict__ irow, const int64_t *__restrict__ ibeg,
                                                  const int64_t *__restrict__ ipidx,
                                                  const int64_t *__restrict__ nitems_p, const int32_t *__restrict__ cA,
                                                  const typename SR::val_t *__restrict__ vA,
                                                  const typename SR::val_t *__restrict__ X, int64_t s,
                                                  void *__restrict__ Yv, typename SR::acc_t *__restrict__ P,
                                                  typename SR::acc_t id, int32_t *changed,
                                                  const int32_t *__restrict__ row_inst,
                                                  const uint8_t *__restrict__ inst_active, int32_t *inst_changed,
                                                  const uint8_t *__restrict__ rin, uint8_t *__restrict__ rout) {
  using V = typename SR::val_t;
  using A = typename SR::acc_t;
  // (+,x) SpMM results are stored in the operand type; accumulators are A
  V *Y = reinterpret_cast<V *>(Yv);
  constexpr int PER_WAVE = WAVE / G;
  const int64_t nitems = *nitems_p;
  const int lane = lane_id();
  const int grp = lane / G, c = lane % G;
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / WAVE;
  const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) / WAVE;
  // work units: (item, chunk of G columns); wider than G only when G = 64,
  // so each wave then takes one chunk of one item at a time
  const int64_t nch = (s + G - 1) / G;
  for (int64_t u = wave * PER_WAVE + grp; u < nitems * nch; u += nwaves * PER_WAVE) {
    const int64_t it = nch == 1 ? u : u / nch;
    const int64_t row = irow[it];
    if (MODE == 1 && row_inst && !inst_active[row_inst[row]]) continue;
    const int64_t b = ibeg[it], e = ibeg[it + 1];
    const int64_t pi = ipidx[it];
    {
      const int64_t c0 = (u - it * nch) * G;
      const int64_t col = c0 + c;
      const bool on = col < s;
      A acc = id;
      if (on) {
        int64_t p = b;
        if (MODE == 1 && rin) {
          // only rows that changed in the previous step can lower this one:
          // an unchanged row's term is already part of the row's value
          for (; p + 4 <= e; p += 4) {
            const int32_t k0 = cA[p], k1 = cA[p + 1], k2 = cA[p + 2], k3 = cA[p + 3];
            const bool u0 = rin[k0], u1 = rin[k1], u2 = rin[k2], u3 = rin[k3];
            const V a0 = vA[p], a1 = vA[p + 1], a2 = vA[p + 2], a3 = vA[p + 3];
            const V x0 = u0 ? X[(int64_t)k0 * s + col] : id, x1 = u1 ? X[(int64_t)k1 * s + col] : id;
            const V x2 = u2 ? X[(int64_t)k2 * s + col] : id, x3 = u3 ? X[(int64_t)k3 * s + col] : id;
            if (!SR::absent(a0, id) && !SR::absent(x0, id)) acc = SR::add(acc, SR::mul(a0, x0));
            if (!SR::absent(a1, id) && !SR::absent(x1, id)) acc = SR::add(acc, SR::mul(a1, x1));
            if (!SR::absent(a2, id) && !SR::absent(x2, id)) acc = SR::add(acc, SR::mul(a2, x2));
            if (!SR::absent(a3, id) && !SR::absent(x3, id)) acc = SR::add(acc, SR::mul(a3, x3));
          }
          for (; p < e; p++) {
            const int32_t k = cA[p];
            if (!rin[k]) continue;
            const V a = vA[p];
            const V x = X[(int64_t)k * s + col];
            if (!SR::absent(a, id) && !SR::absent(x, id)) acc = SR::add(acc, SR::mul(a, x));
          }
        } else {
          for (; p + 4 <= e; p += 4) {
            const int32_t k0 = cA[p], k1 = cA[p + 1], k2 = cA[p + 2], k3 = cA[p + 3];
            const V a0 = vA[p], a1 = vA[p + 1], a2 = vA[p + 2], a3 = vA[p + 3];
            const V x0 = X[(int64_t)k0 * s + col], x1 = X[(int64_t)k1 * s + col];
            const V x2 = X[(int64_t)k2 * s + col], x3 = X[(int64_t)k3 * s + col];
            if (!SR::absent(a0, id) && !SR::absent(x0, id)) acc = SR::add(acc, SR::mul(a0, x0));
            if (!SR::absent(a1, id) && !SR::absent(x1, id)) acc = SR::add(acc, SR::mul(a1, x1));
            if (!SR::absent(a2, id) && !SR::absent(x2, id)) acc = SR::add(acc, SR::mul(a2, x2));
            if (!SR::absent(a3, id) && !SR::absent(x3, id)) acc = SR::add(acc, SR::mul(a3, x3));
          }
          for (; p < e; p++) {
            const int32_t k = cA[p];
            const V a = vA[p];
            const V x = X[(int64_t)k * s + col];
            if (!SR::absent(a, id) && !SR::absent(x, id)) acc = SR::add(acc, SR::mul(a, x));
          }
        }
      }
      bool diff = false;
      if (on) {
        if (pi >= 0) {
          P[pi * s + col] = acc;
        } else {
          if (MODE == 1) {
            const V old = X[row * s + col];
            if (!SR::absent(old, id)) acc = SR::add(acc, (A)old);
          }
          if (ACC) {
            const V prev = Y[row * s + col];
            if (!SR::absent(prev, id)) acc = SR::add(acc, (A)prev);
          }
          const V o = out_clamped<SR>(acc, id);
          Y[row * s + col] = o;
          if (MODE == 1) diff = o != X[row * s + col];
        }
      }
      if (MODE == 1) {
        // one store per lane group that saw a change
        const uint64_t bal = __ballot(diff);
        const uint64_t gmask = G >= WAVE ? ~0ull : (((1ull << G) - 1) << (grp * G));
        if (diff && (bal & gmask & lanemask_lt()) == 0) {
          *changed = 1;
          if (row_inst) inst_changed[row_inst[row]] = 1;
          if (rout) rout[row] = 1;
        }
      }
    }
  }
}

// Rows split into several items: combine partials in item order.  A wave looks
// at `look` (up to 64) items at a time for first items of split rows, brings
// those it found to its first lanes, and each group of G lanes (one per
// column) takes one of them, eight partials in flight.  With one item per look
// the search through many unsplit rows took 31 us of an R-MAT 18 step; with 64
// items per look always, and one row after the other in one lane per column,
// small products and narrow ones, where most rows are split, took up to twice
// the time (product alone, fp64, so / now / with one item per look: 1,000 rows
// of 100 nonzeros x 1 column 29 / 14 / 13 us; 100,000 of 40 x 1 83 / 48 / 48;
// 20,000 of 80 x 32 112 / 88 / 90; 300 of 1,000 x 64 59 / 36 / 45).
template <class SR, int G, int MODE, bool ACC>
__global__ void __launch_bounds__(256) spmm_combine(const int32_t *__restrict__ irow, const int64_t *__restrict__ ibeg,
                                                    const int64_t *__restrict__ ipidx, const int64_t *__restrict__ nitems_p,
                                                    int look, const int64_t *__restrict__ rp, int64_t T,
                                                    const typename SR::val_t *__restrict__ X, int64_t s,
                                                    void *__restrict__ Yv, const typename SR::acc_t *__restrict__ P,
                                                    typename SR::acc_t id, int32_t *changed,
                                                    const int32_t *__restrict__ row_inst,
                                                    const uint8_t *__restrict__ inst_active, int32_t *inst_changed,
                                                    uint8_t *__restrict__ rout) {
  using V = typename SR::val_t;
  using A = typename SR::acc_t;
  constexpr int U = 8, PER_WAVE = WAVE / G;
  V *Y = reinterpret_cast<V *>(Yv);
  const int64_t nitems = *nitems_p;
  const int lane = lane_id();
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / WAVE;
  const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) / WAVE;
  // (`look` items, chunk of G columns) per turn
  const int64_t nch = (s + G - 1) / G, looks = (nitems + look - 1) / look;
  for (int64_t g = wave; g < looks * nch; g += nwaves) {
    const int64_t it = g / nch * look + lane;
    int64_t pi0 = -1;
    int32_t row0 = 0;
    if (lane < look && it < nitems) {
      pi0 = ipidx[it];
      row0 = irow[it];
      if (pi0 >= 0 && ibeg[it] != rp[row0]) pi0 = -1;  // only the first item of a split row
    }
    const uint64_t mk = __ballot(pi0 >= 0);
    const int found = __popcll(mk);
    if (found == 0) continue;
    if (G < WAVE) {
      // found rows to lanes 0 .. found-1 (the others' values behind them)
      const int below = __popcll(mk & lanemask_lt());
      const int to = 4 * (pi0 >= 0 ? below : found + lane - below);
      const uint32_t lo = __builtin_amdgcn_ds_permute(to, (int)(uint32_t)pi0);
      const uint32_t hi = __builtin_amdgcn_ds_permute(to, (int)(uint32_t)(pi0 >> 32));
      pi0 = (int64_t)((uint64_t)hi << 32 | lo);
      row0 = __builtin_amdgcn_ds_permute(to, row0);
    }
    const int64_t col = g % nch * G + lane % G;
    uint64_t left = mk;
    for (int t = 0; t < found; t += PER_WAVE, left &= left - 1) {
      const int src = G < WAVE ? t + lane / G : __ffsll((unsigned long long)left) - 1;
      const int64_t pi = G < WAVE ? (int64_t)__shfl((long long)pi0, src, WAVE) : lane_value(pi0, src);
      const int64_t row = G < WAVE ? __shfl(row0, src, WAVE) : lane_value(row0, src);
      if (src >= (G < WAVE ? found : WAVE) || col >= s) continue;
      if (MODE == 1 && row_inst && !inst_active[row_inst[row]]) continue;
      const int64_t cnt = (rp[row + 1] - rp[row] + T - 1) / T;
      A acc = id;
      for (int64_t t = 0; t < cnt; t += U) {
        A x[U];
#pragma unroll
        for (int u = 0; u < U; u++) x[u] = t + u < cnt ? P[(pi + t + u) * s + col] : id;
#pragma unroll
        for (int u = 0; u < U; u++)
          if (t + u < cnt) acc = SR::add(acc, x[u]);
      }
      if (MODE == 1) {
        const V old = X[row * s + col];
        if (!SR::absent(old, id)) acc = SR::add(acc, (A)old);
      }
      if (ACC) {
        const V prev = Y[row * s + col];
        if (!SR::absent(prev, id)) acc = SR::add(acc, (A)prev);
      }
      const V o = out_clamped<SR>(acc, id);
      Y[row * s + col] = o;
      if (MODE == 1 && o != X[row * s + col]) {
        *changed = 1;
        if (row_inst) inst_changed[row_inst[row]] = 1;
        if (rout) rout[row] = 1;
      }
    }
  }
}

template <class SR, int G, int MODE, bool ACC>
void run_items(const SpmmPlan &pl, const CsrView &A, const void *X, int64_t s, void *Y, IdVal idv,
               int32_t *changed, const int32_t *row_inst, const uint8_t *inst_active, int32_t *inst_changed,
               const uint8_t *rin, uint8_t *rout, hipStream_t st) {
  using V = typename SR::val_t;
  using Acc = typename SR::acc_t;
  const Acc id = id_as<SR>(idv);
  const int64_t nch = (s + G - 1) / G;
  const unsigned grid =
      (unsigned)std::max<int64_t>(1, std::min<int64_t>(pl.max_items * nch * G / 256 + 1, pl.grid_cap));
  bool done = false;
  if constexpr (G == WAVE) {
    const int64_t waves = pl.nunits * nch;
    if (pl.nunits > 0 && !row_inst && waves < (1ll << 31) && s < (1ll << 29)) {
      unsigned gu = (unsigned)std::max<int64_t>(1, std::min<int64_t>((waves + 3) / 4, pl.grid_cap / 2));
      if (gu > 8) gu -= gu % 8;
      auto launch = [&](auto kern) {
        kern<<<gu, 256, 0, st>>>(pl.ufirst, (int32_t)pl.nunits, pl.irow, pl.ibeg, pl.ipidx, A.col, (const V *)A.val,
                                 (const V *)X, s, pl.grain, Y, (Acc *)pl.partial, id, changed, rin, rout);
      };
      if constexpr (MODE == 1) {
        if (rin) launch(spmm_units<SR, MODE, ACC, true>);
        else launch(spmm_units<SR, MODE, ACC, false>);
      } else {
        launch(spmm_units<SR, MODE, ACC, false>);
      }
      SRTC_LAUNCH_CHECK("spmm_units");
      done = true;
    }
  }
  if (!done) {
    spmm_items<SR, G, MODE, ACC><<<grid, 256, 0, st>>>(pl.irow, pl.ibeg, pl.ipidx, pl.nitems, A.col,
                                                        (const V *)A.val, (const V *)X, s, Y, (Acc *)pl.partial, id,
                                                        changed, row_inst, inst_active, inst_changed, rin, rout);
    SRTC_LAUNCH_CHECK("spmm_items");
  }
  if (pl.may_split) {
    // Fewer items per look where the chip has waves to spare and a look could
    // find more than one split row for each group (at most nnz / T rows are
    // split): 16 instead of 64 take a Bellman-Ford run on 100,000 skewed rows
    // of 16 with 64 sources from 1,717 to 1,356 us, but 8 instead of 64 one on
    // even rows of 4 with 8 sources from 800 to 845.
    int look = WAVE;
    while (look > WAVE / G && (pl.max_items + look - 1) / look * nch < 2 * pl.grid_cap &&
           look * (A.nnz / pl.T) > (WAVE / G) * pl.max_items)
      look /= 2;
    const int64_t cw = (pl.max_items + look - 1) / look * nch;
    const unsigned gc = (unsigned)std::max<int64_t>(1, std::min<int64_t>((cw + 3) / 4, pl.grid_cap));
    spmm_combine<SR, G, MODE, ACC><<<gc, 256, 0, st>>>(pl.irow, pl.ibeg, pl.ipidx, pl.nitems, look, A.rowptr, pl.T,
                                                       (const V *)X, s, Y, (const Acc *)pl.partial, id, changed, row_inst,
                                                       inst_active, inst_changed, rout);
    SRTC_LAUNCH_CHECK("spmm_combine");
  }
}

template <class SR, int MODE, bool ACC>
void run_by_width(const SpmmPlan &pl, const CsrView &A, const void *X, int64_t s, void *Y, IdVal id,
                  int32_t *changed, const int32_t *row_inst, const uint8_t *inst_active, int32_t *inst_changed,
                  const uint8_t *rin, uint8_t *rout, hipStream_t st) {
  switch (pl.G) {
    case 1: run_items<SR, 1, MODE, ACC>(pl, A, X, s, Y, id, changed, row_inst, inst_active, inst_changed, rin, rout, st); break;
    case 2: run_items<SR, 2, MODE, ACC>(pl, A, X, s, Y, id, changed, row_inst, inst_active, inst_changed, rin, rout, st); break;
    case 4: run_items<SR, 4, MODE, ACC>(pl, A, X, s, Y, id, changed, row_inst, inst_active, inst_changed, rin, rout, st); break;
    case 8: run_items<SR, 8, MODE, ACC>(pl, A, X, s, Y, id, changed, row_inst, inst_active, inst_changed, rin, rout, st); break;
    case 16: run_items<SR, 16, MODE, ACC>(pl, A, X, s, Y, id, changed, row_inst, inst_active, inst_changed, rin, rout, st); break;
    case 32: run_items<SR, 32, MODE, ACC>(pl, A, X, s, Y, id, changed, row_inst, inst_active, inst_changed, rin, rout, st); break;
    default: run_items<SR, 64, MODE, ACC>(pl, A, X, s, Y, id, changed, row_inst, inst_active, inst_changed, rin, rout, st); break;
  }
}

struct SpmmCall {
  const SpmmPlan *pl;
  const CsrView *A;
  const void *X;
  int64_t s;
  void *Y;
  IdVal id;
  int mode;
  int acc;
  int32_t *changed;
  const int32_t *row_inst;
  const uint8_t *inst_active;
  int32_t *inst_changed;
  const uint8_t *rin;
  uint8_t *rout;
  hipStream_t st;
};

template <class SR> void spmm_dispatch(const SpmmCall &q) {
  if (q.mode == 1)
    run_by_width<SR, 1, false>(*q.pl, *q.A, q.X, q.s, q.Y, q.id, q.changed, q.row_inst, q.inst_active,
                               q.inst_changed, q.rin, q.rout, q.st);
  else if (q.acc)
    run_by_width<SR, 0, true>(*q.pl, *q.A, q.X, q.s, q.Y, q.id, nullptr, nullptr, nullptr, nullptr, nullptr,
                              nullptr, q.st);
  else
    run_by_width<SR, 0, false>(*q.pl, *q.A, q.X, q.s, q.Y, q.id, nullptr, nullptr, nullptr, nullptr, nullptr,
                               nullptr, q.st);
}

// --------------------------------------------------------------------- BFS --
// One level: a row gathers its neighbours' frontier words and keeps the
// sources that had not reached it.  Sixteen lanes per row, four entries each
// in flight; the rows of a block with more than BFS_LONG entries are then
// taken by the whole block.  Either stops once every missing source is found
// (the hubs of a skewed graph find theirs in a few entries; with one wave per
// row, 64 entries at a time to the end, they bound the level: R-MAT 18, 64
// sources, 76 us per level, now 36).
constexpr int BFS_G = 16, BFS_U = 4, BFS_LONG = 512;
__global__ void __launch_bounds__(256) bfs_step_kernel(const int64_t *__restrict__ rp, const int32_t *__restrict__ cA,
                                                       int64_t n, const uint64_t *__restrict__ front,
                                                       uint64_t *__restrict__ visited, uint64_t *__restrict__ next,
                                                       int32_t *__restrict__ levels, int nsrc, int level,
                                                       uint64_t full, int32_t *changed) {
  constexpr int ROWS = 256 / BFS_G;
  __shared__ uint64_t found[ROWS], miss[ROWS];
  __shared__ int32_t has_long;
  const int t = threadIdx.x, g = t / BFS_G, l = t % BFS_G;
  auto take = [&](int64_t p, int64_t e, int64_t stride) {
    int32_t k[BFS_U];
    uint64_t acc = 0;
#pragma unroll
    for (int u = 0; u < BFS_U; u++) k[u] = p + u * stride < e ? cA[p + u * stride] : -1;
#pragma unroll
    for (int u = 0; u < BFS_U; u++)
      if (k[u] >= 0) acc |= front[k[u]];
    return acc;
  };
  for (int64_t i0 = (int64_t)blockIdx.x * ROWS; i0 < n; i0 += (int64_t)gridDim.x * ROWS) {
    const int64_t i = i0 + g;
    if (t == 0) has_long = 0;
    __syncthreads();
    int64_t a = 0, e = 0;
    uint64_t want = 0, acc = 0;
    if (i < n) {
      want = full & ~visited[i];
      if (want) {
        a = rp[i];
        e = rp[i + 1];
      }
    }
    // (the lanes of a row take the same trips: its bits are combined each time)
    for (int64_t p = a; p < min(e, a + BFS_LONG) && (acc & want) != want; p += BFS_G * BFS_U) {
      acc |= take(p + l, e, BFS_G);
#pragma unroll
      for (int d = BFS_G / 2; d >= 1; d >>= 1) acc |= __shfl_xor((unsigned long long)acc, d, WAVE);
    }
    if (l == 0) {
      found[g] = acc & want;
      miss[g] = want;
      if (e - a > BFS_LONG && (acc & want) != want) has_long = 1;
    }
    __syncthreads();
    if (has_long) {  // the same on every thread
      for (int q = 0; q < ROWS; q++) {
        const uint64_t w = miss[q];
        uint64_t f = found[q];
        const int64_t ri = i0 + q;
        if (f == w) continue;
        // every wave has looked at found[q] before any of them adds to it: one
        // that came late and saw the row complete would skip its barriers
        __syncthreads();
        const int64_t re = rp[ri + 1];
        for (int64_t p = rp[ri] + BFS_LONG; p < re && f != w; p += 256 * BFS_U) {
          uint64_t x = take(p + t, re, 256) & w;
#pragma unroll
          for (int d = WAVE / 2; d >= 1; d >>= 1) x |= __shfl_xor((unsigned long long)x, d, WAVE);
          if (lane_id() == 0 && x) atomicOr((unsigned long long *)&found[q], (unsigned long long)x);
          __syncthreads();
          f = found[q];
          __syncthreads();
        }
      }
    }
    const uint64_t fresh = found[g];
    if (i < n) {
      if (l == 0) {
        next[i] = fresh;
        if (fresh) {
          visited[i] = (full & ~miss[g]) | fresh;
          *changed = 1;
        }
      }
      for (int q = l; q < nsrc; q += BFS_G)
        if ((fresh >> q) & 1ull) levels[i * nsrc + q] = level;
    }
    __syncthreads();  // found and miss are rewritten by the next rows
  }
}

}  // namespace

void SpmmPlan::shape(Ctx *c, const CsrView &A, int64_t s_width) {
  ctx = c;
  rows = A.m;
  int g = 1;
  while (g < s_width && g < WAVE) g <<= 1;
  G = g;
  // an item times one chunk of G columns is the least that a wave (G = 64) or
  // a lane group takes at a time.  Shorter items for wide operands in a batch,
  // whose items are taken one by one; elsewhere 64 nonzeros an item would
  // split every row of the MP3 tensor (164 nonzeros) and write and read
  // partial sums three times the size of its result.
  T = s_width > 128 && batched ? 64 : (G >= 64 ? T_MAX : (G >= 8 ? 64 : 32));
  // wide operands still add up 64 nonzeros at a time
  grain = s_width > 128 ? 64 : T_MAX;
  max_items = A.m + A.nnz / T + 1;
  // a split row of z > T nonzeros has ceil(z / T) < 2 z / T items
  max_partial = 2 * (A.nnz / T) + 1;
  may_split = true;
  grid_cap = (int64_t)c->num_cus * 16;
  // Units of wide products: a full item's work each, or less where that would
  // not give every resident wave a unit (8,192 waves; product alone, 64
  // columns fp64: 10,000 rows of 10 nonzeros 29 us with full units, 15 so, 18
  // with one wave per row; 1,000 rows 42, 9 and 9).  Smaller units for the
  // larger products too, two to four turns of each wave, cost R-MAT 18 with 64
  // sources 3 to 9% and gained at most 4% on even rows.  The units' table fits
  // where max_items entries do.
  nunits = 0;
  if (G < WAVE || batched) return;
  const int64_t work = A.nnz + UNIT_ITEM * max_items, nch = (s_width + WAVE - 1) / WAVE;
  const int64_t full = T + UNIT_ITEM, resident = (int64_t)c->num_cus * 32;
  const double each = (double)work * (double)nch / (double)resident;
  ucost = (int64_t)std::min((double)full, std::max(each, 16.0));
  // (at least the average item's work)
  ucost = std::max(ucost, work / max_items + 2);
  nunits = work / ucost + 1;
  if (nunits + 1 > max_items) nunits = 0;
}

void SpmmPlan::fill(const CsrView &A, int64_t *cnt_p, int64_t *pcnt_p, int64_t *ioff_p, int64_t *poff_p,
                    int64_t *sums, int32_t *irow_p, int64_t *ibeg_p, int64_t *ufirst_p, int64_t *ipidx_p,
                    void *partial_p, hipStream_t st) {
  const int64_t m = A.m;
  if (m > 0) {
    items_count<<<gridn(m), 256, 0, st>>>(A.rowptr, m, T, cnt_p, pcnt_p);
    SRTC_LAUNCH_CHECK("items_count");
  }
  // the two scans run one after the other on st and share the tile sums
  excl_scan_i64_ws(cnt_p, ioff_p, m, sums, st);
  excl_scan_i64_ws(pcnt_p, poff_p, m, sums, st);
  if (m > 0) {
    items_fill<<<gridn(m), 256, 0, st>>>(A.rowptr, m, T, ioff_p, poff_p, irow_p, ibeg_p, ipidx_p);
    SRTC_LAUNCH_CHECK("items_fill");
    if (nunits > 0) {
      units_fill<<<gridn(nunits + 1), 256, 0, st>>>(ibeg_p, ioff_p + m, ucost, nunits, ufirst_p);
      SRTC_LAUNCH_CHECK("units_fill");
    }
  }
  irow = irow_p;
  ibeg = ibeg_p;
  ufirst = ufirst_p;
  ipidx = ipidx_p;
  nitems = ioff_p + m;
  partial = partial_p;
}

void SpmmPlan::build(Ctx *c, const CsrView &A, int64_t s_width, hipStream_t st) {
  shape(c, A, s_width);
  const int64_t m = A.m;
  const size_t rows = (size_t)std::max<int64_t>(m, 1);
  cnt = Buf(c, sizeof(int64_t) * rows);
  pcnt = Buf(c, sizeof(int64_t) * rows);
  ioff = Buf(c, sizeof(int64_t) * (size_t)(m + 1));
  poff = Buf(c, sizeof(int64_t) * (size_t)(m + 1));
  Buf sums(c, sizeof(int64_t) * (size_t)std::max<int64_t>(excl_scan_workspace(m), 1));
  irow_b = Buf(c, sizeof(int32_t) * (size_t)max_items);
  ibeg_b = Buf(c, sizeof(int64_t) * (size_t)max_items);
  ufirst_b = Buf(c, sizeof(int64_t) * (size_t)max_items);
  ipidx_b = Buf(c, sizeof(int64_t) * (size_t)max_items);
  partial_b = Buf(c, (size_t)max_partial * (size_t)s_width * 8);
  fill(A, cnt.as<int64_t>(), pcnt.as<int64_t>(), ioff.as<int64_t>(), poff.as<int64_t>(), sums.as<int64_t>(),
       irow_b.as<int32_t>(), ibeg_b.as<int64_t>(), ufirst_b.as<int64_t>(), ipidx_b.as<int64_t>(), partial_b.p, st);
}

namespace {
// Consecutive 256-byte aligned regions of one buffer, in the order they are
// taken; the same sequence sizes the buffer (base = null) and lays it out.
struct Carve {
  char *base;
  int64_t off = 0;
  template <class T> T *take(int64_t count) {
    T *p = base ? reinterpret_cast<T *>(base + off) : nullptr;
    off += (int64_t)(((uint64_t)std::max<int64_t>(count, 1) * sizeof(T) + 255) & ~(uint64_t)255);
    return p;
  }
};

struct PlanParts {
  int64_t *cnt, *pcnt, *ioff, *poff, *sums;
  int32_t *irow;
  int64_t *ibeg, *ufirst, *ipidx;
  double *partial;
};

int64_t carve_plan(const SpmmPlan &pl, int64_t m, int64_t s_width, char *base, PlanParts *out) {
  Carve cv{base};
  PlanParts q;
  q.cnt = cv.take<int64_t>(m);
  q.pcnt = cv.take<int64_t>(m);
  q.ioff = cv.take<int64_t>(m + 1);
  q.poff = cv.take<int64_t>(m + 1);
  q.sums = cv.take<int64_t>(excl_scan_workspace(m));
  q.irow = cv.take<int32_t>(pl.max_items);
  q.ibeg = cv.take<int64_t>(pl.max_items);
  q.ufirst = cv.take<int64_t>(pl.max_items);
  q.ipidx = cv.take<int64_t>(pl.max_items);
  q.partial = cv.take<double>(pl.max_partial * s_width);
  if (out) *out = q;
  return cv.off;
}
}  // namespace

int64_t SpmmPlan::workspace_bytes(int64_t s_width) const {
  // sizes far beyond any device memory are reported as INT64_MAX instead of
  // overflowing
  const double approx = 40.0 * (double)rows + 32.0 * (double)max_items + 8.0 * (double)max_partial * (double)s_width;
  if (approx > 0x1p60) return INT64_MAX;
  return carve_plan(*this, rows, s_width, nullptr, nullptr);
}

void SpmmPlan::build_in(const CsrView &A, int64_t s_width, void *ws, hipStream_t st) {
  PlanParts q;
  carve_plan(*this, A.m, s_width, static_cast<char *>(ws), &q);
  fill(A, q.cnt, q.pcnt, q.ioff, q.poff, q.sums, q.irow, q.ibeg, q.ufirst, q.ipidx, q.partial, st);
}

void spmm_with_plan(const SpmmPlan &pl, int sr, int dt, IdVal id, const CsrView &A, const void *X,
                    int64_t s_width, void *Y, int mode, int accumulate, int32_t *changed, const int32_t *row_inst,
                    const uint8_t *inst_active, int32_t *inst_changed, hipStream_t st, const uint8_t *rin,
                    uint8_t *rout) {
  SpmmCall q{&pl, &A, X, s_width, Y, id, mode, accumulate, changed, row_inst, inst_active, inst_changed, rin, rout, st};
  // algorithmic bytes: A once, X once, Y written (and read for the self
  // term / accumulation)
  const double es = (double)dtype_size(dt);
  const double xy = es * (double)s_width * (double)(A.m + A.n);
  ProfScope ps(pl.ctx, mode == 1 ? "spmm.fixpoint_step" : "spmm.product",
               (4.0 + es) * A.nnz + 8.0 * (A.m + 1) + xy + (mode == 1 || accumulate ? es * s_width * A.m : 0.0), st);
  SRTC_DISPATCH_SR(sr, dt, spmm_dispatch, q);
}

void spmm(Ctx *c, int sr, int dt, IdVal id, const CsrView &A, const void *X, int64_t s_width, void *Y,
          int accumulate, hipStream_t st) {
  if (A.m == 0 || s_width == 0) return;
  SpmmPlan pl;
  pl.build(c, A, s_width, st);
  spmm_with_plan(pl, sr, dt, id, A, X, s_width, Y, 0, accumulate, nullptr, nullptr, nullptr, nullptr, st);
}

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_fixed_mu;
void *g_fixed_ptr[kMaxDevices] = {};
}  // namespace

size_t spmm_fixed_scratch_bytes() { return kFixedScratchBytes; }

void *spmm_fixed_scratch_init(int device) {
  if (device < 0 || device >= kMaxDevices) fail(SRTC_ERR_DEVICE, "device ordinal beyond 63");
  std::lock_guard<std::mutex> lock(g_fixed_mu);
  if (!g_fixed_ptr[device]) {
    void *p = nullptr;
    SRTC_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) fail(SRTC_ERR_DEVICE, "no device address for the fixed buffer");
    g_fixed_ptr[device] = p;
  }
  return g_fixed_ptr[device];
}

void spmm_fixed(Ctx *c, int sr, int dt, IdVal id, const CsrView &A, const void *X, int64_t s_width, void *Y,
                int accumulate, hipStream_t st) {
  if (A.m == 0 || s_width == 0) return;
  if (!c->fixed_scratch) fail(SRTC_ERR_DEVICE, "the fixed buffer was not set up for this device");
  SpmmPlan pl;
  pl.shape(c, A, s_width);
  const int64_t need = pl.workspace_bytes(s_width);
  if (need > (int64_t)kFixedScratchBytes)
    fail(SRTC_ERR_TOO_LARGE, "the product's plan needs " + std::to_string(need) + " bytes; the fixed buffer holds " +
                                 std::to_string(kFixedScratchBytes) + " (call srtc_contract)");
  // every plan array is written before it is read, so the previous call's
  // contents need no clearing
  pl.build_in(A, s_width, c->fixed_scratch, st);
  // no profile record: its HIP events are resources this call must not take
  pl.ctx = nullptr;
  spmm_with_plan(pl, sr, dt, id, A, X, s_width, Y, 0, accumulate, nullptr, nullptr, nullptr, nullptr, st);
}

void bfs_step(const CsrView &A, const uint64_t *front, uint64_t *visited, uint64_t *next, int32_t *levels,
              int nsrc, int level, int32_t *changed, hipStream_t s) {
  const uint64_t full = nsrc >= 64 ? ~0ull : ((1ull << nsrc) - 1);
  bfs_step_kernel<<<gridn(A.m * BFS_G, 256, 16384), 256, 0, s>>>(A.rowptr, A.col, A.m, front, visited, next,
                                                                 levels, nsrc, level, full, changed);
  SRTC_LAUNCH_CHECK("bfs_step");
}

}  // namespace srtc
