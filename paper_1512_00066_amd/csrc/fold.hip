// Fold: index-value pairs -> CSR matrix (the mode folding of Section 5.1 and
// the local transposition/reordering of Section 6.2).
//
// Keys (row*ncols + col) are sorted, carrying their values, by a stable LSD
// radix sort whose per-tile digit ranking runs with wave ballots; the first
// pass reads the tensor's own keys and maps them to matrix keys on the way.
// Equal keys then form segments that are combined with the semiring's
// additive op in input order (float (+) accumulated in fp64 and rounded
// once), identity results are dropped and the row pointer is filled from the
// row boundaries of the sorted keys.
#include "internal.hpp"

namespace srtc {

namespace {

// ----------------------------------------------------------- radix sort --
// One pass per 8-bit digit.  A tile is 8,192 keys, so that a digit's run in it
// is 32 keys on average and the tile's writes are whole lines; keys and
// values pass through the same 64 KB of LDS one after the other, which lets
// two blocks of 1,024 threads share a CU.  A pass is bound by its reads and
// writes (12 bytes a pair in and out with 4-byte values).  2^24 R-MAT keys of
// 40 bits with fp32 values: 76 us a scatter (5.3 TB/s; 64 registers a thread
// are two blocks a CU, and spilling a few of them costs it 176 us), 27 us a
// histogram; whole fold 2,335 us with 2,048-key tiles, a gather of the values
// after the sort and segment arrays in memory, 723 us so.
constexpr int RS_BS = 1024;           // threads per tile
constexpr int RS_IT = 8;              // keys per thread
constexpr int RS_TILE = RS_BS * RS_IT;
constexpr int RS_NW = RS_BS / WAVE;
constexpr int RS_DIG = 256;           // 8-bit digits
constexpr int RS_REP = 4;             // copies of the histogram's counters
constexpr int RS_GMAX = 512;          // most groups of tiles
constexpr int NXCD = 8;

// x mod d and x / d by a multiplication with floor((2^64 - 1) / d), short of
// the quotient by at most one
__device__ __forceinline__ uint64_t fast_div(uint64_t x, uint64_t d, uint64_t magic, uint64_t *rem) {
  uint64_t q = __umul64hi(x, magic);
  uint64_t r = x - q * d;
  if (r >= d) {
    r -= d;
    q++;
  }
  *rem = r;
  return q;
}

template <bool MAP> __device__ __forceinline__ uint64_t map_key(uint64_t k, const KeyMap &a) {
  if (!MAP) return k;
  uint64_t out = 0;
  for (int m = a.order - 1; m >= 0; m--) {
    uint64_t x;
    k = fast_div(k, a.dim[m], a.magic[m], &x);
    out += x * a.mul[m];
  }
  return out;
}

// Digit counts of a group of `per` consecutive tiles: toff[tile][digit] = keys
// of the digit in the group's earlier tiles, gsum[digit][group] = all.
template <bool MAP>
__global__ void __launch_bounds__(RS_BS) radix_hist(const uint64_t *__restrict__ keys, int64_t n, int shift, KeyMap km,
                                                    int64_t ntiles, int64_t per, uint32_t *__restrict__ toff,
                                                    uint32_t *__restrict__ gsum) {
  __shared__ uint32_t cnt[RS_REP][RS_DIG + 1];
  const int t = threadIdx.x, rep = t & (RS_REP - 1);
  const int64_t t0 = (int64_t)blockIdx.x * per, t1 = min(ntiles, t0 + per);
  uint32_t run = 0;
  for (int u = t; u < RS_REP * (RS_DIG + 1); u += RS_BS) (&cnt[0][0])[u] = 0;
  __syncthreads();
  for (int64_t tile = t0; tile < t1; tile++) {
    const int64_t base = tile * RS_TILE + t;
    uint64_t k[RS_IT];
#pragma unroll
    for (int r = 0; r < RS_IT; r++) k[r] = base + r * RS_BS < n ? keys[base + r * RS_BS] : 0;
#pragma unroll
    for (int r = 0; r < RS_IT; r++)
      if (base + r * RS_BS < n) atomicAdd(&cnt[rep][(map_key<MAP>(k[r], km) >> shift) & 0xFF], 1u);
    __syncthreads();
    if (t < RS_DIG) {
      toff[tile * RS_DIG + t] = run;
      for (int q = 0; q < RS_REP; q++) {
        run += cnt[q][t];
        cnt[q][t] = 0;
      }
    }
    __syncthreads();
  }
  if (t < RS_DIG) gsum[(int64_t)t * gridDim.x + blockIdx.x] = run;
}

// One block per digit: goff[group][digit] = keys of the digit in earlier
// groups, dtot[digit] = all.
__global__ void __launch_bounds__(RS_GMAX) radix_groups(const uint32_t *__restrict__ gsum, int ng,
                                                        uint32_t *__restrict__ goff, uint32_t *__restrict__ dtot) {
  __shared__ uint32_t tmp[RS_GMAX / WAVE + 1];
  const int d = blockIdx.x, g = threadIdx.x;
  uint32_t total;
  const uint32_t pre = block_excl_scan<RS_GMAX, uint32_t>(g < ng ? gsum[(int64_t)d * ng + g] : 0, tmp, &total);
  if (g < ng) goff[(int64_t)g * RS_DIG + d] = pre;
  if (g == 0) dtot[d] = total;
}

// Ranks of a tile's keys by digit, stable.  Wave w holds `it` rounds of 64
// consecutive keys (of positions below cnt) and counts each digit's keys
// among its own in wcnt[w]: a round's lanes with one digit find each other by
// ballots, take the count so far and the lowest adds theirs; LDS operations
// of one wave complete in order, so rounds need no barrier.  Then the counts
// become the tile positions of each wave's first key of a digit, and pos[r]
// the key's position in the sorted tile.  Returns, in threads below RS_DIG,
// where the digit starts in the tile (FULL: of RS_TILE keys), and with `dtot`, in *gbase, in the
// whole output.
template <bool FULL>
__device__ __forceinline__ uint32_t radix_rank(const uint64_t *key, int it, int cnt, int shift,
                                               uint16_t (*wcnt)[RS_DIG], uint64_t *tmp, int32_t *pos,
                                               const uint32_t *dtot, uint32_t *gbase) {
  const int t = threadIdx.x, w = t / WAVE;
  const uint64_t lt = lanemask_lt();
  for (int u = lane_id(); u < RS_DIG; u += WAVE) wcnt[w][u] = 0;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
  for (int r = 0; r < RS_IT; r++) {
    const int p0 = (w * it + r) * WAVE;
    if (!FULL && (r >= it || p0 >= cnt)) continue;  // the same for the whole wave
    const bool valid = FULL || p0 + lane_id() < cnt;
    const int d = (int)((key[r] >> shift) & 0xFF);
    uint64_t peers = FULL ? ~(uint64_t)0 : __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; b++) {
      const int32_t bit = __builtin_amdgcn_sbfe(d, b, 1);  // all ones where bit b is set
      const uint64_t m = __ballot(bit != 0);
      peers &= ~(m ^ (uint64_t)(int64_t)bit);
    }
    const int rw = __popcll(peers & lt);
    const int before = wcnt[w][d];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (valid && rw == 0) wcnt[w][d] = (uint16_t)(before + __popcll(peers));
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    pos[r] = before + rw;
    __builtin_amdgcn_sched_barrier(0);  // one round's ballots at a time in registers
  }
  __syncthreads();
  // both prefixes in one scan over the threads below RS_DIG: the tile's in
  // the low half
  uint64_t mine = 0, inc = 0;
  if (t < RS_DIG) {
    uint32_t sum = 0;
#pragma unroll 4
    for (int q = 0; q < RS_NW; q++) sum += wcnt[q][t];
    mine = ((uint64_t)(dtot ? dtot[t] : 0) << 32) | sum;
    inc = wave_incl_scan(mine);
    if (lane_id() == WAVE - 1) tmp[w] = inc;
  }
  __syncthreads();
  uint64_t pre = inc - mine;
#pragma unroll
  for (int q = 0; q < RS_DIG / WAVE - 1; q++) pre += q < w ? tmp[q] : 0;
  const uint32_t start = (uint32_t)pre;
  *gbase = (uint32_t)(pre >> 32);
  if (t < RS_DIG) {
    uint32_t x = start;
#pragma unroll 4
    for (int q = 0; q < RS_NW; q++) {
      const uint32_t c = wcnt[q][t];
      wcnt[q][t] = (uint16_t)x;
      x += c;
    }
  }
  __syncthreads();
  asm volatile("" : "+s"(shift));  // digits are formed again, not held in registers
#pragma unroll
  for (int r = 0; r < RS_IT; r++) {
    const int p0 = (w * it + r) * WAVE;
    if (!FULL && (r >= it || p0 >= cnt)) continue;
    pos[r] += wcnt[w][(key[r] >> shift) & 0xFF];
  }
  return start;
}

// Stable scatter of one tile.  Blocks of one XCD take consecutive tiles, whose
// runs of a digit adjoin in the output, so that its L2 completes their lines.
template <class P, bool MAP>
__global__ void __launch_bounds__(RS_BS, 8) radix_scatter(const uint64_t *__restrict__ kin, const P *__restrict__ pin,
                                                          uint64_t *__restrict__ kout, P *__restrict__ pout, int64_t n,
                                                          int shift, KeyMap km, int64_t ntiles, int64_t per,
                                                          const uint32_t *__restrict__ toff,
                                                          const uint32_t *__restrict__ goff,
                                                          const uint32_t *__restrict__ dtot) {
  __shared__ uint64_t skey[RS_TILE];
  __shared__ uint16_t wcnt[RS_NW][RS_DIG];
  __shared__ uint32_t dst[RS_DIG];
  __shared__ uint64_t tmp[RS_DIG / WAVE];
  const int64_t tile = (int64_t)(blockIdx.x % NXCD) * (gridDim.x / NXCD) + blockIdx.x / NXCD;
  if (tile >= ntiles) return;
  const int t = threadIdx.x, w = t / WAVE;
  const int64_t base = tile * RS_TILE;
  const int cnt = (int)min((int64_t)RS_TILE, n - base);
  const int p0 = w * RS_IT * WAVE + lane_id();
  const uint64_t *kt = kin + base + p0;
  const P *pt = pin + base + p0;
  // (whole tiles without tests of positions, which cost registers: 64 a
  // thread are two blocks a CU)
  auto body = [&](auto full) {
    constexpr bool FULL = decltype(full)::value;
    uint64_t key[RS_IT];
    P pay[RS_IT];
    int32_t pos[RS_IT];
#pragma unroll
    for (int r = 0; r < RS_IT; r++) key[r] = FULL || p0 + r * WAVE < cnt ? kt[r * WAVE] : 0;
    if (MAP) {
#pragma unroll
      for (int r = 0; r < RS_IT; r++) key[r] = map_key<MAP>(key[r], km);
    }
    uint32_t gbase;
    const uint32_t start = radix_rank<FULL>(key, RS_IT, cnt, shift, wcnt, tmp, pos, dtot, &gbase);
    if (t < RS_DIG) dst[t] = gbase + goff[tile / per * RS_DIG + t] + toff[tile * RS_DIG + t] - start;
#pragma unroll
    for (int r = 0; r < RS_IT; r++)
      if (FULL || p0 + r * WAVE < cnt) skey[pos[r]] = key[r];
    // in flight while the keys are written
#pragma unroll
    for (int r = 0; r < RS_IT; r++) pay[r] = FULL || p0 + r * WAVE < cnt ? pt[r * WAVE] : (P)0;
    __syncthreads();
    uint32_t to[RS_IT];
#pragma unroll
    for (int r = 0; r < RS_IT; r++) {
      const int p = r * RS_BS + t;
      if (FULL || p < cnt) {
        const uint64_t k = skey[p];
        to[r] = dst[(k >> shift) & 0xFF] + (uint32_t)p;
        kout[to[r]] = k;
      }
    }
    __syncthreads();
    P *const spay = reinterpret_cast<P *>(skey);
#pragma unroll
    for (int r = 0; r < RS_IT; r++)
      if (FULL || p0 + r * WAVE < cnt) spay[pos[r]] = pay[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RS_IT; r++) {
      const int p = r * RS_BS + t;
      if (FULL || p < cnt) pout[to[r]] = spay[p];
    }
  };
  if (cnt == RS_TILE) body(std::true_type{});
  else body(std::false_type{});
}

// All passes over at most one tile, in one block and one launch.
template <class P, bool MAP>
__global__ void __launch_bounds__(RS_BS) radix_one_tile(const uint64_t *kin, const P *pin, uint64_t *kout, P *pout,
                                                        int cnt, int passes, KeyMap km) {
  __shared__ uint64_t skey[RS_TILE];
  __shared__ uint16_t wcnt[RS_NW][RS_DIG];
  __shared__ uint64_t tmp[RS_DIG / WAVE];
  const int w = threadIdx.x / WAVE, it = (cnt + RS_BS - 1) / RS_BS;
  P *const spay = reinterpret_cast<P *>(skey);
  uint64_t key[RS_IT];
  P pay[RS_IT];
  int32_t pos[RS_IT];
  auto at = [&](int r) { return r < it ? (w * it + r) * WAVE + lane_id() : RS_TILE; };
#pragma unroll
  for (int r = 0; r < RS_IT; r++) {
    const int p = at(r);
    key[r] = p < cnt ? map_key<MAP>(kin[p], km) : 0;
    pay[r] = p < cnt ? pin[p] : (P)0;
  }
  for (int ps = 0; ps < passes; ps++) {
    uint32_t gbase;
    radix_rank<false>(key, it, cnt, ps * 8, wcnt, tmp, pos, nullptr, &gbase);
#pragma unroll
    for (int r = 0; r < RS_IT; r++)
      if (at(r) < cnt) skey[pos[r]] = key[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RS_IT; r++)
      if (at(r) < cnt) key[r] = skey[at(r)];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RS_IT; r++)
      if (at(r) < cnt) spay[pos[r]] = pay[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RS_IT; r++)
      if (at(r) < cnt) pay[r] = spay[at(r)];
    __syncthreads();
  }
#pragma unroll
  for (int r = 0; r < RS_IT; r++) {
    const int p = at(r);
    if (p < cnt) {
      kout[p] = key[r];
      pout[p] = pay[r];
    }
  }
}

// Sorted pairs end in ka/pa when `passes` is odd, in kb/pb when it is even
// (pass 0 reads kin/pin and writes ka/pa), also where one tile takes all passes
// at once.  kin/pin may be kb/pb, and with one tile either pair.
template <class P, bool MAP>
void radix_sort(Ctx *c, const uint64_t *kin, const P *pin, const KeyMap &km, int64_t n, int passes, uint64_t *ka, P *pa,
                uint64_t *kb, P *pb, hipStream_t s) {
  if (n <= RS_TILE) {
    ProfScope pr(c, "fold.radix_one_tile", 2.0 * (8.0 + sizeof(P)) * n, s);
    radix_one_tile<P, MAP><<<1, RS_BS, 0, s>>>(kin, pin, passes % 2 ? ka : kb, passes % 2 ? pa : pb, (int)n, passes, km);
    SRTC_LAUNCH_CHECK("radix_one_tile");
    return;
  }
  const int64_t ntiles = (n + RS_TILE - 1) / RS_TILE;
  const int64_t per = (ntiles + RS_GMAX - 1) / RS_GMAX;
  const int ng = (int)((ntiles + per - 1) / per);
  Buf tab(c, sizeof(uint32_t) * (size_t)(RS_DIG * (ntiles + 2 * ng + 1)));
  uint32_t *toff = tab.as<uint32_t>(), *gsum = toff + RS_DIG * ntiles, *goff = gsum + RS_DIG * ng;
  uint32_t *dtot = goff + RS_DIG * ng;
  const unsigned grid = (unsigned)((ntiles + NXCD - 1) / NXCD * NXCD);
  for (int ps = 0; ps < passes; ps++) {
    const uint64_t *ki = ps == 0 ? kin : ps % 2 ? ka : kb;
    const P *pi = ps == 0 ? pin : ps % 2 ? pa : pb;
    uint64_t *ko = ps % 2 ? kb : ka;
    P *po = ps % 2 ? pb : pa;
    const bool map = MAP && ps == 0;
    {
      ProfScope pr(c, "fold.radix_hist", 8.0 * n + 4.0 * RS_DIG * ntiles, s);
      if (map) radix_hist<MAP><<<ng, RS_BS, 0, s>>>(ki, n, ps * 8, km, ntiles, per, toff, gsum);
      else radix_hist<false><<<ng, RS_BS, 0, s>>>(ki, n, ps * 8, km, ntiles, per, toff, gsum);
      SRTC_LAUNCH_CHECK("radix_hist");
    }
    radix_groups<<<RS_DIG, RS_GMAX, 0, s>>>(gsum, ng, goff, dtot);
    SRTC_LAUNCH_CHECK("radix_groups");
    {
      ProfScope pr(c, "fold.radix_scatter", 2.0 * (8.0 + sizeof(P)) * n + 4.0 * RS_DIG * ntiles, s);
      if (map)
        radix_scatter<P, MAP><<<grid, RS_BS, 0, s>>>(ki, pi, ko, po, n, ps * 8, km, ntiles, per, toff, goff, dtot);
      else
        radix_scatter<P, false><<<grid, RS_BS, 0, s>>>(ki, pi, ko, po, n, ps * 8, km, ntiles, per, toff, goff, dtot);
      SRTC_LAUNCH_CHECK("radix_scatter");
    }
  }
}

// ------------------------------------------------------------- segments --
// A segment (a run of equal keys) belongs to the thread at its first entry,
// which combines it in sorted (= input) order.  Two passes over the sorted
// pairs, one to count each tile's kept segments and one to write them: the
// second forms the results again, which reads less than storing them would.
// A tile's last segment may run on past the tile: the count pass then brings
// the rest through LDS, a tile's worth at a time by the whole block and the
// next on its way while the segment's thread adds this one, and leaves the
// result for the write pass.  What bounds a long segment is the chain of its
// additions, 31 ns each (2^20 entries of one key, fp32: 146 ms by one thread
// with the bounds known, 329 ms in two passes with a test of each key, 31.5 ms
// so; 2^22 entries, 300 a key, 548, 677 and 359 us).
constexpr int SG_BS = 256, SG_IT = 8, SG_TILE = SG_BS * SG_IT, SG_NW = SG_BS / WAVE;
constexpr int SG_WORDS = SG_TILE / WAVE;

// A tile's values in LDS, with KEYS its keys too (entry r of thread t is
// position r*SG_BS + t; key 0 is the entry's before the tile).  load leaves in
// mask[r] the first entries of segments among the wave's 64 of round r.
template <class SR, bool KEYS> struct SegTile {
  using V = typename SR::val_t;
  using A = typename SR::acc_t;
  uint64_t key[KEYS ? SG_TILE + 1 : 1];
  V val[SG_TILE];
  uint64_t heads[SG_WORDS];  // first entries of segments, by position
  uint64_t last;             // key of a whole tile's last entry
  int32_t runs_on;           // its segment goes on after the tile
  __device__ __forceinline__ void load(const uint64_t *__restrict__ keys, const V *__restrict__ vals, int64_t n,
                                       int64_t base, int cnt, uint64_t *mask) {
    const int t = threadIdx.x;
    uint64_t k[SG_IT], before[SG_IT], next = 0;
    V v[SG_IT];
#pragma unroll
    for (int r = 0; r < SG_IT; r++) {
      const int64_t i = base + min(r * SG_BS + t, cnt - 1);
      k[r] = keys[i];
      v[r] = vals[i];
      before[r] = lane_id() == 0 && i > 0 ? keys[i - 1] : 0;
    }
    const bool ends = t == SG_BS - 1 && base + cnt < n;
    if (ends) next = keys[base + cnt];
#pragma unroll
    for (int r = 0; r < SG_IT; r++) {
      const int p = r * SG_BS + t;
      if (KEYS) key[1 + p] = k[r];
      val[p] = v[r];
      const uint64_t left = dpp_move<0x138, 0xf>(k[r]);  // wave_shr:1
      mask[r] = __ballot(p < cnt && (base + p == 0 || (lane_id() == 0 ? before[r] : left) != k[r]));
      if (lane_id() == 0) heads[r * SG_NW + t / WAVE] = mask[r];
    }
    if (KEYS && t == 0) key[0] = before[0];
    if (t == SG_BS - 1) {
      last = k[SG_IT - 1];
      runs_on = ends && next == k[SG_IT - 1];
    }
    __syncthreads();
  }
  // End within the tile of the segment that starts at this thread's entry p,
  // whose word of heads is m.
  __device__ __forceinline__ int end_of(uint64_t m, int p, int cnt) const {
    m = m >> lane_id() >> 1;
    if (m) return p + __ffsll((unsigned long long)m);
    for (int w = p / WAVE + 1; w * WAVE < cnt; w++) {
      m = heads[w];
      if (m) return w * WAVE + __ffsll((unsigned long long)m) - 1;
    }
    return cnt;
  }
  // Adds entries p .. e-1 to a segment's sum.
  __device__ __forceinline__ void add(int p, int e, A id, A *acc, bool *any) const {
    auto take = [&](V v) {
      if (SR::absent(v, id)) return;
      const A x = SR::HAS_VALS ? (A)v : (A)1;
      *acc = *any ? SR::add(*acc, x) : x;
      *any = true;
    };
    if (p < e) take(val[p++]);  // most segments are one entry
    for (; p + 8 <= e; p += 8) {
      V v[8];
#pragma unroll
      for (int u = 0; u < 8; u++) v[u] = val[p + u];
#pragma unroll
      for (int u = 0; u < 8; u++) take(v[u]);
    }
    for (; p < e; p += 4) {
      V v[4];
#pragma unroll
      for (int u = 0; u < 4; u++) v[u] = val[min(p + u, e - 1)];
#pragma unroll
      for (int u = 0; u < 4; u++)
        if (p + u < e) take(v[u]);
    }
  }
};

// run_val, run_keep [tile]: result of the segment that runs on past the tile,
// and whether it is kept.
template <class SR>
__global__ void __launch_bounds__(SG_BS) seg_count(const uint64_t *__restrict__ keys,
                                                   const typename SR::val_t *__restrict__ vals, int64_t n,
                                                   typename SR::acc_t id, int32_t *__restrict__ tcnt,
                                                   typename SR::val_t *__restrict__ run_val,
                                                   int32_t *__restrict__ run_keep) {
  using V = typename SR::val_t;
  using A = typename SR::acc_t;
  __shared__ int32_t cw[SG_NW];
  const int64_t base = (int64_t)blockIdx.x * SG_TILE;
  const int cnt = (int)min((int64_t)SG_TILE, n - base);
  __shared__ SegTile<SR, false> T;
  uint64_t mask[SG_IT];
  T.load(keys, vals, n, base, cnt, mask);
  int32_t kept = 0;
  bool mine = false, run_any = false;  // this thread's segment runs on: its sum so far
  A run_acc = id;
#pragma unroll
  for (int r = 0; r < SG_IT; r++) {
    const int p = r * SG_BS + threadIdx.x;
    if (!((mask[r] >> lane_id()) & 1)) continue;
    A acc = id;
    bool any = false;
    const int e = T.end_of(mask[r], p, cnt);
    T.add(p, e, id, &acc, &any);
    if (e == cnt && T.runs_on) {
      mine = true;
      run_any = any;
      run_acc = acc;
    } else if (any && !SR::absent(SR::out(acc), id)) {
      kept++;
    }
  }
  if (T.runs_on && __syncthreads_or(mine)) {  // (no thread's where the tile lies inside a segment)
    const uint64_t k = T.last;
    int64_t at = base + SG_TILE;
    V v[SG_IT];
    int same;
    // entries at, at + 1, ... with the same key, up to a tile's worth: values
    // in v, their number in `same` of each thread
    auto fetch = [&]() {
      same = 0;
#pragma unroll
      for (int r = 0; r < SG_IT; r++) {
        const int64_t i = min(at + r * SG_BS + (int)threadIdx.x, n - 1);
        v[r] = vals[i];
        same += at + r * SG_BS + threadIdx.x < n && keys[i] == k ? 1 : 0;
      }
      at += SG_TILE;
    };
    fetch();
    for (bool more = true; more;) {
      // (the barrier of the count ends the reading of the values before)
      const int w = wave_sum(same);
      if (lane_id() == 0) cw[threadIdx.x / WAVE] = w;
      __syncthreads();
      int len = 0;
      for (int q = 0; q < SG_NW; q++) len += cw[q];
#pragma unroll
      for (int r = 0; r < SG_IT; r++) T.val[r * SG_BS + threadIdx.x] = v[r];
      more = len == SG_TILE;
      __syncthreads();
      if (more) fetch();
      if (mine) T.add(0, len, id, &run_acc, &run_any);
    }
    if (mine) {
      const V o = SR::out(run_acc);
      const bool keep = run_any && !SR::absent(o, id);
      run_val[blockIdx.x] = o;
      run_keep[blockIdx.x] = keep;
      kept += keep;
    }
    __syncthreads();
  }
  kept = wave_sum(kept);
  if (lane_id() == 0) cw[threadIdx.x / WAVE] = kept;
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t x = 0;
    for (int q = 0; q < SG_NW; q++) x += cw[q];
    tcnt[blockIdx.x] = x;
  }
}

// Kept segments to their places (toff[tile]: those of earlier tiles), and the
// row pointers: rows after the one of the entry before a segment's first, up
// to its own, start with the segment's place.
template <class SR>
__global__ void __launch_bounds__(SG_BS) seg_write(const uint64_t *__restrict__ keys,
                                                   const typename SR::val_t *__restrict__ vals, int64_t n,
                                                   typename SR::acc_t id, const int64_t *__restrict__ toff,
                                                   const typename SR::val_t *__restrict__ run_val,
                                                   const int32_t *__restrict__ run_keep, int64_t nrows, uint64_t ncols,
                                                   uint64_t magic, int32_t *__restrict__ col,
                                                   typename SR::val_t *__restrict__ val, int64_t *__restrict__ rowptr) {
  using A = typename SR::acc_t;
  __shared__ int32_t cw[SG_WORDS];
  const int w = threadIdx.x / WAVE;
  const int64_t base = (int64_t)blockIdx.x * SG_TILE;
  const int cnt = (int)min((int64_t)SG_TILE, n - base);
  __shared__ SegTile<SR, true> T;
  uint64_t mask[SG_IT];
  T.load(keys, vals, n, base, cnt, mask);
  typename SR::val_t o[SG_IT];
  uint32_t below[SG_IT];
  uint32_t heads = 0, kept = 0;
#pragma unroll
  for (int r = 0; r < SG_IT; r++) {
    const int p = r * SG_BS + threadIdx.x;
    const bool head = (mask[r] >> lane_id()) & 1;
    bool k = false;
    if (head) {
      const int e = T.end_of(mask[r], p, cnt);
      if (e == cnt && T.runs_on) {
        o[r] = run_val[blockIdx.x];
        k = run_keep[blockIdx.x] != 0;
      } else {
        A acc = id;
        T.add(p, e, id, &acc, &k);
        o[r] = SR::out(acc);
        k = k && !SR::absent(o[r], id);
      }
    }
    heads |= head ? 1u << r : 0;
    kept |= k ? 1u << r : 0;
    const uint64_t m = __ballot(k);
    below[r] = (uint32_t)__popcll(m & lanemask_lt());
    if (lane_id() == 0) cw[r * SG_NW + w] = __popcll(m);
  }
  __syncthreads();
  if (w == 0) {
    static_assert(SG_WORDS <= WAVE, "one wave scans the tile's counts");
    const int32_t x = lane_id() < SG_WORDS ? cw[lane_id()] : 0;
    const int32_t inc = wave_incl_scan(x);
    if (lane_id() < SG_WORDS) cw[lane_id()] = inc - x;
  }
  __syncthreads();
  const int64_t t0 = toff[blockIdx.x];
#pragma unroll
  for (int r = 0; r < SG_IT; r++) {
    const int64_t i = base + r * SG_BS + threadIdx.x;
    if (i >= n) continue;
    const int64_t at = t0 + cw[r * SG_NW + w] + below[r];
    if (!((heads >> r) & 1) && i != n - 1) continue;
    uint64_t c;
    const uint64_t kr = T.key[1 + r * SG_BS + threadIdx.x], kp = T.key[r * SG_BS + threadIdx.x];
    const uint64_t row = fast_div(kr, ncols, magic, &c);
    if ((kept >> r) & 1) {
      col[at] = (int32_t)c;
      val[at] = o[r];
    }
    if (i == 0) {
      for (uint64_t q = 0; q <= row; q++) rowptr[q] = 0;
    } else if (kp < row * ncols) {
      uint64_t pc;
      for (uint64_t q = fast_div(kp, ncols, magic, &pc) + 1; q <= row; q++) rowptr[q] = at;
    }
    if (i == n - 1) {
      const int64_t end = at + ((kept >> r) & 1);
      for (int64_t q = (int64_t)row + 1; q <= nrows; q++) rowptr[q] = end;
    }
  }
}

__global__ void csr_keys_kernel(const int64_t *rowptr, const int32_t *col, int64_t m, int64_t ncols,
                                int64_t *keys) {
  // one wave per row
  const int64_t wid = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / WAVE;
  const int64_t nw = ((int64_t)gridDim.x * blockDim.x) / WAVE;
  for (int64_t i = wid; i < m; i += nw)
    for (int64_t p = rowptr[i] + lane_id(); p < rowptr[i + 1]; p += WAVE) keys[p] = i * ncols + col[p];
}

inline unsigned grid_for(int64_t n, int bs = 256, int64_t cap = 65536) {
  int64_t g = (n + bs - 1) / bs;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (unsigned)g;
}

template <class SR>
void seg_count_launch(const uint64_t *keys, const void *vals, int64_t n, IdVal id, int32_t *tcnt, void *run_val,
                      int32_t *run_keep, hipStream_t s) {
  seg_count<SR><<<(unsigned)((n + SG_TILE - 1) / SG_TILE), SG_BS, 0, s>>>(
      keys, (const typename SR::val_t *)vals, n, id_as<SR>(id), tcnt, (typename SR::val_t *)run_val, run_keep);
  SRTC_LAUNCH_CHECK("seg_count");
}

uint64_t magic_of(uint64_t d) { return ~(uint64_t)0 / std::max<uint64_t>(d, 1); }

template <class SR>
void seg_write_launch(const uint64_t *keys, const void *vals, int64_t n, IdVal id, const int64_t *toff,
                      const void *run_val, const int32_t *run_keep, int64_t nrows, int64_t ncols, int32_t *col, void *val,
                      int64_t *rowptr, hipStream_t s) {
  using V = typename SR::val_t;
  seg_write<SR><<<(unsigned)((n + SG_TILE - 1) / SG_TILE), SG_BS, 0, s>>>(
      keys, (const V *)vals, n, id_as<SR>(id), toff, (const V *)run_val, run_keep, nrows, (uint64_t)ncols,
      magic_of((uint64_t)ncols), col, (V *)val, rowptr);
  SRTC_LAUNCH_CHECK("seg_write");
}

}  // namespace

KeyMap key_map(int order, const int64_t *dims, int nrow_modes, const int *row_modes, int ncol_modes,
               const int *col_modes) {
  KeyMap a{};
  a.order = order;
  for (int m = 0; m < order; m++) {
    a.dim[m] = (uint64_t)dims[m];
    a.magic[m] = magic_of(a.dim[m]);
  }
  uint64_t mul = 1;
  for (int q = ncol_modes - 1; q >= 0; q--) {
    a.mul[col_modes[q]] += mul;  // (a letter of all three tensors is a row and a column mode)
    mul *= a.dim[col_modes[q]];
  }
  for (int q = nrow_modes - 1; q >= 0; q--) {
    a.mul[row_modes[q]] += mul;
    mul *= a.dim[row_modes[q]];
  }
  return a;
}

void radix_sort_pairs(Ctx *c, int64_t *keys, uint32_t *payload, int64_t n, int bits,
                      hipStream_t s) {
  if (n <= 1 || bits <= 0) return;
  // the spare buffers take the odd passes: pass 0 writes them
  const bool one = n <= RS_TILE;
  const int passes = (bits + 7) / 8;
  uint64_t *k = reinterpret_cast<uint64_t *>(keys);
  if (one) {  // in place (the block has read all pairs before it writes)
    radix_sort<uint32_t, false>(c, k, payload, KeyMap{}, n, passes, k, payload, k, payload, s);
    return;
  }
  Buf k2(c, sizeof(uint64_t) * (size_t)n), p2(c, sizeof(uint32_t) * (size_t)n);
  radix_sort<uint32_t, false>(c, k, payload, KeyMap{}, n, passes, k2.as<uint64_t>(), p2.as<uint32_t>(), k, payload, s);
  if (passes % 2) {
    SRTC_HIP(hipMemcpyAsync(keys, k2.p, sizeof(uint64_t) * (size_t)n, hipMemcpyDeviceToDevice, s));
    SRTC_HIP(hipMemcpyAsync(payload, p2.p, sizeof(uint32_t) * (size_t)n, hipMemcpyDeviceToDevice, s));
  }
}

void fold_keys_to_csr(Ctx *c, int sr, int dt, IdVal id, const KeyMap *map, const int64_t *keys_in, const void *vals,
                      int64_t nnz, int64_t nrows, int64_t ncols, CsrOut *out, hipStream_t s) {
  if (nnz >= (int64_t(1) << 32)) fail(SRTC_ERR_UNSUPPORTED, "fold: more than 2^32 entries");
  const size_t es = dtype_size(dt);
  out->m = nrows;
  out->n = ncols;
  out->rowptr = Buf(c, sizeof(int64_t) * (size_t)(nrows + 1), out->kind);
  if (nnz == 0) {
    fill_i64(out->rowptr.as<int64_t>(), nrows + 1, 0, s);
    out->nnz = 0;
    out->col = Buf(c, 4, out->kind);
    out->val = Buf(c, es, out->kind);
    return;
  }
  const unsigned __int128 span = (unsigned __int128)nrows * (unsigned __int128)ncols;
  int bits = 1;
  while (bits < 63 && ((unsigned __int128)1 << bits) < span) bits++;
  c->tracef("fold: %lld keys, %lld x %lld, %d key bits", (long long)nnz, (long long)nrows, (long long)ncols, bits);
  // sort (key, value)
  const int passes = (bits + 7) / 8;
  const size_t two = passes > 1 ? 2 : 1;
  Buf kbuf(c, sizeof(uint64_t) * (size_t)nnz * two), vbuf(c, es * (size_t)nnz * two);
  uint64_t *ka = kbuf.as<uint64_t>(), *kb = ka + (two - 1) * nnz;
  const uint64_t *kin = reinterpret_cast<const uint64_t *>(keys_in);
  auto sort = [&](auto p0) {
    using P = decltype(p0);
    P *va = vbuf.as<P>(), *vb = va + (two - 1) * nnz;
    if (map) radix_sort<P, true>(c, kin, (const P *)vals, *map, nnz, passes, ka, va, kb, vb, s);
    else radix_sort<P, false>(c, kin, (const P *)vals, KeyMap{}, nnz, passes, ka, va, kb, vb, s);
  };
  if (es == 8) sort(uint64_t{});
  else if (es == 4) sort(uint32_t{});
  else sort(uint8_t{});
  const uint64_t *keys = passes % 2 ? ka : kb;
  const void *sval = passes % 2 ? vbuf.p : (const void *)(vbuf.as<char>() + es * (size_t)nnz * (two - 1));
  // segments of equal keys
  const int64_t nst = (nnz + SG_TILE - 1) / SG_TILE;
  // per tile: first place, count, and the segment that runs on
  Buf toff(c, sizeof(int64_t) * (size_t)(nst + 1)), run(c, (8 + 2 * sizeof(int32_t)) * (size_t)nst);
  int32_t *tcnt = reinterpret_cast<int32_t *>(run.as<char>() + 8 * (size_t)nst), *run_keep = tcnt + nst;
  SRTC_DISPATCH_SR(sr, dt, seg_count_launch, keys, sval, nnz, id, tcnt, run.p, run_keep, s);
  excl_scan_i32(c, tcnt, toff.as<int64_t>(), nst, s);
  const int64_t total = read_i64(c, toff.as<int64_t>() + nst, s);
  c->tracef("fold: %lld entries after combining duplicates", (long long)total);
  out->nnz = total;
  out->col = Buf(c, sizeof(int32_t) * (size_t)(total > 0 ? total : 1), out->kind);
  out->val = Buf(c, es * (size_t)(total > 0 ? total : 1), out->kind);
  SRTC_DISPATCH_SR(sr, dt, seg_write_launch, keys, sval, nnz, id, toff.as<int64_t>(), run.p, run_keep, nrows, ncols,
                   out->col.as<int32_t>(), out->val.p, out->rowptr.as<int64_t>(), s);
}

void csr_to_keys(const CsrView &a, int64_t *keys, hipStream_t s) {
  if (a.nnz == 0 || a.m == 0) return;
  csr_keys_kernel<<<grid_for(a.m * WAVE, 256, 16384), 256, 0, s>>>(a.rowptr, a.col, a.m, a.n, keys);
  SRTC_LAUNCH_CHECK("csr_keys_kernel");
}

}  // namespace srtc
