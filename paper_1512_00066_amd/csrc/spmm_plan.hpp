// Work items of a sparse x dense product (rows cut into pieces of at most T
// nonzeros); built once per matrix and reused by every fixpoint step.
#pragma once

#include "internal.hpp"

namespace srtc {

struct SpmmPlan {
  Ctx *ctx = nullptr;
  int G = 64;          // lanes per item (power of two covering the width)
  int64_t T = 256;     // nonzeros per item
  int64_t max_items = 0;
  int64_t grid_cap = 4096;
  bool may_split = true;
  int grain = 256;         // nonzeros of an item summed before they join its total
  bool batched = false;    // rows of several instances (set before build)
  Buf cnt, pcnt, ioff, poff, irow_b, ibeg_b, ufirst_b, ipidx_b, partial_b;
  const int32_t *irow = nullptr;
  const int64_t *ibeg = nullptr, *ufirst = nullptr, *ipidx = nullptr, *nitems = nullptr;
  void *partial = nullptr;
  int64_t rows = 0;         // rows of A
  int64_t ucost = 0;        // work of a unit: nonzeros and a constant per item
  int64_t nunits = 0;       // units of items taken by one wave each (0: none)
  int64_t max_partial = 0;  // rows of s_width accumulators for split rows
  // item length, lanes per item and buffer sizes for A and s_width
  void shape(Ctx *c, const CsrView &A, int64_t s_width);
  // shape, then allocate the buffers from the context and fill them
  void build(Ctx *c, const CsrView &A, int64_t s_width, hipStream_t st);
  // bytes of one caller-supplied buffer holding every plan array
  int64_t workspace_bytes(int64_t s_width) const;
  // shape() first; lays the plan out in ws (workspace_bytes, 256-byte
  // aligned) and fills it; allocates nothing
  void build_in(const CsrView &A, int64_t s_width, void *ws, hipStream_t st);

 private:
  void fill(const CsrView &A, int64_t *cnt_p, int64_t *pcnt_p, int64_t *ioff_p, int64_t *poff_p, int64_t *sums,
            int32_t *irow_p, int64_t *ibeg_p, int64_t *ufirst_p, int64_t *ipidx_p, void *partial_p, hipStream_t st);
};

// The (unit, chunk of 64 columns) pairs that one wave of a wide product takes.
// With at least eight chunks the first turns go to the chunks of the wave's
// XCD (block id mod 8) and the others to the chunks shared by all; with fewer
// every chunk is shared.  Shared pairs go chunk by chunk, or, where rows of X
// are no whole lines of 128 bytes and neighbouring chunks share lines, unit by
// unit (20,000 rows of 30 nonzeros, int32, product alone: 300 columns 138 us
// chunk by chunk, 124 unit by unit; 320 columns 103 and 110).  There are fewer
// than 2^31 pairs and a turn advances by at most the grid's waves, so unsigned
// numbers hold the turn past the last.
struct UnitTurns {
  uint32_t nunits, t, mine, all, st_own, st_all, w_all, shared, rest, xcd;
  bool own, by_unit;
  __host__ __device__ UnitTurns(uint32_t nunits_, uint32_t nch, uint32_t grid, uint32_t wpb, uint32_t block,
                                uint32_t wave, bool by_unit_)
      : nunits(nunits_), xcd(block % 8), by_unit(by_unit_) {
    own = nch >= 8 && grid % 8 == 0;
    mine = own ? nunits * (nch / 8) : 0;
    shared = own ? nch / 8 * 8 : 0;
    rest = nch - shared;
    all = nunits * rest;
    st_own = grid / 8 * wpb;
    st_all = grid * wpb;
    w_all = block * wpb + wave;
    t = own ? block / 8 * wpb + wave : w_all;
  }
  __host__ __device__ bool next(int32_t *unit, int32_t *chunk) {
    if (own && t >= mine) {
      own = false;
      t = w_all;
    }
    if (!own && t >= all) return false;
    const bool unit_first = by_unit && !own;
    const uint32_t d = unit_first ? rest : nunits, hi = t / d, lo = t - hi * d;
    const uint32_t ch = unit_first ? lo : hi;
    *unit = (int32_t)(unit_first ? hi : lo);
    *chunk = (int32_t)(own ? xcd + 8 * ch : shared + ch);
    t += own ? st_own : st_all;
    return true;
  }
};

// mode 0: Y = A (x) X (accumulate: Y (+)= A (x) X); mode 1: fixpoint step
// Y = X (+) A (x) X raising *changed (and per-instance flags) on change.
// In mode 1, rin (one byte per row, optional) limits the gathers to rows
// that changed in the previous step, and rout (optional) marks the rows
// this step changed; both need an idempotent additive op.
void spmm_with_plan(const SpmmPlan &pl, int sr, int dt, IdVal id, const CsrView &A, const void *X,
                    int64_t s_width, void *Y, int mode, int accumulate, int32_t *changed, const int32_t *row_inst,
                    const uint8_t *inst_active, int32_t *inst_changed, hipStream_t st, const uint8_t *rin = nullptr,
                    uint8_t *rout = nullptr);

// The sparse x dense product with its plan in the library's fixed per-device
// buffer: Y = A (x) X (accumulate: Y (+)= A (x) X).  No device memory is
// allocated; SRTC_ERR_TOO_LARGE if the plan needs more than
// spmm_fixed_scratch_bytes().  Calls that overlap on one device race.
void spmm_fixed(Ctx *c, int sr, int dt, IdVal id, const CsrView &A, const void *X, int64_t s_width, void *Y,
                int accumulate, hipStream_t st);
size_t spmm_fixed_scratch_bytes();
// Device address of the fixed buffer on `device` (the current device),
// looked up once per device and kept for the life of the process.
void *spmm_fixed_scratch_init(int device);

}  // namespace srtc
