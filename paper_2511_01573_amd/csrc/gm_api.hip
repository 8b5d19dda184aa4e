// gm_api.hip -- libgm host driver (the C ABI of include/gm.h) and the control
// kernels of the breadth-first adaptive loop (arXiv 2511.01573, Sec. 3):
//
//   init      initial uniform partition into SoA storage
//   rule      (gm_rule.hip) Q, err, split axis of every active region
//   reduce    I = I_fin + sum Q, E = E_fin + sum err, T, stopping rule (Sec. 4)
//   classify  retire regions whose error share is negligible (+ guards),
//             per-tile keep counts and retired partial sums
//   scan      tile offsets of the kept regions; commit the retired sums
//   list      the kept regions in stable order; the next iteration's rule
//             kernel halves them along their axes (child "-" of entry p is
//             region p, child "+" region n_keep + p); retired leaves appended
//             in gradient mode
//
// Active sets of at most kStepRegions regions do everything after the rule in
// one workgroup (step_kernel).
//
// All iteration state lives in a device Status block; kernels read the active
// count and the ping-pong index from it and return at once when a final
// status is set, so an iteration is a fixed sequence of launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "../../include/gm.h"
#include "gm_common.hpp"
#include "gm_internal.hpp"

namespace gm {

// ---------------------------------------------------------------------------
// Control kernels.
// ---------------------------------------------------------------------------
constexpr int kTile = 1024;        // regions per classify tile
constexpr int kTileThreads = 256;  // 4 regions per thread per tile
constexpr int kMaxRuleGrid = 16384;
constexpr int kPruneBins = 66;  // budget factors 2^1 .. 2^64, bin 65 = beyond
constexpr int kMaxTileGrid = 8192;
constexpr int64_t kHostListCoords = 32768;  // region lists up to this many coordinates (gm_eval_regions)
// The one-workgroup bookkeeping kernel (step_kernel): its threads, and the
// largest active set it takes.
constexpr int kStepThreads = 1024;
constexpr int kStepTiles = 32;
constexpr int64_t kStepRegions = (int64_t)kStepTiles * kTile;

struct InitArgs {
  double* C;
  double* H;
  uint16_t* L;
  int64_t cap;
  int64_t n0;
  int d;
  int m;  // cells per axis = 2^m
  double lo[kMaxDim];
  double half[kMaxDim];  // (hi - lo) / 2
  Status* st;
  Status status;  // the run's first status block
};

// Words of the status block (it is copied by the word).
constexpr int kStatusWords = sizeof(Status) / 8;
static_assert(sizeof(Status) % 8 == 0 && kStatusWords <= 64, "one wavefront copies the status");

// Initial partition and status block.
__global__ void init_kernel(InitArgs A) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *A.st = A.status;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t mask = ((int64_t)1 << A.m) - 1;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < A.n0; t += stride) {
    if (!GM_INB(t, A.cap)) continue;
    for (int j = 0; j < A.d; ++j) {
      const int64_t kj = (t >> (A.m * j)) & mask;
      const double hj = ldexp(A.half[j], -A.m);
      A.H[j * A.cap + t] = hj;
      A.C[j * A.cap + t] = fma((double)(2 * kj + 1), hj, A.lo[j]);
    }
    A.L[t] = (uint16_t)(A.m * A.d);
  }
}

// A caller's region list, row-major as it was copied in, into the store's
// coordinate-major layout (d strided reads per region: at the list sizes that a
// host array allows they stay in the L2), and its split axes as the caller's
// 32-bit integers on the way out.
__global__ void list_in_kernel(const double* c, const double* h, const int32_t* lvl, int d,
                               int64_t n, double* C, double* H, uint16_t* L) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  for (int j = 0; j < d; ++j) {
    C[j * n + r] = c[r * d + j];
    H[j * n + r] = h[r * d + j];
  }
  L[r] = (uint16_t)lvl[r];
}

__global__ void list_out_kernel(const uint8_t* axis, int64_t n, int32_t* out) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r < n) out[r] = axis[r];
}

// Host copies of the status block: the last kernel of an iteration stores the
// block and then the iteration's number into a slot of pinned host memory that
// the host reads, so a status read costs neither a copy nor a stream
// synchronisation (together 12 to 20 us on the host, with the GPU idle behind
// them).  Called by the whole first wavefront; the number is stored after the
// words are visible to the host.
struct alignas(256) StatusSlot {
  int64_t words[kStatusWords];
  int64_t seq;
};
struct Mirror {
  StatusSlot* slot;  // null: the host copies the block itself
  int64_t seq;
};

__device__ __forceinline__ void mirror_status(const Mirror& M, const Status* st) {
  if (M.slot == nullptr) return;
  if (threadIdx.x < kStatusWords)
    __hip_atomic_store(&M.slot->words[threadIdx.x], ((const int64_t*)st)[threadIdx.x],
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __threadfence_system();
  if (threadIdx.x == 0)
    __hip_atomic_store(&M.slot->seq, M.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Thread 0 of the reduction: the waves' sums, the retired totals, the
// iteration counters and the stopping rule (Sec. 4).
__device__ __forceinline__ void reduce_commit(Status* st, dd q, dd e, const dd* sq, const dd* se,
                                              int nw) {
  for (int w = 1; w < nw; ++w) {
    q = dd_sum(q, sq[w]);
    e = dd_sum(e, se[w]);
  }
  q = dd_sum(q, dd{st->ifin_hi, st->ifin_lo});
  e = dd_sum(e, dd{st->efin_hi, st->efin_lo});
  const double I = dd_val(q), E = dd_val(e);
  const int64_t n = st->n_active;
  if (st->pending) {  // the rule kernel has written the set's records
    st->pending = 0;
    st->buf = 1 - st->buf;
    st->split = 1;
    st->n_par = st->n_keep;
  }
  st->iter += 1;
  st->regions_evaluated += n;
  if (n > st->max_active) st->max_active = n;
  if (st->nonfinite) {
    st->I = NAN;
    st->E = NAN;
    st->status = GM_NONFINITE;
    st->done = 1;
    return;
  }
  const double T = fmax(st->abs_tol, st->rel_tol * fabs(I));
  st->I = I;
  st->E = E;
  st->T = T;
  if (E <= T) {
    st->status = GM_OK;
    st->done = 1;
  } else if (st->iter >= st->max_iters) {
    st->status = GM_MAX_ITERS;
    st->done = 1;
  }
}

// Global reduction of the rule kernel's block partials and the stopping rule
// (the body of reduce_kernel and of step_kernel, kReduceLanes threads): thread
// v adds partials v, v + kReduceLanes, ..., the wavefronts' sums are combined
// in order (those that had any; adding a zero sum changes nothing).
constexpr int kReduceLanes = 1024;

__device__ __forceinline__ void reduce_body(Status* st, const double* partials, int np,
                                            int64_t* hist) {
  const int tid = threadIdx.x;
  for (int b = tid; b < kPruneBins; b += kReduceLanes) hist[b] = 0;
  __shared__ dd sq[kReduceLanes / 64], se[kReduceLanes / 64];
  const int nw = np >= kReduceLanes ? kReduceLanes / 64 : (np + 63) / 64;
  if (tid < 64 * nw) {
    dd q = {0.0, 0.0}, e = {0.0, 0.0};
    for (int p = tid; p < np; p += kReduceLanes) {
      q = dd_sum(q, dd{partials[4 * p + 0], partials[4 * p + 1]});
      e = dd_sum(e, dd{partials[4 * p + 2], partials[4 * p + 3]});
    }
    q = wave_sum_dd(q);
    e = wave_sum_dd(e);
    if ((tid & 63) == 0) {
      sq[tid >> 6] = q;
      se[tid >> 6] = e;
    }
  }
  __syncthreads();
  if (tid == 0) reduce_commit(st, sq[0], se[0], sq, se, nw);
}

__global__ __launch_bounds__(1024) void reduce_kernel(Status* st, const double* partials, int np,
                                                      int64_t* hist) {
  if (st->done) return;
  reduce_body(st, partials, np, hist);
}

struct ClassifyArgs {
  Status* st;
  const uint16_t* L[2];
  const double* Q;
  const double* ERR;
  const uint8_t* AXIS;
  uint8_t* FLAG;  // 1 = retired
  int64_t* TK;    // kept per tile
  double* TQ;     // retired Q per tile (double-double)
  double* TE;     // retired err per tile
  int64_t* HIST;  // kept regions per smallest sufficient budget factor (pruning)
};

// Smallest k in 1..64 with err <= T 2^(k - lvl), 65 if none: the budget factor
// that would retire the region (memory-pressure pruning).
__device__ __forceinline__ int prune_level(double err, double T, int lvl) {
  for (int k = 1; k <= 64; ++k)
    if (err <= ldexp(T, k - lvl)) return k;
  return 65;
}

// Classifier (reading of Sec. 3's "discards subregions whose contribution to
// the error is negligible"): retire when err <= T * 2^-lvl (the region's
// error density is within the global budget), when |I| + err == |I|
// (round-off guard), or when halving along the axis changes nothing
// (geometry guard, flagged by the rule kernel in bit 7 of the axis byte).
// With memory-pressure pruning on, the first pass also histograms the kept
// regions by the budget factor that would retire them; when the kept set
// overflows the store the scan kernel picks the smallest sufficient factor
// 2^k and the second pass (SECOND) classifies again with err <= T 2^(k - lvl)
// added to the retire test.
// Blocks of kTileThreads threads, a tile at a time.
__device__ __forceinline__ bool retires(double err, double T, double aI, int lvl, uint8_t ax) {
  return (err <= ldexp(T, -lvl)) || (aI + err == aI) || (ax & kGeoBit);
}

template <bool SECOND>
__global__ __launch_bounds__(kTileThreads) void classify_kernel(ClassifyArgs A) {
  const Status* st = A.st;
  if (st->done) return;
  if (SECOND && !st->reclassify) return;
  const int64_t n = st->n_active;
  const double T = st->T;
  const double aI = fabs(st->I);
  const int prune_k = SECOND ? st->prune_k : 0;
  const bool hist_on = !SECOND && st->prune_on;
  const uint16_t* __restrict__ L = A.L[st->buf];
  const int split = st->split;
  const int64_t npar = st->n_par;
  const int64_t nt = (n + kTile - 1) / kTile;
  __shared__ int64_t sk[kTileThreads / 64];
  __shared__ dd sq[kTileThreads / 64], se[kTileThreads / 64];
  __shared__ unsigned int shist[kPruneBins];
  if (hist_on) {
    for (int b = threadIdx.x; b < kPruneBins; b += kTileThreads) shist[b] = 0;
    __syncthreads();
  }
  for (int64_t tile = blockIdx.x; tile < nt; tile += gridDim.x) {
    int64_t keep = 0;
    dd q = {0.0, 0.0}, e = {0.0, 0.0};
    // Every row's inputs are loaded first, by every lane (index clamped into
    // the set, Q whether or not it is needed), so the tile costs one memory
    // round trip instead of two per row (the flag stores would otherwise keep
    // the next row's loads behind them).
    constexpr int kRows = kTile / kTileThreads;
    double errv[kRows], qv[kRows];
    int lvlv[kRows];
    uint8_t axv[kRows];
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
      const int64_t r = tile * kTile + k * kTileThreads + threadIdx.x;
      const int64_t rc = r < n ? r : n - 1;
      errv[k] = A.ERR[rc];
      qv[k] = A.Q[rc];
      axv[k] = A.AXIS[rc];
      lvlv[k] = L[(split && rc >= npar) ? rc - npar : rc];  // (+ split below)
    }
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
      const int64_t r = tile * kTile + k * kTileThreads + threadIdx.x;
      if (r < n && GM_INB(r, st->cap)) {
        const double err = errv[k];
        const int lvl = lvlv[k] + (split ? 1 : 0);
        bool fin = retires(err, T, aI, lvl, axv[k]);
        if (SECOND && !fin) fin = err <= ldexp(T, prune_k - lvl);
        if (hist_on && !fin) atomicAdd(&shist[prune_level(err, T, lvl)], 1u);
        A.FLAG[r] = fin ? 1 : 0;
        if (fin) {
          dd_add(q, qv[k]);
          dd_add(e, err);
        } else {
          keep += 1;
        }
      }
    }
    keep = wave_sum_i64(keep);
    q = wave_sum_dd(q);
    e = wave_sum_dd(e);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
      sk[w] = keep;
      sq[w] = q;
      se[w] = e;
    }
    __syncthreads();
    if (threadIdx.x == 0 && GM_INB(tile, (st->cap + kTile - 1) / kTile + 1)) {
      int64_t kk = sk[0];
      dd tq = sq[0], te = se[0];
      for (int i = 1; i < kTileThreads / 64; ++i) {
        kk += sk[i];
        tq = dd_sum(tq, sq[i]);
        te = dd_sum(te, se[i]);
      }
      A.TK[tile] = kk;
      A.TQ[2 * tile] = tq.hi;
      A.TQ[2 * tile + 1] = tq.lo;
      A.TE[2 * tile] = te.hi;
      A.TE[2 * tile + 1] = te.lo;
    }
    __syncthreads();
  }
  if (hist_on) {
    for (int b = threadIdx.x; b < kPruneBins; b += kTileThreads)
      if (shist[b]) atomicAdd((unsigned long long*)&A.HIST[b], (unsigned long long)shist[b]);
  }
}

// Exclusive scan of the per-tile keep counts (one workgroup), capacity and
// precision checks, and the commit of the retired partial sums.  When the
// kept set overflows the store and pruning is on, the first pass picks the
// budget factor and leaves the commit to the second pass (SECOND), which runs
// after the second classification.
template <bool SECOND>
__device__ void scan_commit(Status* st, int64_t total, dd tq, dd te, const int64_t* HIST);

// Thread t takes `per` consecutive tiles.
template <bool SECOND>
__global__ __launch_bounds__(1024) void scan_kernel(Status* st, const int64_t* TK, int64_t* TOFF,
                                                    const double* TQ, const double* TE,
                                                    const int64_t* HIST) {
  if (st->done) return;
  if (SECOND && !st->reclassify) return;
  constexpr int nthr = 1024;
  const int64_t n = st->n_active;
  const int64_t nt = (n + kTile - 1) / kTile;
  const int64_t per = (nt + nthr - 1) / nthr;
  const int64_t t0 = (int64_t)threadIdx.x * per;
  int64_t t1 = t0 + per < nt ? t0 + per : nt;
  if (t1 > t0 && !GM_INB(t1 - 1, (st->cap + kTile - 1) / kTile + 1)) t1 = t0;
  int64_t sum = 0;
  dd q = {0.0, 0.0}, e = {0.0, 0.0};
  for (int64_t t = t0; t < t1; ++t) {
    sum += TK[t];
    q = dd_sum(q, dd{TQ[2 * t], TQ[2 * t + 1]});
    e = dd_sum(e, dd{TE[2 * t], TE[2 * t + 1]});
  }
  // Inclusive scan within the wavefront.
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int64_t inc = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int64_t y = __shfl_up(inc, o, 64);
    if (lane >= o) inc += y;
  }
  __shared__ int64_t wtot[16];
  __shared__ dd sq[16], se[16];
  q = wave_sum_dd(q);
  e = wave_sum_dd(e);
  if (lane == 63) wtot[w] = inc;
  if (lane == 0) {
    sq[w] = q;
    se[w] = e;
  }
  __syncthreads();
  int64_t woff = 0, total = 0;
  for (int i = 0; i < nthr / 64; ++i) {
    if (i < w) woff += wtot[i];
    total += wtot[i];
  }
  int64_t run = woff + inc - sum;
  for (int64_t t = t0; t < t1; ++t) {
    TOFF[t] = run;
    run += TK[t];
  }
  if (threadIdx.x != 0) return;
  dd tq = sq[0], te = se[0];
  for (int i = 1; i < nthr / 64; ++i) {
    tq = dd_sum(tq, sq[i]);
    te = dd_sum(te, se[i]);
  }
  scan_commit<SECOND>(st, total, tq, te, HIST);
}

// Thread 0 of the scan: capacity and precision checks, the choice of the
// pruning factor, the commit of the retired sums and the new active count.
template <bool SECOND>
__device__ void scan_commit(Status* st, int64_t total, dd tq, dd te, const int64_t* HIST) {
  const int64_t n = st->n_active;
  if (SECOND) st->reclassify = 0;
  if (total == 0) {
    // a run that pruned and then ran out of regions was limited by the store
    st->status = st->pruned ? GM_MAX_REGIONS : GM_PRECISION_LIMIT;
    st->done = 1;
    return;
  }
  if (2 * total > st->cap) {
    if (!SECOND && st->prune_on) {
      int64_t above = total;
      for (int k = 1; k <= 64; ++k) {
        above -= HIST[k];
        if (2 * above <= st->cap) {
          st->prune_k = k;
          st->pruned = 1;
          st->reclassify = 1;
          return;
        }
      }
    }
    st->status = GM_MAX_REGIONS;
    st->done = 1;
    return;
  }
  const dd fi = dd_sum(dd{st->ifin_hi, st->ifin_lo}, tq);
  const dd fe = dd_sum(dd{st->efin_hi, st->efin_lo}, te);
  st->ifin_hi = fi.hi;
  st->ifin_lo = fi.lo;
  st->efin_hi = fe.hi;
  st->efin_lo = fe.lo;
  st->finished += n - total;
  st->leaf_base = st->leaf_count;
  st->leaf_count += n - total;
  st->n_prev = n;
  st->n_keep = total;
  st->n_active = 2 * total;
  st->pending = 1;
}

// The set being split, after the scan (records in `buf`, the kept list to the
// other buffer), and the leaf store of gradient mode.
struct ListArgs {
  Status* st;
  double* C[2];
  double* H[2];
  uint16_t* L[2];
  uint8_t* PAX[2];
  int64_t cap;
  const uint8_t* AXIS;
  const uint8_t* FLAG;
  const int64_t* TOFF;
  // retired leaves (SoA, capacity leaf_cap); null outside gradient mode
  double* LC;
  double* LH;
  uint16_t* LL;
  int64_t leaf_cap;
};

// Kept region r with split axis `axis` as entry p of the kept list.  (p < cap /
// 2 holds by the scan's capacity check; the guard keeps the store inside the
// list whatever the offsets hold.)
__device__ __forceinline__ void list_kept(int64_t* idx, int64_t cap, int64_t p, int64_t r,
                                          uint8_t axis) {
  if (GM_GUARD(p, cap / 2)) idx[p] = (r << 8) | (axis & kAxisMask);
}

// Stable compaction (Sec. 3: filtering and splitting fused): the kept regions'
// list.  Ranks inside a tile come from wavefront ballots and an LDS prefix over
// the four wavefronts; the tile's base offset comes from the scan kernel.  D > 0
// (gradient mode): the retired regions of dimension D are appended to the leaf
// store as well; KEPT = false leaves the list alone (step_kernel has written it).
// Without leaves it moves 2 B in and 8 B out per kept region, which at the sizes
// that matter costs less than the launch (8 us at 10^6 regions).
template <int D, bool KEPT>
__global__ __launch_bounds__(kTileThreads) void list_kernel(ListArgs A, Mirror M) {
  const Status* st = A.st;
  if (blockIdx.x == 0 && threadIdx.x < 64) mirror_status(M, st);
  if (st->done) return;
  const int64_t n = st->n_prev;
  const int in = st->buf;
  const int64_t leaf_base = st->leaf_base;
  const int64_t cap = A.cap;
  int64_t* __restrict__ idx = kept_list(A.C[1 - in], cap);
  RegionSrc R{};
  R.C = A.C[in];
  R.H = A.H[in];
  R.L = A.L[in];
  R.PAX = A.PAX[in];
  R.cap = cap;
  R.npar = st->n_par;
  R.split = st->split;
  const int64_t nt = (n + kTile - 1) / kTile;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  constexpr int kRows = kTile / kTileThreads;
  __shared__ int wc[kRows][kTileThreads / 64];
  for (int64_t tile = blockIdx.x; tile < nt; tile += gridDim.x) {
    // every row's flag and axis and the tile's offset in one memory round trip
    uint8_t fl[kRows], ax[kRows];
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
      const int64_t r0 = tile * kTile + k * kTileThreads + threadIdx.x;
      const int64_t r = r0 < n ? r0 : n - 1;
      fl[k] = A.FLAG[r];
      ax[k] = A.AXIS[r];
    }
    int64_t base = GM_INB(tile, (cap + kTile - 1) / kTile + 1) ? A.TOFF[tile] : 0;
    uint64_t masks[kRows];
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
      const int64_t r = tile * kTile + k * kTileThreads + threadIdx.x;
      masks[k] = __ballot(r < n && fl[k] == 0);
      if (lane == 0) wc[k][w] = __popcll(masks[k]);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
      const int64_t r = tile * kTile + k * kTileThreads + threadIdx.x;
      int64_t off = base;
#pragma unroll
      for (int i = 0; i < kTileThreads / 64; ++i) {
        if (i < w) off += wc[k][i];
        base += wc[k][i];
      }
      const int64_t before = off + __popcll(masks[k] & ((1ull << lane) - 1ull));
      if ((masks[k] >> lane) & 1ull) {
        if (KEPT) list_kept(idx, cap, before, r, ax[k]);
      } else if (D > 0 && r < n) {
        const int64_t slot = leaf_base + (r - before);
        if (GM_GUARD(slot, A.leaf_cap)) {
          constexpr int DD = D > 0 ? D : 1;
          double c[DD], h[DD];
          const int lvl = load_region<DD>(R, r, c, h);
#pragma unroll
          for (int j = 0; j < DD; ++j) {
            A.LC[j * A.leaf_cap + slot] = c[j];
            A.LH[j * A.leaf_cap + slot] = h[j];
          }
          A.LL[slot] = (uint16_t)lvl;
        }
      }
    }
    __syncthreads();
  }
}

// One iteration's bookkeeping for an active set of at most kStepRegions regions
// in a single workgroup: the reduction and stopping rule, the classification,
// the scan and the kept list of reduce_kernel, classify_kernel<false>,
// scan_kernel<false> and list_kernel, in that order and with the same results
// bit for bit, separated by workgroup barriers instead of kernel boundaries.
// The four launches cost 4 to 8 us each for such sets, almost all of it launch
// and memory latency: here the status block lives in LDS, a group of
// kTileThreads threads takes a tile (four at a time), and the counts, ranks and
// tile sums never leave the workgroup.  Not for memory-pressure pruning (its
// second classification pass).  In gradient mode (ca.FLAG used by list_kernel
// for the retired leaves) the flags and tile offsets are stored too.
__global__ __launch_bounds__(kStepThreads) void step_kernel(Status* st, const double* partials,
                                                            int np, ClassifyArgs ca, ListArgs la,
                                                            int64_t* TOFF, Mirror M) {
  constexpr int kGroups = kStepThreads / kTileThreads;  // tiles at a time
  constexpr int kRows = kTile / kTileThreads;
  constexpr int kTrips = kStepTiles / kGroups;
  constexpr int kWaves = kTileThreads / 64;  // wavefronts of a group
  __shared__ Status ss;
  __shared__ int cnt[kStepTiles][kRows][kWaves];
  __shared__ dd sq[kStepTiles][kWaves], se[kStepTiles][kWaves];
  __shared__ int64_t toff[kStepTiles];
  const int tid = threadIdx.x, lane = tid & 63;
  if (tid < kStatusWords) ((int64_t*)&ss)[tid] = ((const int64_t*)st)[tid];
  __syncthreads();
  if (ss.done) return;
  reduce_body(&ss, partials, np, ca.HIST);
  __syncthreads();
  const int64_t n = ss.n_active;
  const int g = tid / kTileThreads, gt = tid % kTileThreads, w = gt >> 6;
  const int nt = (int)((n + kTile - 1) / kTile);
  uint32_t keepbits = 0;  // bit trip * kRows + row
  if (!ss.done) {
    const double T = ss.T, aI = fabs(ss.I);
    const uint16_t* __restrict__ L = ca.L[ss.buf];
    const int split = ss.split;
    const int64_t npar = ss.n_par;
    for (int trip = 0; trip < kTrips; ++trip) {
      const int tile = trip * kGroups + g;
      if (tile >= nt) break;
      double errv[kRows], qv[kRows];
      int lvlv[kRows];
      uint8_t axv[kRows];
#pragma unroll
      for (int k = 0; k < kRows; ++k) {
        const int64_t r = (int64_t)tile * kTile + k * kTileThreads + gt;
        const int64_t rc = r < n ? r : n - 1;
        errv[k] = ca.ERR[rc];
        qv[k] = ca.Q[rc];
        axv[k] = ca.AXIS[rc];
        lvlv[k] = L[(split && rc >= npar) ? rc - npar : rc] + (split ? 1 : 0);
      }
      dd q = {0.0, 0.0}, e = {0.0, 0.0};
#pragma unroll
      for (int k = 0; k < kRows; ++k) {
        const int64_t r = (int64_t)tile * kTile + k * kTileThreads + gt;
        bool keep = false;
        if (r < n && GM_INB(r, ss.cap)) {
          const bool fin = retires(errv[k], T, aI, lvlv[k], axv[k]);
          keep = !fin;
          if (la.LC != nullptr) ca.FLAG[r] = fin ? 1 : 0;
          if (fin) {
            dd_add(q, qv[k]);
            dd_add(e, errv[k]);
          }
        }
        if (keep) keepbits |= 1u << (trip * kRows + k);
        const uint64_t mask = __ballot(keep);
        if (lane == 0) cnt[tile][k][w] = __popcll(mask);
      }
      q = wave_sum_dd(q);
      e = wave_sum_dd(e);
      if (lane == 0) {
        sq[tile][w] = q;
        se[tile][w] = e;
      }
    }
  }
  __syncthreads();
  if (!ss.done && tid < 64) {
    // a lane per tile: its count and retired sums, then the scan over the tiles
    int64_t sum = 0;
    dd q = {0.0, 0.0}, e = {0.0, 0.0};
    if (lane < nt) {
#pragma unroll
      for (int k = 0; k < kRows; ++k)
#pragma unroll
        for (int i = 0; i < kWaves; ++i) sum += cnt[lane][k][i];
      dd tq = sq[lane][0], te = se[lane][0];
#pragma unroll
      for (int i = 1; i < kWaves; ++i) {
        tq = dd_sum(tq, sq[lane][i]);
        te = dd_sum(te, se[lane][i]);
      }
      q = dd_sum(q, tq);
      e = dd_sum(e, te);
    }
    int64_t inc = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int64_t y = __shfl_up(inc, o, 64);
      if (lane >= o) inc += y;
    }
    if (lane < nt) {
      toff[lane] = inc - sum;
      if (la.LC != nullptr && GM_INB(lane, (ss.cap + kTile - 1) / kTile + 1)) TOFF[lane] = inc - sum;
    }
    q = wave_sum_dd(q);
    e = wave_sum_dd(e);
    const int64_t total = __shfl(inc, 63, 64);
    if (lane == 0) scan_commit<false>(&ss, total, q, e, ca.HIST);
  }
  __syncthreads();
  if (!ss.done) {
    int64_t* __restrict__ idx = kept_list(la.C[1 - ss.buf], la.cap);
    for (int trip = 0; trip < kTrips; ++trip) {
      const int tile = trip * kGroups + g;
      if (tile >= nt) break;
      int64_t base = toff[tile];
#pragma unroll
      for (int k = 0; k < kRows; ++k) {
        const int64_t r = (int64_t)tile * kTile + k * kTileThreads + gt;
        const bool keep = (keepbits >> (trip * kRows + k)) & 1u;
        const uint64_t mask = __ballot(keep);
        int64_t off = base;
#pragma unroll
        for (int i = 0; i < kWaves; ++i) {
          if (i < w) off += cnt[tile][k][i];
          base += cnt[tile][k][i];
        }
        if (keep)
          list_kept(idx, la.cap, off + __popcll(mask & ((1ull << lane) - 1ull)), r, ca.AXIS[r]);
      }
    }
  }
  if (tid < kStatusWords) ((int64_t*)st)[tid] = ((const int64_t*)&ss)[tid];
  if (tid < 64) mirror_status(M, &ss);
}

using ListFn = void (*)(ListArgs, Mirror);

// The gradient mode's leaf store wants the dimension (kept: the list as well).
static ListFn leaf_list_fn(int d, bool kept) {
  switch (d) {
#define GM_LEAF_CASE(D) \
  case D: return kept ? list_kernel<D, true> : list_kernel<D, false>;
    GM_LEAF_CASE(2) GM_LEAF_CASE(3) GM_LEAF_CASE(4) GM_LEAF_CASE(5) GM_LEAF_CASE(6)
    GM_LEAF_CASE(7) GM_LEAF_CASE(8) GM_LEAF_CASE(9) GM_LEAF_CASE(10) GM_LEAF_CASE(11)
    GM_LEAF_CASE(12) GM_LEAF_CASE(13) GM_LEAF_CASE(14) GM_LEAF_CASE(15) GM_LEAF_CASE(16)
#undef GM_LEAF_CASE
    default: return nullptr;
  }
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
namespace {

Options g_opt;
gm_stats g_stats;
std::string g_hip_err = "no HIP error";
std::string g_enomem_text;

// Device memory: either the caller's registered workspace or a cached
// library allocation that only grows.
void* g_ext_ptr = nullptr;
size_t g_ext_bytes = 0;
void* g_own_ptr = nullptr;
size_t g_own_bytes = 0;

// The last run, for gm_last_active.
struct LastRun {
  bool valid = false;
  int d = 0;
  int64_t n = 0, cap = 0;
  int64_t npar = 0;  // records behind a split set
  int split = 0;
  Layout lay;
  int buf = 0;
  char* base = nullptr;  // device buffers of that run
} g_last;

int hip_fail(hipError_t e) {
  g_hip_err = hipGetErrorString(e);
  (void)hipGetLastError();
  return GM_EHIP;
}

#define GM_HIP(call)                      \
  do {                                    \
    hipError_t _e = (call);               \
    if (_e != hipSuccess) return hip_fail(_e); \
  } while (0)

}  // namespace

Options& options() { return g_opt; }

std::mutex& api_mutex() {
  static std::mutex mu;
  return mu;
}

int record_hip_error(hipError_t e) { return hip_fail(e); }

GM_CHECK_UNIT(api)

#ifdef GM_CHECK
// Self-test of the check path: one index one past its bound, checked and not
// used (no memory is accessed).
__global__ void check_selftest_kernel(int64_t n) {
  if (threadIdx.x == 0 && blockIdx.x == 0) (void)GM_INB(n, n);
}

int check_bounds(int rc) {
  using PollFn = int (*)(CheckRec*);
#define GM_POLL_F(name)                                                               \
  {#name " f1", gm_check_poll_##name##_f1}, {#name " f2", gm_check_poll_##name##_f2}, \
  {#name " f3", gm_check_poll_##name##_f3}, {#name " f4", gm_check_poll_##name##_f4}, \
  {#name " f5", gm_check_poll_##name##_f5}, {#name " f6", gm_check_poll_##name##_f6}, \
  {#name " f7", gm_check_poll_##name##_f7}
#define GM_POLL_FACTOR(name)                                                              \
  {#name " f8", gm_check_poll_##name##_f8}, {#name " f9", gm_check_poll_##name##_f9},     \
  {#name " f10", gm_check_poll_##name##_f10}, {#name " f11", gm_check_poll_##name##_f11}, \
  {#name " f12", gm_check_poll_##name##_f12}
  static const struct {
    const char* name;
    PollFn fn;
  } units[] = {{"api", gm_check_poll_api}, {"batch", gm_check_poll_batch},
               {"grad", gm_check_poll_grad}, GM_POLL_F(rule), GM_POLL_F(rule9),
               GM_POLL_F(adjoint), GM_POLL_F(gk), GM_POLL_FACTOR(factor),
               GM_POLL_FACTOR(factor9), GM_POLL_FACTOR(factor_adjoint),
               {"rule f13", gm_check_poll_rule_f13}};
#undef GM_POLL_F
#undef GM_POLL_FACTOR
  std::string first;
  unsigned long long total = 0;
  for (const auto& u : units) {
    CheckRec r = {};
    if (u.fn(&r) != 0) return hip_fail(hipGetLastError());
    if (r.count != 0 && first.empty()) {
      char buf[256];
      std::snprintf(buf, sizeof buf, "bounds check failed in unit %s, line %d: index %lld, bound %lld",
                    u.name, r.line, r.index, r.bound);
      first = buf;
    }
    total += r.count;
  }
  if (total == 0) return rc;
  g_hip_err = first + " (" + std::to_string(total) + " violations)";
  return GM_EHIP;
}
#else
int check_bounds(int rc) { return rc; }
#endif

void stats_reset() { std::memset(&g_stats, 0, sizeof g_stats); }
gm_stats& stats_ref() { return g_stats; }

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

Layout make_layout(int d, int64_t cap) {
  Layout L;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off += align256(bytes);
    return o;
  };
  const int64_t ntiles = (cap + kTile - 1) / kTile + 1;
  for (int b = 0; b < 2; ++b) {
    L.C[b] = take(sizeof(double) * d * cap);
    L.H[b] = take(sizeof(double) * d * cap);
    L.L[b] = take(sizeof(uint16_t) * cap);
    L.PAX[b] = take(cap);
  }
  L.Q = take(sizeof(double) * cap);
  L.ERR = take(sizeof(double) * cap);
  L.AXIS = take(cap);
  L.FLAG = take(cap);
  L.TK = take(sizeof(int64_t) * ntiles);
  L.TOFF = take(sizeof(int64_t) * ntiles);
  L.TQ = take(sizeof(double) * 2 * ntiles);
  L.TE = take(sizeof(double) * 2 * ntiles);
  L.PART = take(sizeof(double) * 4 * kMaxRuleGrid);
  L.ST = take(sizeof(Status));
  L.HIST = take(sizeof(int64_t) * kPruneBins);
  L.total = off;
  return L;
}

int acquire_workspace(size_t bytes, char** base) {
  g_last.valid = false;  // the last run's buffers are written over, or go away
  if (g_ext_ptr) {
    if (bytes > g_ext_bytes) return GM_ENOMEM;
    *base = (char*)g_ext_ptr;
    return GM_OK;
  }
  if (bytes > g_own_bytes) {
    if (g_own_ptr) {
      GM_HIP(hipDeviceSynchronize());
      GM_HIP(hipFree(g_own_ptr));
      g_own_ptr = nullptr;
      g_own_bytes = 0;
    }
    hipError_t e = hipMalloc(&g_own_ptr, bytes);
    if (e != hipSuccess) {
      g_hip_err = hipGetErrorString(e);
      (void)hipGetLastError();
      g_own_ptr = nullptr;
      return GM_ENOMEM;
    }
    g_own_bytes = bytes;
  }
  *base = (char*)g_own_ptr;
  return GM_OK;
}

void fill_consts(int d, RuleConsts& K) {
  const int64_t D = d;
  K.lam2 = std::sqrt(9.0 / 70.0);
  K.lam3 = std::sqrt(9.0 / 10.0);
  K.lam4 = std::sqrt(9.0 / 10.0);
  K.lam5 = std::sqrt(9.0 / 19.0);
  K.w[0] = (double)(400 * D * D - 9120 * D + 12824) / 19683.0;
  K.w[1] = 980.0 / 6561.0;
  K.w[2] = (double)(1820 - 400 * D) / 19683.0;
  K.w[3] = 200.0 / 19683.0;
  K.w[4] = std::ldexp(6859.0 / 19683.0, -d);
  K.e[0] = (double)(-19 * (50 * D * D - 870 * D + 361)) / 19683.0;
  K.e[1] = -4655.0 / 13122.0;
  K.e[2] = (double)(95 * (20 * D - 37)) / 39366.0;
  K.e[3] = -475.0 / 19683.0;
  K.e[4] = K.w[4];
  K.r7 = 1.0 / 7.0;
  K.axis_band = 1e-10;
  // degree-9 rule: the unique solution of its even-moment equations (degree
  // <= 8), each weight one correctly rounded division of exact integers
  K.lam6 = std::sqrt(759.0 / 1190.0);
  K.w9[0] = (double)(-160 * (6325 * D * D * D - 345345 * D * D + 1801355 * D - 1902813)) /
            403363719.0;
  K.w9[1] = (double)(-490 * (2020 * D - 8711)) / 17891847.0;
  K.w9[2] = (double)(5 * (10400 * D * D - 236080 * D + 404019)) / 13817466.0;
  K.w9[3] = (double)(-1000 * (2 * D - 9)) / 531441.0;
  K.w9[4] = std::ldexp(130321.0 / 531441.0, -d);
  K.w9[5] = 20462645.0 / 484331562.0;
  K.w9[6] = 4900.0 / 177147.0;
  K.w9[7] = 1000.0 / 531441.0;
  // minus the degree-7 weights (zero on classes 6..8), exact, rounded once
  K.e9[0] = (double)(-8 * (126500 * D * D * D - 5882250 * D * D + 12665080 * D - 5205981)) /
            403363719.0;
  K.e9[1] = (double)(-490 * (2020 * D - 3257)) / 17891847.0;
  K.e9[2] = (double)(5 * (10400 * D * D - 179920 * D + 148491)) / 13817466.0;
  K.e9[3] = (double)(-400 * (5 * D - 9)) / 531441.0;
  K.e9[4] = std::ldexp(-54872.0 / 531441.0, -d);
  K.e9[5] = K.w9[5];
  K.e9[6] = K.w9[6];
  K.e9[7] = K.w9[7];
  // degree-3 rule on the centre and the +-l3 e_i nodes (exact on 1 and x^2)
  K.q3[0] = (double)(27 - 10 * D) / 27.0;
  K.q3[1] = 5.0 / 27.0;
  K.err_model = g_opt.err_model;
}

void fill_params(int fam, int d, const double* params, DevParams& P) {
  std::memset(&P, 0, sizeof P);
  P.d = d;
  P.fam = fam;
  for (int j = 0; j < d; ++j) {
    P.a[j] = params[j];
    P.u[j] = params[d + j];
    P.inv_a2[j] = 1.0 / (P.a[j] * P.a[j]);
  }
  P.c0 = 6.283185307179586476925286766559 * P.u[0];
}

int validate(int fam, const double* params, int d, const double* lo, const double* hi,
             double rel_tol, double abs_tol) {
  if (fam < 1 || fam > 7) return GM_EINVAL;
  if (d < kMinDim || d > kMaxDim) return GM_EINVAL;
  if (!params || !lo || !hi) return GM_EINVAL;
  if (!(rel_tol >= 0.0) || !(abs_tol >= 0.0) || !std::isfinite(rel_tol) || !std::isfinite(abs_tol))
    return GM_EINVAL;
  if (rel_tol == 0.0 && abs_tol == 0.0) return GM_EINVAL;
  if (g_opt.rule == 1 && d > kGkMaxDim) return GM_EINVAL;
  for (int j = 0; j < d; ++j)
    if (!std::isfinite(lo[j]) || !std::isfinite(hi[j]) || !(lo[j] < hi[j])) return GM_EINVAL;
  for (int j = 0; j < 2 * d; ++j)
    if (!std::isfinite(params[j])) return GM_EINVAL;
  return GM_OK;
}

// The kernel family of integrand fam on [lo, hi]: the factored one (gm_nodes.hpp)
// where the family has it and the parameters allow.  The product families need
// every partial product to stay in the range of a double: the axes' largest
// |log factor| add up to at most 500 (e^708 is the end).  Beyond it a partial
// product could overflow or vanish although the integrand does not (a C0
// integrand with large negative a_j), and node values below e^-500 are no more
// accurate than the rounding of their exponent, which only the definition's
// order of summation reproduces: those run in chain form.  The seeded families
// stay below 100 and the paper's f2 below 16 per axis; its f4 (a = 25, u = 1/2)
// passes the line from d = 4 on.  The rotations of the oscillatory family have
// no such limit.
// The corner peak's quotient form multiplies four powers (1 + s)^(d+1): 1 + s, by
// its exact range over the box (it is linear in x), stays within 2^+-(250 / (d + 1)),
// so products and quotients stay within 2^+-1000, and its terms are not so much
// larger than it that their rounding could reach its sign.
int kernel_family(int fam, int d, const double* params, const double* lo, const double* hi) {
  if (d < kFactorMinDim) return fam;
  if (fam == kOsc) return kOscF;
  if (fam == kCornerPeak) {
    double smin = 1.0, smax = 1.0, mag = 1.0;
    for (int j = 0; j < d; ++j) {
      const double p = params[j] * lo[j], q = params[j] * hi[j];
      smin += std::min(p, q);
      smax += std::max(p, q);
      mag += std::max(std::fabs(p), std::fabs(q));
    }
    const double lim = std::exp2(250.0 / (d + 1));
    return smin * lim >= 1.0 && smax <= lim && mag <= 0x1p40 * smin ? kCornerPeakQ : fam;
  }
  if (fam != kProductPeak && fam != kGaussian && fam != kC0 && fam != kDiscontinuous) return fam;
  double span = 0.0;
  for (int j = 0; j < d; ++j) {
    const double a = params[j], u = params[d + j];
    const double far = std::max(std::fabs(lo[j] - u), std::fabs(hi[j] - u));
    if (fam == kProductPeak) {  // the factor lies between 1 / (a^-2 + far^2) and a^2
      const double inv_a2 = 1.0 / (a * a);
      span += std::max(std::fabs(std::log(inv_a2)), std::fabs(std::log(inv_a2 + far * far)));
    } else if (fam == kGaussian) {
      span += (a * far) * (a * far);
    } else if (fam == kC0) {
      span += std::fabs(a) * far;
    } else {
      span += std::fabs(a) * std::max(std::fabs(lo[j]), std::fabs(hi[j]));
    }
  }
  if (!(span <= 500.0)) return fam;  // (NaN: the chain form)
  return fam == kProductPeak ? kProductPeakF
         : fam == kGaussian  ? kGaussianF
         : fam == kC0        ? kC0F
                             : kDiscontinuousF;
}

int init_cells_log2(int d) { return g_opt.init_log2 / d; }

RuleKernelFn rule_kernel(int d, int fam, int log2l, bool batch) {
  switch (fam) {
    case 1: return rule_kernel_f1(d, log2l, batch);
    case 2: return rule_kernel_f2(d, log2l, batch);
    case 3: return rule_kernel_f3(d, log2l, batch);
    case 4: return rule_kernel_f4(d, log2l, batch);
    case 5: return rule_kernel_f5(d, log2l, batch);
    case 6: return rule_kernel_f6(d, log2l, batch);
    case 7: return rule_kernel_f7(d, log2l, batch);
    case kOscF: return factor_kernel_f8(d, log2l, batch);
    case kProductPeakF: return factor_kernel_f9(d, log2l, batch);
    case kGaussianF: return factor_kernel_f10(d, log2l, batch);
    case kC0F: return factor_kernel_f11(d, log2l, batch);
    case kDiscontinuousF: return factor_kernel_f12(d, log2l, batch);
    case kCornerPeakQ: return rule_kernel_f13(d, log2l, batch);
    default: return nullptr;
  }
}

RuleKernelFn gk_kernel(int d, int fam, bool batch) {
  switch (fam) {
    case 1: return gk_kernel_f1(d, batch);
    case 2: return gk_kernel_f2(d, batch);
    case 3: return gk_kernel_f3(d, batch);
    case 4: return gk_kernel_f4(d, batch);
    case 5: return gk_kernel_f5(d, batch);
    case 6: return gk_kernel_f6(d, batch);
    case 7: return gk_kernel_f7(d, batch);
    default: return nullptr;
  }
}

RuleKernelFn r9_kernel(int d, int fam, bool batch, int log2l) {
  const bool wide = log2l != rule9_log2l(d);
  switch (fam) {
    case 1: return rule9_kernel_f1(d, batch, wide);
    case 2: return rule9_kernel_f2(d, batch, wide);
    case 3:
    case kCornerPeakQ: return rule9_kernel_f3(d, batch, wide);
    case 4: return rule9_kernel_f4(d, batch, wide);
    case 5: return rule9_kernel_f5(d, batch, wide);
    case 6: return rule9_kernel_f6(d, batch, wide);
    case 7: return rule9_kernel_f7(d, batch, wide);
    case kOscF: return batch ? nullptr : factor9_kernel_f8(d, log2l);
    case kProductPeakF: return batch ? nullptr : factor9_kernel_f9(d, log2l);
    case kGaussianF: return batch ? nullptr : factor9_kernel_f10(d, log2l);
    case kC0F: return batch ? nullptr : factor9_kernel_f11(d, log2l);
    case kDiscontinuousF: return batch ? nullptr : factor9_kernel_f12(d, log2l);
    default: return nullptr;
  }
}

// Mapping codes: the Gauss-Kronrod kernel (gk_threads(d) per region), and the
// degree-9 kernel with 2^(code - kMapR9) lanes per region (kMapR9Tpr: one lane).
constexpr int kMapGk = 100;
constexpr int kMapR9 = 200;
constexpr int kMapR9Tpr = kMapR9 - 1;

int lanes_of_mapping(int map, int d) {
  return map == kMapGk ? gk_threads(d) : map >= kMapR9 ? (1 << (map - kMapR9)) : map < 0 || map == kMapR9Tpr ? 1 : (1 << map);
}

int64_t nodes_per_region(int d) {
  if (g_opt.rule == 1) {
    int64_t n = 1;
    for (int j = 0; j < d; ++j) n *= 15;
    return n;
  }
  if (g_opt.rule == 2) {
    const int64_t D = d;
    return 1 + 6 * D + 6 * D * (D - 1) + 4 * D * (D - 1) * (D - 2) / 3 + ((int64_t)1 << d);
  }
  return gm_num_nodes(d);
}

hipError_t launch_rule(int d, int fam, int log2l, const RuleArgs& a, int grid, hipStream_t s) {
  RuleKernelFn fn = log2l == kMapGk    ? gk_kernel(d, fam, false)
                    : log2l >= kMapR9Tpr ? r9_kernel(d, fam, false, log2l - kMapR9)
                                      : rule_kernel(d, fam, log2l, false);
  if (!fn) return hipErrorInvalidValue;
  hipLaunchKernelGGL(fn, dim3(grid), dim3(kRuleBlockSize), 0, s, a);
  return hipGetLastError();
}

bool mapping_allowed(int d, int log2l) {
  if (log2l < 0) return d <= kTprMaxDim;
  if (log2l == 2) return d >= 6;
  if (log2l == 4) return d >= 8;
  if (log2l == 6) return d >= 10;
  return false;
}

// log2 of the lanes per region the option asks for (-1: one lane).
static int forced_log2l() {
  int l = -1;
  if (g_opt.lanes_per_region > 1) {
    l = 0;
    while ((1 << l) < g_opt.lanes_per_region) ++l;
  }
  return l;
}

// Lanes a launch should occupy before it takes fewer lanes per region: the
// whole GPU at two wavefronts per SIMD is 256 CUs x 4 SIMDs x 2 x 64 = 131072,
// but a lane's whole region costs less than several lanes' shares with their
// common work, so the one-lane kernel wins from fewer on.  Corner peak (quotient
// form) at d = 8, us for 1 / 4 / 16 lanes: n = 8192: 19 / 18 / 19, 32768: 20 / 27 /
// 45, 65536: 23 / 40 / 78; d = 10: n = 32768: 47 / 41 / 60, 65536: 56 / 70 / 106.
// Factored, 1 / 4 / 16 / 64 lanes, product peak, d = 11: n = 4096: 18 / 18 / 13 /
// 19, 16384: 17 / 19 / 21 / 51, 65536: 22 / 42 / 61 / 180; d = 13: n = 1: 39 / 24 /
// 13 / 12, 8192: 35 / 26 / 18 / 32, 32768: 39 / 37 / 46 / 107, 65536: 42 / 67 / 81 /
// 208; d = 16, where the one-lane kernel spills 100 registers: n = 64: 198 / 71 / 27
// / 17, 65536: 206 / 275 / 253 / 428, 262144: 733 / 1057 / 997 / 1430 (oscillatory,
// Gaussian and C0 cross at the same sizes; at d = 11 one lane is ahead from 32768 on
// already, 18 / 24).  Up to d = 10 one lane is the fastest at every n (d = 8
// Gaussian, n = 256: 11 / 15 / 19 us, 49166: 18 / 30 / 65).
constexpr int64_t kTargetLanes = 131072;
static int64_t target_lanes(int d, bool factored) {
  if (factored) return d <= kTprMaxDim ? 0 : 65536;
  return d < 10 ? 32768 : d == 10 ? 65536 : kTargetLanes;
}
// Active sets from which the factored degree-9 rule runs one lane per region: at
// every size up to d = 8 (Gaussian, one lane against the several of the chain form,
// n = 256: 16 / 17 us, 3684: 20 / 30, 22090: 18 / 41); above, the 64-lane kernel is
// ahead in small sets (one / 64 lanes, d = 9 C0, n = 1024: 26 / 13, 4096: 25 / 21,
// 8192: 25 / 34; d = 10, n = 1024: 31 / 14, 4096: 32 / 23, 8192: 31 / 35; the
// rotations cross at the same sizes).
constexpr int64_t r9_tpr_regions(int d) {
  return d < kFactor9WideMinDim ? 0 : d == 9 ? 5120 : 6144;
}

int choose_mapping(int d, int kfam, int64_t n, bool list) {
  const bool factored = is_factored(kfam);
  if (g_opt.rule == 1) return kMapGk;
  if (g_opt.rule == 2) {
    if (factored && d <= kTprMaxDim && n >= r9_tpr_regions(d)) return kMapR9Tpr;
    // the wide mapping while the default one would leave the GPU mostly idle (the
    // factored several-lane kernels have no other)
    const bool wide = factored || (n << rule9_log2l(d)) < kTargetLanes;
    return kMapR9 + (wide ? rule9_log2l_wide(d) : rule9_log2l(d));
  }
  const bool tpr = d <= kTprMaxDim || factored;
  if (g_opt.lanes_per_region > 0) {
    const int l = forced_log2l();
    if (l < 0 ? tpr : mapping_allowed(d, l)) return l;
  }
  // (a list's mapping, and with it the order in which its class sums are
  // combined, stays that of the full GPU)
  const int64_t target = list ? kTargetLanes : target_lanes(d, factored);
  const int cands[4] = {-1, 2, 4, 6};
  int best = -2;
  for (int k = 0; k < 4; ++k) {
    const int l = cands[k];
    if (!(l < 0 ? tpr : mapping_allowed(d, l))) continue;
    best = l;
    const int64_t lanes = (l < 0) ? n : (n << l);
    if (lanes >= target) break;
  }
  return best;
}

// The factored one-lane kernels read a region's record while they evaluate the one
// before (load_record), so their workgroups stay and stride: two fit a CU, 512 in
// all, and twice as many even out the end.  Before, one workgroup per 256 regions
// waited for status, list and record in turn: d = 8 Gaussian at 1e-7, ms for 16384
// workgroups / without the read ahead / 512 / 1024 / 2048: 3.74 / 3.82 / 3.45 /
// 3.47 / 3.44, oscillatory 2.19 / 2.21 / 2.12 / 2.07 / 2.08; 3.24e6 regions in one
// launch 259 -> 219 us.  The degree-9 kernel has no registers for a second record
// and gains by the start alone (C0 1.22 / - / 1.18 / 1.20 / 1.21).  The chain
// kernels spend far longer on a region and only lose by the uneven end (corner
// peak 6.80 / - / 6.95 / 6.83 / 6.77), as do more than ten dimensions.
static int max_rule_grid(int log2l, int d, int kfam) {
  if (!is_factored(kfam) || d > kTprMaxDim) return kMaxRuleGrid;
  return log2l == kMapR9Tpr ? 512 : log2l < 0 ? 1024 : kMaxRuleGrid;
}

int rule_grid(int log2l, int64_t n, int d, int kfam) {
  const int64_t per_block = log2l == kMapGk    ? kRuleBlockSize / gk_threads(d)
                            : log2l >= kMapR9 ? (kRuleBlockSize >> (log2l - kMapR9))
                            : (log2l < 0 || log2l == kMapR9Tpr) ? kRuleBlockSize
                                            : (kRuleBlockSize >> log2l);
  const int64_t g = (n + per_block - 1) / per_block;
  return (int)std::max<int64_t>(1, std::min<int64_t>(g, max_rule_grid(log2l, d, kfam)));
}

static int tile_grid_for(int64_t n) {
  int64_t g = (n + kTile - 1) / kTile;
  return (int)std::max<int64_t>(1, std::min<int64_t>(g, kMaxTileGrid));
}

// Leaf store of the gradient mode (SoA, grows on demand).
struct LeafStore {
  double* C = nullptr;
  double* H = nullptr;
  uint16_t* L = nullptr;
  int64_t cap = 0;
  int d = 0;
  void release() {
    if (C) (void)hipFree(C);
    if (H) (void)hipFree(H);
    if (L) (void)hipFree(L);
    C = H = nullptr;
    L = nullptr;
    cap = 0;
  }
};

static LeafStore g_leaves;

LeafView leaf_view() { return LeafView{g_leaves.C, g_leaves.H, g_leaves.L, g_leaves.cap}; }

static int leaf_reserve(int d, int64_t need, int64_t have, hipStream_t s) {
  if (need <= g_leaves.cap && g_leaves.d == d) return GM_OK;
  // A store of another dimension holds nothing to keep: free it first and
  // size the new one from this run's need alone (doubling its capacity would
  // compound over calls that alternate dimensions).
  if (g_leaves.d != d) {
    GM_HIP(hipStreamSynchronize(s));
    g_leaves.release();
    g_leaves.d = d;
    have = 0;
  }
  int64_t nc = std::max<int64_t>(need, std::max<int64_t>(1 << 16, 2 * g_leaves.cap));
  double *C = nullptr, *H = nullptr;
  uint16_t* L = nullptr;
  if (hipMalloc(&C, sizeof(double) * d * nc) != hipSuccess ||
      hipMalloc(&H, sizeof(double) * d * nc) != hipSuccess ||
      hipMalloc(&L, sizeof(uint16_t) * nc) != hipSuccess) {
    (void)hipGetLastError();
    if (C) (void)hipFree(C);
    if (H) (void)hipFree(H);
    if (L) (void)hipFree(L);
    return GM_ENOMEM;
  }
  if (have > 0) {
    for (int j = 0; j < d; ++j) {
      GM_HIP(hipMemcpyAsync(C + j * nc, g_leaves.C + j * g_leaves.cap, sizeof(double) * have,
                            hipMemcpyDeviceToDevice, s));
      GM_HIP(hipMemcpyAsync(H + j * nc, g_leaves.H + j * g_leaves.cap, sizeof(double) * have,
                            hipMemcpyDeviceToDevice, s));
    }
    GM_HIP(hipMemcpyAsync(L, g_leaves.L, sizeof(uint16_t) * have, hipMemcpyDeviceToDevice, s));
    GM_HIP(hipStreamSynchronize(s));
  }
  g_leaves.release();
  g_leaves.C = C;
  g_leaves.H = H;
  g_leaves.L = L;
  g_leaves.cap = nc;
  g_leaves.d = d;
  return GM_OK;
}

// Pinned host slots of the status block (Mirror), one per iteration in flight.
// create = false returns them only if an earlier call made them.
constexpr int kMaxAhead = 8;
constexpr int kSlots = 2 * kMaxAhead;
static StatusSlot* status_slots(bool create) {
  static StatusSlot* p = nullptr;
  if (!p && create) {
    if (hipHostMalloc((void**)&p, sizeof(StatusSlot) * kSlots,
                      hipHostMallocPortable | hipHostMallocCoherent) != hipSuccess) {
      (void)hipGetLastError();
      p = nullptr;
    } else {
      std::memset((void*)p, 0, sizeof(StatusSlot) * kSlots);
    }
  }
  return p;
}
static int64_t g_status_seq = 0;  // numbers the iterations of every run

// How the process wants HIP to wait (hipDeviceSchedule...): the slots are for one
// that spins, as HIP does by default.
static unsigned wait_mode() {
  unsigned flags = 0;
  if (hipGetDeviceFlags(&flags) != hipSuccess) (void)hipGetLastError();
  return flags & hipDeviceScheduleMask;
}

// Wait until the GPU has filled the slot for iteration number seq.  Ends with
// an error if the stream drains or fails without it.
static int await_slot(const StatusSlot* slot, int64_t seq, bool yield, hipStream_t s, Status* out) {
  for (int64_t spin = 1;; ++spin) {
    if (__atomic_load_n(&slot->seq, __ATOMIC_ACQUIRE) == seq) break;
    if (yield) std::this_thread::yield();
    if ((spin & 0x3fff) == 0) {
      const hipError_t e = hipStreamQuery(s);
      if (e == hipSuccess && __atomic_load_n(&slot->seq, __ATOMIC_ACQUIRE) != seq) {
        g_hip_err = "internal error: an iteration ended without a status";
        return GM_EHIP;
      }
      if (e != hipSuccess && e != hipErrorNotReady) return hip_fail(e);
      (void)hipGetLastError();
    }
  }
  std::memcpy(out, slot->words, sizeof *out);
  return GM_OK;
}

// Fixed device scratch of gm_integrate_noalloc (callers that cannot allocate):
// a file-scope array each device holds until the process ends.  In host code
// `scratch` names a host-side stand-in, never the device address: the address
// is looked up once per device with hipGetSymbolAddress (that device current)
// and only that pointer is handed to kernels and copies.
constexpr size_t kNoallocScratchBytes = size_t(64) << 20;
static __device__ __align__(256) unsigned char scratch[kNoallocScratchBytes];
constexpr int kMaxDevices = 64;
static char* g_scratch_dev[kMaxDevices] = {};

static int noalloc_scratch(char** out) {
  int dev = 0;
  GM_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) {
    g_hip_err = "device index beyond the no-allocation scratch table";
    return GM_EHIP;
  }
  if (!g_scratch_dev[dev]) {
    void* p = nullptr;
    GM_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p || ((uintptr_t)p & 255u) != 0) {
      g_hip_err = "no-allocation scratch: unexpected device address";
      return GM_EHIP;
    }
    g_scratch_dev[dev] = (char*)p;
  }
  *out = g_scratch_dev[dev];
  return GM_OK;
}

// A run's timing events.
struct RunEvents {
  hipEvent_t ev[kMaxAhead][5] = {};
  ~RunEvents() {
    for (auto& row : ev)
      for (auto& e : row)
        if (e) (void)hipEventDestroy(e);
  }
};

// One adaptive run on the device (gm_integrate and the forward pass of
// gm_integrate_grad).  On return the status block holds the final state.
int run_adaptive(int fam, const double* params, int d, const double* lo, const double* hi,
                 double rel_tol, double abs_tol, int64_t max_regions, hipStream_t s,
                 bool keep_leaves, RunResult* out, char* fixed_base) {
  const auto t_start = std::chrono::steady_clock::now();
  std::memset(&g_stats, 0, sizeof g_stats);
  const int m = init_cells_log2(d);
  const int64_t n0 = (int64_t)1 << (m * d);
  if (max_regions < n0) return GM_EINVAL;
  const int64_t cap = max_regions;
  const Layout lay = make_layout(d, cap);
  // (the Gauss-Kronrod kernel has no factored form, nor have several lanes per
  // region, which the option can ask for, up to d = 10)
  const bool lanes = g_opt.rule == 0 && d <= kTprMaxDim && g_opt.lanes_per_region > 1 &&
                     mapping_allowed(d, forced_log2l());
  int kfam = g_opt.rule == 1 ? fam : kernel_family(fam, d, params, lo, hi);
  if (lanes && is_factored(kfam)) kfam = fam;
  g_last.valid = false;  // (before the workspace may move)
  char* base = fixed_base;
  int rc = GM_OK;
  if (!base) {
    rc = acquire_workspace(lay.total, &base);
    if (rc != GM_OK) return rc;
  }

  RuleArgs ra;
  std::memset(&ra, 0, sizeof ra);
  fill_params(fam, d, params, ra.P);
  fill_consts(d, ra.K);
  for (int b = 0; b < 2; ++b) {
    ra.C[b] = (double*)(base + lay.C[b]);
    ra.H[b] = (double*)(base + lay.H[b]);
    ra.L[b] = (uint16_t*)(base + lay.L[b]);
    ra.PAX[b] = (uint8_t*)(base + lay.PAX[b]);
  }
  ra.cap = cap;
  ra.Q = (double*)(base + lay.Q);
  ra.ERR = (double*)(base + lay.ERR);
  ra.AXIS = (uint8_t*)(base + lay.AXIS);
  ra.partials = (double*)(base + lay.PART);
  Status* st = (Status*)(base + lay.ST);
  ra.st = st;
  double vol = 1.0;
  for (int j = 0; j < d; ++j) vol = vol * (hi[j] - lo[j]);
  ra.vol_omega = vol;
  ra.n_fixed = -1;

  InitArgs ia;
  std::memset(&ia, 0, sizeof ia);
  ia.C = ra.C[0];
  ia.H = ra.H[0];
  ia.L = ra.L[0];
  ia.cap = cap;
  ia.n0 = n0;
  ia.d = d;
  ia.m = m;
  for (int j = 0; j < d; ++j) {
    ia.lo[j] = lo[j];
    ia.half[j] = (hi[j] - lo[j]) * 0.5;
  }

  ClassifyArgs ca;
  ca.st = st;
  ca.L[0] = ra.L[0];
  ca.L[1] = ra.L[1];
  ca.Q = ra.Q;
  ca.ERR = ra.ERR;
  ca.AXIS = ra.AXIS;
  ca.FLAG = (uint8_t*)(base + lay.FLAG);
  ca.TK = (int64_t*)(base + lay.TK);
  ca.TQ = (double*)(base + lay.TQ);
  ca.TE = (double*)(base + lay.TE);
  ca.HIST = (int64_t*)(base + lay.HIST);

  int64_t* const toff = (int64_t*)(base + lay.TOFF);
  ListArgs la;
  std::memset(&la, 0, sizeof la);
  la.st = st;
  for (int b = 0; b < 2; ++b) {
    la.C[b] = ra.C[b];
    la.H[b] = ra.H[b];
    la.L[b] = ra.L[b];
    la.PAX[b] = ra.PAX[b];
  }
  la.cap = cap;
  la.AXIS = ra.AXIS;
  la.FLAG = ca.FLAG;
  la.TOFF = toff;

  Status hst;
  std::memset(&hst, 0, sizeof hst);
  hst.n_active = n0;
  hst.cap = cap;
  hst.max_iters = g_opt.max_iters;
  hst.rel_tol = rel_tol;
  hst.abs_tol = abs_tol;
  hst.prune_on = g_opt.prune;
  ia.st = st;
  ia.status = hst;
  RunEvents events;
  DrainOnError drain{s};
  {
    int g = (int)std::min<int64_t>((n0 + 255) / 256, 4096);
    hipLaunchKernelGGL(init_kernel, dim3(g), dim3(256), 0, s, ia);
    GM_HIP(hipGetLastError());
  }

  // Kernels take the active count from the device and return at once after a
  // final status, so iterations can be launched before the host knows that they
  // are needed; grids are sized for the largest count one can have (n doubles at
  // most per iteration).  The host reads each iteration's status from its slot
  // and keeps `ahead` iterations in flight: two, so that the GPU never waits for
  // the host (an iteration takes 15 us or more, a read and its launches 5), and
  // at most one is launched in vain.  Gradient mode keeps one (the leaf store
  // grows on the host's side).  Without slots (none made before a call on the
  // no-allocation path) the host launches a few iterations and copies the status
  // behind them: 6 below 2^16 active regions, 3 below 2^20, 2 above; and so it does
  // in a process that asked HIP to block while it waits.
  //
  // How many are in flight decides neither the kernels nor a bit of the result:
  // with more than one, iteration k takes the rule-kernel mapping of twice
  // iteration k - 1's count (what is known of it with two in flight), and is not
  // launched before that count is known unless every count it could have gives
  // the same mapping.  (The grid only bounds the workgroups: a region's
  // workgroup, and with it the order of the sums, is the same in every grid.)
  // (events are created per run: not on the no-allocation path)
  const bool timing = g_opt.timing != 0 && !fixed_base;  // rule kernel only
  const bool phases = timing && g_opt.timing >= 2;       // every phase
  if (timing)
    for (auto& row : events.ev)
      for (auto& e : row) GM_HIP(hipEventCreate(&e));
  StatusSlot* const slots = status_slots(fixed_base == nullptr);
  const unsigned wait = wait_mode();
  const bool mirrored = slots && wait != hipDeviceScheduleBlockingSync;

  const ListFn list_fn = keep_leaves ? leaf_list_fn(d, true) : list_kernel<0, true>;
  int64_t n = n0;             // active regions of iteration `seen`
  int64_t n_before = 0;       // ... and of the one before it
  int64_t leaves_have = 0;
  int64_t seen = 0, launched = 0;  // iterations whose status is known / launched
  const int64_t seq0 = g_status_seq;
  for (;;) {
    int ahead = 1;
    if (!keep_leaves) {
      if (g_opt.graph_iters > 0) ahead = std::min(g_opt.graph_iters, kMaxAhead);
      else if (mirrored) ahead = 2;
      else ahead = n < (1 << 16) ? 6 : n < (1 << 20) ? 3 : 2;
    } else {
      // Room for every region of this iteration to retire.
      rc = leaf_reserve(d, leaves_have + n, leaves_have, s);
      if (rc != GM_OK) return rc;
      la.LC = g_leaves.C;
      la.LH = g_leaves.H;
      la.LL = g_leaves.L;
      la.leaf_cap = g_leaves.cap;
    }
    int64_t nb = n;
    for (int64_t k = seen; k < launched; ++k) nb = std::min<int64_t>(cap, 2 * nb);
    for (; launched < seen + ahead; ++launched) {
      int64_t nm = nb;  // the count the mapping goes by
      if (ahead > 1 && launched > 0) {
        const int64_t k = launched - seen;
        if (k < 2) nm = std::min<int64_t>(cap, 2 * (k == 0 ? n_before : n));
        else if (choose_mapping(d, kfam, nb, false) != choose_mapping(d, kfam, 2, false)) break;
      }
      const int map = choose_mapping(d, kfam, nm, false);
      const int rg = rule_grid(map, nb, d, kfam);
      const int tg = tile_grid_for(nb);
      g_stats.lanes_per_region = lanes_of_mapping(map, d);
      hipEvent_t* const e = events.ev[launched % kMaxAhead];
      const int64_t seq = ++g_status_seq;
      const Mirror mir{mirrored ? slots + seq % kSlots : nullptr, seq};
      if (timing) GM_HIP(hipEventRecord(e[0], s));
      GM_HIP(launch_rule(d, kfam, map, ra, rg, s));
      if (timing) GM_HIP(hipEventRecord(e[1], s));
      if (!g_opt.prune && !phases && nb <= kStepRegions) {
        hipLaunchKernelGGL(step_kernel, dim3(1), dim3(kStepThreads), 0, s, st, ra.partials, rg, ca,
                           la, toff, mir);
        GM_HIP(hipGetLastError());
        if (keep_leaves) {
          hipLaunchKernelGGL(leaf_list_fn(d, false), dim3(tg), dim3(kTileThreads), 0, s, la,
                             Mirror{});
          GM_HIP(hipGetLastError());
        }
        nb = std::min<int64_t>(cap, 2 * nb);
        continue;
      }
      hipLaunchKernelGGL(reduce_kernel, dim3(1), dim3(1024), 0, s, st, ra.partials, rg, ca.HIST);
      GM_HIP(hipGetLastError());
      if (phases) GM_HIP(hipEventRecord(e[2], s));
      hipLaunchKernelGGL(classify_kernel<false>, dim3(tg), dim3(kTileThreads), 0, s, ca);
      GM_HIP(hipGetLastError());
      if (phases) GM_HIP(hipEventRecord(e[3], s));
      hipLaunchKernelGGL(scan_kernel<false>, dim3(1), dim3(1024), 0, s, st, ca.TK, toff, ca.TQ,
                         ca.TE, ca.HIST);
      GM_HIP(hipGetLastError());
      if (g_opt.prune) {
        hipLaunchKernelGGL(classify_kernel<true>, dim3(tg), dim3(kTileThreads), 0, s, ca);
        GM_HIP(hipGetLastError());
        hipLaunchKernelGGL(scan_kernel<true>, dim3(1), dim3(1024), 0, s, st, ca.TK, toff, ca.TQ,
                           ca.TE, ca.HIST);
        GM_HIP(hipGetLastError());
      }
      hipLaunchKernelGGL(list_fn, dim3(tg), dim3(kTileThreads), 0, s, la, mir);
      GM_HIP(hipGetLastError());
      if (phases) GM_HIP(hipEventRecord(e[4], s));
      nb = std::min<int64_t>(cap, 2 * nb);
    }
    const int64_t before = seen;
    if (mirrored) {
      const int64_t seq = seq0 + seen + 1;
      // A gradient's first iteration, with which the tiny ones end: with one in
      // flight nothing runs meanwhile, and the stream's wait, which the call owes at
      // its end anyway, costs less here than after a loop on the slot (gradients of
      // one iteration: 83 -> 65 us, of several the same; a copy of the status in its
      // place slows the launches after it, 12 iterations 433 -> 457).
      if (keep_leaves && seen == 0) GM_HIP(hipStreamSynchronize(s));
      rc = await_slot(slots + seq % kSlots, seq, wait == hipDeviceScheduleYield, s, &hst);
      if (rc != GM_OK) return rc;
      seen += 1;
    } else {
      Status* const to = slots ? (Status*)slots[0].words : &hst;
      GM_HIP(hipMemcpyAsync(to, st, sizeof hst, hipMemcpyDeviceToHost, s));
      GM_HIP(hipStreamSynchronize(s));
      if (to != &hst) std::memcpy((void*)&hst, to, sizeof hst);
      seen = hst.done ? hst.iter : launched;
    }
    if (hst.iter < seen) {
      // the status block did not advance: never loop on it
      g_hip_err = "internal error: the device loop made no progress";
      return GM_EHIP;
    }
    if (timing) {
      for (int64_t k = before; k < seen; ++k) {
        hipEvent_t* const e = events.ev[k % kMaxAhead];
        float t[4] = {0, 0, 0, 0};
        GM_HIP(hipEventSynchronize(e[phases ? 4 : 1]));  // (the slot is filled before it)
        for (int q = 0; q < (phases ? 4 : 1); ++q) GM_HIP(hipEventElapsedTime(&t[q], e[q], e[q + 1]));
        g_stats.rule_ms += t[0];
        g_stats.reduce_ms += t[1];
        g_stats.classify_ms += t[2];
        g_stats.split_ms += t[3];
        g_stats.rule_launches += 1;
      }
    }
    if (g_opt.log)
      std::fprintf(stderr, "gm: iter %lld n %lld I %.17g E %.6g T %.6g done %lld\n",
                   (long long)hst.iter, (long long)hst.n_active, hst.I, hst.E, hst.T,
                   (long long)hst.done);
    leaves_have = hst.leaf_count;
    if (hst.done) break;
    n = hst.n_active;
    n_before = hst.n_prev;
  }
  // (an iteration launched in vain returns at once, but is part of this call; the
  // adjoint kernels of gradient mode, which has none, follow on the stream)
  drain.owed = false;
  if (mirrored && !keep_leaves) GM_HIP(hipStreamSynchronize(s));

  out->I = hst.I;
  out->E = hst.E;
  out->status = (int)hst.status;
  out->final_n = hst.n_active;
  out->final_npar = hst.n_par;
  out->final_split = hst.split;
  out->buf = hst.buf;
  out->leaf_count = keep_leaves ? hst.leaf_count : 0;
  out->base = base;
  out->lay = lay;
  out->cap = cap;
  out->vol_omega = vol;
  g_stats.iterations = hst.iter;
  g_stats.regions_evaluated = hst.regions_evaluated;
  g_stats.evals = hst.regions_evaluated * nodes_per_region(d);
  g_stats.max_active = hst.max_active;
  g_stats.final_active = hst.n_active;
  g_stats.finished = hst.finished;
  g_stats.status = hst.status;
  g_stats.total_ms =
      std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t_start).count();
  g_last.valid = true;
  g_last.base = base;
  g_last.d = d;
  g_last.n = hst.n_active;
  g_last.npar = hst.n_par;
  g_last.split = hst.split;
  g_last.cap = cap;
  g_last.lay = lay;
  g_last.buf = hst.buf;
  return GM_OK;
}

}  // namespace gm

using namespace gm;

extern "C" {

int64_t gm_num_nodes(int d) {
  if (d < 1 || d > 62) return -1;
  return ((int64_t)1 << d) + 2 * (int64_t)d * d + 2 * (int64_t)d + 1;
}

int gm_integrate(int integrand_id, const double* params, int d, const double* lo, const double* hi,
                 double rel_tol, double abs_tol, int64_t max_regions, double* out_est,
                 double* out_err, void* stream) {
  int rc = validate(integrand_id, params, d, lo, hi, rel_tol, abs_tol);
  if (rc != GM_OK) return rc;
  if (!out_est || !out_err) return GM_EINVAL;
  std::lock_guard<std::mutex> lk(api_mutex());
  RunResult rr;
  rc = check_bounds(run_adaptive(integrand_id, params, d, lo, hi, rel_tol, abs_tol, max_regions,
                                 (hipStream_t)stream, false, &rr));
  if (rc != GM_OK) return rc;
  *out_est = rr.I;
  *out_err = rr.E;
  return rr.status;
}

int gm_integrate_noalloc(int integrand_id, const double* params, int d, const double* lo,
                         const double* hi, double rel_tol, double abs_tol, int64_t max_regions,
                         double* out_est, double* out_err, void* stream) {
  int rc = validate(integrand_id, params, d, lo, hi, rel_tol, abs_tol);
  if (rc != GM_OK) return rc;
  if (!out_est || !out_err || max_regions < 1) return GM_EINVAL;
  if (make_layout(d, max_regions).total > kNoallocScratchBytes) return GM_EINVAL;
  std::lock_guard<std::mutex> lk(api_mutex());
  char* base = nullptr;
  rc = noalloc_scratch(&base);
  if (rc != GM_OK) return rc;
  RunResult rr;
  rc = check_bounds(run_adaptive(integrand_id, params, d, lo, hi, rel_tol, abs_tol, max_regions,
                                 (hipStream_t)stream, false, &rr, base));
  if (rc != GM_OK) return rc;
  *out_est = rr.I;
  *out_err = rr.E;
  return rr.status;
}

int gm_eval_regions(int integrand_id, const double* params, int d, const double* lo,
                    const double* hi, int64_t n, const double* c, const double* h,
                    const int32_t* lvl, double* out_q, double* out_err, int32_t* out_axis,
                    void* stream) {
  int rc = validate(integrand_id, params, d, lo, hi, 1.0, 1.0);
  if (rc != GM_OK) return rc;
  if (n < 0 || (n > 0 && (!c || !h || !lvl || !out_q || !out_err || !out_axis))) return GM_EINVAL;
  for (int64_t r = 0; r < n; ++r)
    if (lvl[r] < 0 || lvl[r] > 65535) return GM_EINVAL;
  if (n == 0) return GM_OK;
  std::lock_guard<std::mutex> lk(api_mutex());
  hipStream_t s = (hipStream_t)stream;
  const int64_t cap = n;
  const int64_t lg = (n + 255) / 256;  // workgroups of the layout kernels
  if (lg > INT32_MAX) return GM_ENOMEM;  // (5e11 regions: beyond any memory)
  const Layout lay = make_layout(d, cap);
  char* base = nullptr;
  rc = acquire_workspace(lay.total, &base);
  if (rc != GM_OK) return rc;
  RuleArgs ra;
  std::memset(&ra, 0, sizeof ra);
  fill_params(integrand_id, d, params, ra.P);
  fill_consts(d, ra.K);
  ra.C[0] = ra.C[1] = (double*)(base + lay.C[0]);
  ra.H[0] = ra.H[1] = (double*)(base + lay.H[0]);
  ra.L[0] = ra.L[1] = (uint16_t*)(base + lay.L[0]);
  ra.cap = cap;
  ra.Q = (double*)(base + lay.Q);
  ra.ERR = (double*)(base + lay.ERR);
  ra.AXIS = (uint8_t*)(base + lay.AXIS);
  ra.partials = (double*)(base + lay.PART);
  ra.st = (Status*)(base + lay.ST);
  double vol = 1.0;
  for (int j = 0; j < d; ++j) vol = vol * (hi[j] - lo[j]);
  ra.vol_omega = vol;
  ra.n_fixed = n;
  // The caller's arrays as they are into the second buffer (levels: where Q will
  // be), laid out by a kernel: the host neither transposes nor allocates (30011
  // regions at d = 7: 390 -> 277 us a call).  A short list is laid out here: the two
  // layout kernels cost 27 us, the host 0.7 ns a coordinate (3 regions at d = 9: 85
  // / 114 us, 2193 at d = 13: 172 / 194).
  const bool on_host = n <= kHostListCoords / d;
  double* const cin = (double*)(base + (on_host ? lay.C[0] : lay.C[1]));
  double* const hin = (double*)(base + (on_host ? lay.H[0] : lay.H[1]));
  int32_t* const lin = (int32_t*)(base + lay.Q);
  std::vector<double> cs, hs;
  std::vector<uint16_t> ls;
  std::vector<uint8_t> ax;
  DrainOnError drain{s};
  if (on_host) {
    cs.resize((size_t)d * n);
    hs.resize((size_t)d * n);
    ls.resize((size_t)n);
    ax.resize((size_t)n);
    for (int64_t r = 0; r < n; ++r) {
      for (int j = 0; j < d; ++j) {
        cs[(size_t)j * n + r] = c[r * d + j];
        hs[(size_t)j * n + r] = h[r * d + j];
      }
      ls[r] = (uint16_t)lvl[r];
    }
  }
  GM_HIP(hipMemcpyAsync(cin, on_host ? cs.data() : c, sizeof(double) * d * n, hipMemcpyHostToDevice, s));
  GM_HIP(hipMemcpyAsync(hin, on_host ? hs.data() : h, sizeof(double) * d * n, hipMemcpyHostToDevice, s));
  if (on_host) {
    GM_HIP(hipMemcpyAsync(ra.L[0], ls.data(), sizeof(uint16_t) * n, hipMemcpyHostToDevice, s));
  } else {
    GM_HIP(hipMemcpyAsync(lin, lvl, sizeof(int32_t) * n, hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(list_in_kernel, dim3((unsigned)lg), dim3(256), 0, s, cin, hin, lin, d, n,
                       ra.C[0], ra.H[0], ra.L[0]);
    GM_HIP(hipGetLastError());
  }
  const int map = choose_mapping(d, integrand_id, n, true);
  // In chain form for every family: a region's err is a difference that a
  // resolved region cancels down to rounding, and a list's values are returned
  // one by one, so they keep the definition's order of operations (the launch is
  // 7% of the call: 18 of 277 us for 30011 regions at d = 7).
  GM_HIP(launch_rule(d, integrand_id, map, ra, rule_grid(map, n, d, integrand_id), s));
  int32_t* const aout = (int32_t*)hin;
  if (!on_host) {
    hipLaunchKernelGGL(list_out_kernel, dim3((unsigned)lg), dim3(256), 0, s, ra.AXIS, n, aout);
    GM_HIP(hipGetLastError());
  }
  GM_HIP(hipMemcpyAsync(out_q, ra.Q, sizeof(double) * n, hipMemcpyDeviceToHost, s));
  GM_HIP(hipMemcpyAsync(out_err, ra.ERR, sizeof(double) * n, hipMemcpyDeviceToHost, s));
  if (on_host) GM_HIP(hipMemcpyAsync(ax.data(), ra.AXIS, n, hipMemcpyDeviceToHost, s));
  else GM_HIP(hipMemcpyAsync(out_axis, aout, sizeof(int32_t) * n, hipMemcpyDeviceToHost, s));
  GM_HIP(hipStreamSynchronize(s));
  drain.owed = false;
  for (size_t r = 0; r < ax.size(); ++r) out_axis[r] = ax[r];
  rc = check_bounds(GM_OK);
  if (rc != GM_OK) return rc;
  return GM_OK;
}

int64_t gm_last_active(int64_t offset, int64_t n, double* c, double* h, int32_t* lvl, double* q,
                       double* err, int32_t* axis) {
  std::lock_guard<std::mutex> lk(api_mutex());
  if (!g_last.valid) return 0;
  if (offset < 0) return GM_EINVAL;
  char* base = g_last.base;
  const int64_t cnt = std::min<int64_t>(n, g_last.n - offset);
  const int d = g_last.d;
  const int b = g_last.buf;
  const Layout& L = g_last.lay;
  if (cnt <= 0) return g_last.n;
  // Stored records behind regions [offset, offset + cnt): the same records when
  // the set is not split, else the records r mod n_par (one or two ranges).
  const bool split = g_last.split != 0;
  const int64_t npar = g_last.npar;
  auto rec = [&](int64_t r) { return (split && r >= npar) ? r - npar : r; };
  int64_t q0 = rec(offset), q1 = rec(offset + cnt - 1);
  if (split && offset < npar && offset + cnt > npar) {  // the window holds "-" and "+" children
    q0 = 0;
    q1 = npar - 1;
  }
  const int64_t nq = q1 - q0 + 1;
  std::vector<double> pc((size_t)nq * d), ph((size_t)nq * d);
  std::vector<uint16_t> pl((size_t)nq);
  std::vector<uint8_t> pa((size_t)nq, 0);
  for (int j = 0; j < d; ++j) {
    if (hipMemcpy(pc.data() + (size_t)j * nq, base + L.C[b] + sizeof(double) * (j * g_last.cap + q0),
                  sizeof(double) * nq, hipMemcpyDeviceToHost) != hipSuccess)
      return hip_fail(hipGetLastError());
    if (hipMemcpy(ph.data() + (size_t)j * nq, base + L.H[b] + sizeof(double) * (j * g_last.cap + q0),
                  sizeof(double) * nq, hipMemcpyDeviceToHost) != hipSuccess)
      return hip_fail(hipGetLastError());
  }
  if (hipMemcpy(pl.data(), base + L.L[b] + sizeof(uint16_t) * q0, sizeof(uint16_t) * nq,
                hipMemcpyDeviceToHost) != hipSuccess)
    return hip_fail(hipGetLastError());
  if (split && hipMemcpy(pa.data(), base + L.PAX[b] + q0, nq, hipMemcpyDeviceToHost) != hipSuccess)
    return hip_fail(hipGetLastError());
  for (int64_t i = 0; i < cnt; ++i) {
    const int64_t r = offset + i;
    const int64_t k = rec(r) - q0;
    const bool plus = split && r >= npar;
    const int ax = pa[k];
    for (int j = 0; j < d; ++j) {
      double cj = pc[(size_t)j * nq + k], hj = ph[(size_t)j * nq + k];
      if (split && j == ax) {  // the split of the Sec. 3 loop, as the device applies it
        const double hp = hj * 0.5;
        cj = plus ? cj + hp : cj - hp;
        hj = hp;
      }
      if (c) c[i * d + j] = cj;
      if (h) h[i * d + j] = hj;
    }
    if (lvl) lvl[i] = pl[k] + (split ? 1 : 0);
  }
  const size_t o8 = sizeof(double) * (size_t)offset;
  if (q && hipMemcpy(q, base + L.Q + o8, sizeof(double) * cnt, hipMemcpyDeviceToHost) != hipSuccess)
    return hip_fail(hipGetLastError());
  if (err &&
      hipMemcpy(err, base + L.ERR + o8, sizeof(double) * cnt, hipMemcpyDeviceToHost) != hipSuccess)
    return hip_fail(hipGetLastError());
  if (axis) {
    std::vector<uint8_t> a((size_t)cnt);
    if (hipMemcpy(a.data(), base + L.AXIS + offset, cnt, hipMemcpyDeviceToHost) != hipSuccess)
      return hip_fail(hipGetLastError());
    for (int64_t r = 0; r < cnt; ++r) axis[r] = a[r];
  }
  return g_last.n;
}

int gm_set_workspace(void* device_ptr, size_t bytes) {
  std::lock_guard<std::mutex> lk(api_mutex());
  g_last.valid = false;
  if (!device_ptr || bytes == 0) {
    g_ext_ptr = nullptr;
    g_ext_bytes = 0;
    return GM_OK;
  }
  if (((uintptr_t)device_ptr & 255u) != 0) return GM_EINVAL;
  g_ext_ptr = device_ptr;
  g_ext_bytes = bytes;
  return GM_OK;
}

size_t gm_workspace_bytes(int d, int64_t max_regions, int mode) {
  if (d < kMinDim || d > kMaxDim || max_regions < 1) return 0;
  if (mode == 2) return batch_layout_bytes(d, max_regions);
  return make_layout(d, max_regions).total;
}

int gm_set_option(const char* key, int64_t value) {
  if (!key) return GM_EINVAL;
  std::lock_guard<std::mutex> lk(api_mutex());
  const std::string k(key);
#ifdef GM_CHECK
  // (GM_CHECK builds only) "check_selftest" = n: a kernel checks index n
  // against bound n without accessing memory; the call returns what the
  // bounds-check path makes of it (GM_EHIP, the violation in
  // gm_status_string(GM_EHIP)).
  if (k == "check_selftest") {
    hipLaunchKernelGGL(check_selftest_kernel, dim3(1), dim3(64), 0, 0, value);
    GM_HIP(hipGetLastError());
    GM_HIP(hipDeviceSynchronize());
    return check_bounds(GM_OK);
  }
#endif
  if (k == "init_log2_regions") {
    if (value < 0 || value > 30) return GM_EINVAL;
    g_opt.init_log2 = (int)value;
  } else if (k == "max_iters") {
    if (value < 1 || value > 1000000) return GM_EINVAL;
    g_opt.max_iters = value;
  } else if (k == "graph_iters") {
    if (value < 0 || value > 64) return GM_EINVAL;
    g_opt.graph_iters = (int)value;
  } else if (k == "lanes_per_region") {
    if (value < 0 || value > 64 || (value & (value - 1))) return GM_EINVAL;
    g_opt.lanes_per_region = (int)value;
  } else if (k == "timing") {
    if (value < 0 || value > 2) return GM_EINVAL;
    g_opt.timing = (int)value;
  } else if (k == "rule") {
    if (value < 0 || value > 2) return GM_EINVAL;
    g_opt.rule = (int)value;
  } else if (k == "err_model") {
    if (value < 0 || value > 1) return GM_EINVAL;
    g_opt.err_model = (int)value;
  } else if (k == "prune") {
    if (value < 0 || value > 1) return GM_EINVAL;
    g_opt.prune = (int)value;
  } else if (k == "log") {
    g_opt.log = value ? 1 : 0;
  } else {
    return GM_EINVAL;
  }
  return GM_OK;
}

const char* gm_status_string(int status) {
  switch (status) {
    case GM_OK: return "converged: E <= max(abs_tol, rel_tol*|I|)";
    case GM_MAX_REGIONS: return "stopped: region capacity reached";
    case GM_MAX_ITERS: return "stopped: iteration budget used up";
    case GM_PRECISION_LIMIT: return "stopped: every region retired by a numerical guard, E > T";
    case GM_NONFINITE: return "integrand or a rule sum was not finite";
    case GM_EINVAL: return "invalid argument";
    case GM_ENOMEM:
      g_enomem_text = "out of device memory (or workspace too small); last HIP error: " + g_hip_err;
      return g_enomem_text.c_str();
    case GM_EHIP: return g_hip_err.c_str();
    default: return "unknown status";
  }
}

int gm_last_stats(gm_stats* out) {
  if (!out) return GM_EINVAL;
  std::lock_guard<std::mutex> lk(api_mutex());
  *out = g_stats;
  return GM_OK;
}

}  // extern "C"
