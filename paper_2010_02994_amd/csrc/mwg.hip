// libhawkes: Metropolis-within-Gibbs moves of event locations and reweighted
// log-likelihoods, both O(N) given cached per-event terms (arXiv 2010.02994,
// Sec. 3: block-wise Metropolis updates of individual location variables;
// rates and compensator of Sec. 2.1).
//
// Cached state, n x 4 float64 per event (written by hawkes_event_terms):
//   a_i  background rate at event i per unit mu0   (sum over j of the background pair term)
//   b_i  self-excitation rate per unit theta        (sum over earlier j)
//   L_i  log lambda_i, lambda_i = mu0 a_i + theta b_i
//   p_i  theta b_i / lambda_i
// Moving the locations of a block of events changes row i's rate only through
// its pairs with the moved events, so Delta ell = sum_i log(lambda_i'/lambda_i)
// costs O(N * block) plus one full O(N) row per moved event.  The compensator
// does not depend on locations.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "../../include/hawkes.h"
#include "hawkes_common.hpp"
#include "hawkes_internal.hpp"

namespace hawkes {
namespace mwg {

constexpr int kBlock = 256;
constexpr double kGuard = 0x1p-16; // incremental update kept only above this share of its terms
constexpr int kSeg = 32;          // partner segments (workspace per event) of exactly recomputed rows
constexpr int kMaxSeg = 512;      // at most, when few rows are listed
constexpr int kExactGrid = 512;   // workgroups of the exact-row kernel's listed rows (grid-stride over tasks)
constexpr int kListThreads = 1024;
// Steps of fewer than kManyMoved moved events over at most this many events are two
// launches instead of three: the decision kernel (k_mwg_settle_few) merges the moved
// rows' chunk sums and recomputes the listed rows itself, kFewGrid workgroups.
constexpr int kFewEvents = 8192;
constexpr int kFewGrid = 128;
constexpr int kFewSegs = 32;   // partner segments of a listed row there, at most

struct Model {
  double mu0, theta;
  double cbg_unit, cse_unit;  // pair weights per unit mu0 / theta
  double alpha, beta, gamma;  // 1/(2 tau_x^2), 1/(2 tau_t^2), 1/(2 h^2)
  double omega;
};

struct Step {
  Model m;
  double* x;            // n x D, moved rows overwritten on accept
  const double* t;
  int n, nmove;         // events, moved events
  int nrb, rows;        // row blocks and rows per block
  int nchunk, chunk;    // partner chunks of the moved rows' sums and partners per chunk
  int64_t npart;        // segment sums that part holds
  double* terms;        // n x 4 cached state
  const int64_t* idx;   // nmove moved events, strictly increasing
  const double* xnew;   // nmove x D proposed locations
  const double* thresh; // accept iff Delta ell > *thresh
  double* out3;         // [Delta ell, accepted, status]
  // workspace
  double* new_a;        // n each
  double* new_b;
  double* dlog;         // incremental rows: log-rate change; listed and moved rows: old log-rate
  int* flag;            // 0 incremental, 1 recompute exactly, 2 moved
  double* bpart;        // nrb: per row block, sum of dlog over its incremental rows
  int* bcount;          // nrb: rows of the block needing an exact recompute
  int* stage;           // nrb x rows: those rows in index order
  int* list;            // n: all of them in index order
  // one buffer of shared_pairs(n) pairs (a, b), about n x kSeg:
  double* mrow;         // nmove: moved rows' sums
  double* mpart;        // nchunk x nmove: their chunk sums (at most n x kSeg / 2)
  double* part;         // npart: listed rows' segment sums
  int* nlisted;         // length of the list; [1]: workgroups of k_mwg_settle_few that are done with it
};

// Contributions of event j to row i, without the pair weights: background
// (excluded at equal times) and self-excitation (only from strictly earlier j).
template <int D>
__device__ __forceinline__ void pair_ab(const Model& m, const double* xi, double ti, const double* xj, double tj,
                                        double& a, double& b, const double* __restrict__ tab) {
  double r2 = 0.0;
#pragma unroll
  for (int q = 0; q < D; ++q) {
    const double dx = xi[q] - xj[q];
    r2 = fma(dx, dx, r2);
  }
  const double dt = ti - tj;
  a = dt != 0.0 ? exp_tab(-m.alpha * r2 - m.beta * dt * dt, tab) : 0.0;
  b = dt > 0.0 ? exp_tab(-m.omega * dt - m.gamma * r2, tab) : 0.0;
}

// The same without a branch: both exps are computed, and dropped where they do not
// count.
template <int D>
__device__ __forceinline__ void pair_ab_both(const Model& m, const double* xi, double ti, const double* xj, double tj,
                                             double& a, double& b, const double* __restrict__ tab) {
  double r2 = 0.0;
#pragma unroll
  for (int q = 0; q < D; ++q) {
    const double dx = xi[q] - xj[q];
    r2 = fma(dx, dx, r2);
  }
  const double dt = ti - tj;
  const double ea = exp_tab(-m.alpha * r2 - m.beta * dt * dt, tab);
  const double eb = exp_tab(-m.omega * fmax(dt, 0.0) - m.gamma * r2, tab);
  a = dt != 0.0 ? ea : 0.0;
  b = dt > 0.0 ? eb : 0.0;
}

// Position of event j in the moved list, or -1 (binary search; the list is
// read within its bounds whatever it holds).
__device__ __forceinline__ int find_moved(const int64_t* idx, int nmove, int j) {
  int lo = 0, hi = nmove - 1;
  while (lo <= hi) {
    const int mid = (lo + hi) >> 1;
    const int64_t v = idx[mid];
    if (v == j) return mid;
    if (v < j) lo = mid + 1;
    else hi = mid - 1;
  }
  return -1;
}

// Sum over the workgroup in a fixed order: a butterfly within each wave (every
// lane ends with its wave's total; each step adds the same two values on both
// lanes of a pair), then the wave totals in wave order.  Every thread calls it
// and gets the same value; its barriers also order earlier LDS writes.
__device__ __forceinline__ double block_sum(double v, double* sh) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = 0.0;
  for (int w = 0; w < (int)(blockDim.x >> 6); ++w) r += sh[w];
  __syncthreads();   // sh may be written again right after
  return r;
}

// Rows not moved: the change of (a_i, b_i) from the moved events' old and new
// places, and its log-rate change, summed per block in a fixed order.  When the
// change cancels most of the rate or of either part of it (the new value is
// below 2^-16 of the terms it was formed from, so its rounding error could
// exceed ~2^-37 of it) the row is listed for an exact recompute instead, so
// float64 cancellation neither decides a move nor corrupts the cached parts.
// A workgroup covers kBlock / RL rows with RL adjacent lanes per row: each lane
// takes every RL-th moved event, and butterfly steps combine the RL sums in a
// fixed order (the same on every lane), so a block of many moved events is not
// one long chain per row, and N = 50,000 rows make 782 workgroups of four waves
// rather than 196 of sixteen, which left a quarter of the chip idle.  Few moved
// events take one lane per row.
constexpr int kRowLanesMany = 4;
constexpr int kManyMoved = 8;   // moved events from which four lanes per row pay

template <int D, int RL>
__device__ __forceinline__ void moved_change(const Step& s, int blk) {
  constexpr int kRows = kBlock / RL;
  constexpr int kList = 64;    // moved events staged at a time
  __shared__ double s_old[kList][D];
  __shared__ double s_new[kList][D];
  __shared__ double s_t[kList];
  __shared__ int s_j[kList];
  __shared__ double sh[kBlock / 64];
  __shared__ int s_wcnt[kBlock / 64];
  __shared__ double s_exptab[kExpTab];   // 2^(j/kExpTab) for exp_tab (read after the loop's barrier)
  fill_exp_table(s_exptab);
  const int tid = threadIdx.x;
  const int rl = tid / RL, sub = tid % RL;
  const int i = blk * kRows + rl;
  const bool row = i < s.n;
  double xi[D], ti = 0.0;
#pragma unroll
  for (int q = 0; q < D; ++q) xi[q] = row ? s.x[(int64_t)i * D + q] : 0.0;
  if (row) ti = s.t[i];
  double da = 0.0, db = 0.0, oa = 0.0, ob = 0.0;
  int moved = 0;
  for (int c0 = 0; c0 < s.nmove; c0 += kList) {
    const int cn = min(kList, s.nmove - c0);
    __syncthreads();
    if (tid < cn) {
      const int64_t j = s.idx[c0 + tid];
      const bool ok = j >= 0 && j < s.n;
      s_j[tid] = ok ? (int)j : -1;
#pragma unroll
      for (int q = 0; q < D; ++q) {
        s_old[tid][q] = ok ? s.x[j * D + q] : 0.0;
        s_new[tid][q] = s.xnew[(int64_t)(c0 + tid) * D + q];
      }
      s_t[tid] = ok ? s.t[j] : 0.0;
    }
    __syncthreads();
    if (row) {
      for (int k = sub; k < cn; k += RL) {
        const int j = s_j[k];
        if (j < 0) continue;
        if (j == i) {
          moved = 1;
          continue;
        }
        double a0, b0, a1, b1;
        pair_ab<D>(s.m, xi, ti, s_old[k], s_t[k], a0, b0, s_exptab);
        pair_ab<D>(s.m, xi, ti, s_new[k], s_t[k], a1, b1, s_exptab);
        da += a1 - a0;
        db += b1 - b0;
        oa += a0;
        ob += b0;
      }
    }
  }
  // the lanes of a row are adjacent lanes of one wave, all present
#pragma unroll
  for (int o = 1; o < RL; o <<= 1) {
    da += __shfl_xor(da, o);
    db += __shfl_xor(db, o);
    oa += __shfl_xor(oa, o);
    ob += __shfl_xor(ob, o);
    moved |= __shfl_xor(moved, o);
  }
  da *= s.m.cbg_unit;
  oa *= s.m.cbg_unit;
  db *= s.m.cse_unit;
  ob *= s.m.cse_unit;
  int fl = 0;
  double dl = 0.0;
  if (row) {
    if (moved) {
      fl = 2;
    } else {
      const double a = s.terms[(int64_t)i * 4 + 0], b = s.terms[(int64_t)i * 4 + 1];
      const double na = a + da, nb = b + db;
      const double lam = s.m.mu0 * a + s.m.theta * b;
      const double lam1 = s.m.mu0 * na + s.m.theta * nb;
      const double formed_from = lam + s.m.mu0 * oa + s.m.theta * ob;
      const double fa = a + oa, fb = b + ob;   // magnitudes each part was formed from
      const bool kept = lam1 > kGuard * formed_from && !(fa > 0.0 && !(na > kGuard * fa)) &&
                        !(fb > 0.0 && !(nb > kGuard * fb));
      fl = kept ? 0 : 1;
      if (sub == 0) {
        s.new_a[i] = na;
        s.new_b[i] = nb;
      }
      if (fl == 0) dl = log1p((s.m.mu0 * da + s.m.theta * db) / lam);
    }
    if (sub == 0) {
      s.flag[i] = fl;
      // other rows: their old log-rate, for the exact change formed later
      s.dlog[i] = fl == 0 ? dl : s.terms[(int64_t)i * 4 + 2];
    }
  }
  // block sum of the rows' log-rate changes (one lane per row counts)
  const double bs = block_sum(sub == 0 ? dl : 0.0, sh);
  // stage the rows needing an exact recompute, in index order (one lane per row votes)
  const bool listed = row && sub == 0 && fl == 1;
  const unsigned long long msk = __ballot(listed);
  const int lane = tid & 63, w = tid >> 6;
  if (lane == 0) s_wcnt[w] = __popcll(msk);
  __syncthreads();
  int before = 0, total = 0;
#pragma unroll
  for (int ww = 0; ww < kBlock / 64; ++ww) {
    if (ww < w) before += s_wcnt[ww];
    total += s_wcnt[ww];
  }
  if (listed) s.stage[(int64_t)blk * kRows + before + __popcll(msk & ((1ull << lane) - 1ull))] = i;
  if (tid == 0) {
    s.bcount[blk] = total;
    s.bpart[blk] = bs;
    if (blk == 0) s.nlisted[1] = 0;
  }
}

// Moved rows: their sums over one chunk of partners, every event at its proposed
// place.  The workgroup's lanes are moved rows (up to 64; with fewer, 64 / P2
// lanes share a row, P2 the power of two that holds them) and its waves take a
// quarter each of every kBlock partners staged in LDS, which all lanes of a row
// read as a broadcast: no sum crosses lanes until the end.  (One moved row at a
// time, its partners across the lanes, took 33 us for 64 moved events at
// N = 50,000: a workgroup reduction per six partners and lane.)
//
// Launches of few such workgroups leave most SIMDs with one wave of them, bound by the
// latency of the chain through a pair: up to kFewSums they take two partners at a time
// without branches, so four exps are in flight.  N = 20,000 (79 workgroups), 20 moved
// events 19.4 -> 17.1 us a step, 64 moved 27.5 -> 24.7; with 196 workgroups (N = 50,000,
// 64 moved), whose waves hide it for each other, the exps this computes for later
// partners cost more: 30.1 -> 32.1.  (PAIRS: not in the kernel of few moved events, whose
// lanes have a few partners each; one event at N = 2,925 9.4 against 9.5 us a step.)
constexpr int kFewSums = 128;
template <int D, bool PAIRS>
__device__ __forceinline__ void moved_rows(const Step& s, int blk) {
  __shared__ double s_p[kBlock][D + 1];
  __shared__ int64_t s_idx[kBlock];
  __shared__ double s_ab[kBlock / 64][64][2];
  __shared__ double s_exptab[kExpTab];
  fill_exp_table(s_exptab);
  const int groups = (s.nmove + 63) / 64;
  const int c = blk / groups, g = blk % groups;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int in_group = min(64, s.nmove - g * 64);
  int p2 = 1;
  while (p2 < in_group) p2 <<= 1;
  const int e = g * 64 + (lane & (p2 - 1)), sub = lane / p2, subs = 64 / p2;
  const bool few = PAIRS && s.nchunk * groups <= kFewSums;
  const bool staged = s.nmove <= kBlock;   // the moved list fits LDS
  if (staged && tid < s.nmove) s_idx[tid] = s.idx[tid];
  int r = -1;
  double xr[D], tr = 0.0;
#pragma unroll
  for (int q = 0; q < D; ++q) xr[q] = 0.0;
  if (e < s.nmove) {
    const int64_t j = s.idx[e];
    if (j >= 0 && j < s.n) {
      r = (int)j;
      tr = s.t[r];
    }
#pragma unroll
    for (int q = 0; q < D; ++q) xr[q] = s.xnew[(int64_t)e * D + q];
  }
  double a = 0.0, b = 0.0;
  const int j_end = min(s.n, (c + 1) * s.chunk);
  for (int j0 = c * s.chunk; j0 < j_end; j0 += kBlock) {
    __syncthreads();
    const int j = j0 + tid;
    if (j < j_end) {
      const int pos = staged ? find_moved(s_idx, s.nmove, j) : find_moved(s.idx, s.nmove, j);
      const double* src = pos >= 0 ? s.xnew + (int64_t)pos * D : s.x + (int64_t)j * D;
#pragma unroll
      for (int q = 0; q < D; ++q) s_p[tid][q] = src[q];
      s_p[tid][D] = s.t[j];
    }
    __syncthreads();
    const int k_end = min(64 * w + 64, j_end - j0);
    if (r >= 0) {
      if (few) {
        for (int k = 64 * w + sub; k < k_end; k += 2 * subs) {
          // two partners at a time: their exps are independent chains
          const int k1 = min(k + subs, k_end - 1);
          double pa, pb, qa, qb;
          pair_ab_both<D>(s.m, xr, tr, s_p[k], s_p[k][D], pa, pb, s_exptab);
          pair_ab_both<D>(s.m, xr, tr, s_p[k1], s_p[k1][D], qa, qb, s_exptab);
          if (j0 + k != r) {
            a += pa;
            b += pb;
          }
          if (k + subs < k_end && j0 + k1 != r) {
            a += qa;
            b += qb;
          }
        }
      } else {
        for (int k = 64 * w + sub; k < k_end; k += subs) {
          if (j0 + k == r) continue;
          double pa, pb;
          pair_ab<D>(s.m, xr, tr, s_p[k], s_p[k][D], pa, pb, s_exptab);
          a += pa;
          b += pb;
        }
      }
    }
  }
  for (int o = p2; o < 64; o <<= 1) {
    a += __shfl_xor(a, o);
    b += __shfl_xor(b, o);
  }
  s_ab[w][lane][0] = a;
  s_ab[w][lane][1] = b;
  __syncthreads();
  if (w == 0 && lane < in_group) {
#pragma unroll
    for (int ww = 1; ww < kBlock / 64; ++ww) {
      a += s_ab[ww][lane][0];
      b += s_ab[ww][lane][1];
    }
    double* mp = s.mpart + ((int64_t)c * s.nmove + e) * 2;
    mp[0] = a * s.m.cbg_unit;
    mp[1] = b * s.m.cse_unit;
  }
}

// Both in one launch: neither reads what the other writes.  The longer workgroups go
// first: a moved rows' sum is 64 partners a wave whatever the block, a row block's change
// three to four exps for every (four lanes: every fourth) moved event.  N = 50,000: 64
// moved events 35.1 -> 30.2 us a step with the sums first, 300 moved 81.9 -> 92.4.
constexpr int kSumsFirst = 128;
template <int D, int RL>
__global__ void __launch_bounds__(kBlock) k_mwg_rows(Step s) {
  const int sums = (int)gridDim.x - s.nrb;   // workgroups of the moved rows' sums
  const bool sums_first = RL > 1 && s.nmove <= kSumsFirst;
  const int b = (int)blockIdx.x - (sums_first ? sums : 0);
  if (b >= 0 && b < s.nrb) moved_change<D, RL>(s, b);
  else moved_rows<D, (RL > 1)>(s, sums_first ? blockIdx.x : blockIdx.x - s.nrb);
}

// Partner segments per listed row: kSeg, or more when few rows are listed so
// that the tasks still spread over the grid, or fewer when most rows are listed
// and a large block's chunk sums take their part of the workspace (listed and
// moved rows are n at most together, so eight segments always fit).
__device__ __forceinline__ int segs_for(int cnt, const Step& s) {
  int segs = kSeg;
  while (segs > 8 && (int64_t)cnt * segs > s.npart) segs /= 2;
  while (segs < kMaxSeg && (int64_t)cnt * segs * 2 <= kExactGrid && (int64_t)cnt * segs * 2 <= s.npart) segs *= 2;
  return segs;
}

// Inclusive scan over the workgroup (kBlock threads): within each wave by
// shuffles, then the totals of the earlier waves.
__device__ __forceinline__ int block_scan(int v, int* s_wtot) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int u = __shfl_up(v, off);
    if (lane >= off) v += u;
  }
  if (lane == 63) s_wtot[wv] = v;
  __syncthreads();
  for (int w2 = 0; w2 < wv; ++w2) v += s_wtot[w2];
  return v;
}

// The listed rows in index order come from k_mwg_rows' per-block counts and
// staged rows: every workgroup scans the counts (each thread over a chunk of
// consecutive blocks) and finds any row of the list from the scan.
struct Listed {
  int cnt, per;
  const int* scan;   // LDS, kBlock: rows up to and including each thread's chunk
};
__device__ __forceinline__ Listed listed_rows(const Step& s, int* s_scan, int* s_wtot, int& own, int& lo, int& hi) {
  Listed L;
  const int tid = threadIdx.x;
  L.per = (s.nrb + kBlock - 1) / kBlock;
  lo = min(s.nrb, tid * L.per);
  hi = min(s.nrb, lo + L.per);
  own = 0;
  for (int b = lo; b < hi; ++b) own += s.bcount[b];
  s_scan[tid] = block_scan(own, s_wtot);
  __syncthreads();
  L.cnt = s_scan[kBlock - 1];
  L.scan = s_scan;
  return L;
}
__device__ __forceinline__ int listed_row(const Step& s, const Listed& L, int e) {
  // the first chunk whose inclusive count exceeds e, then the block inside it
  int c0 = 0, c1 = kBlock - 1;
  while (c0 < c1) {
    const int mid = (c0 + c1) >> 1;
    if (L.scan[mid] > e) c1 = mid; else c0 = mid + 1;
  }
  int rr = e - (c0 > 0 ? L.scan[c0 - 1] : 0);
  int rb = c0 * L.per;
  for (int cb = s.bcount[rb]; rr >= cb; cb = s.bcount[rb]) { rr -= cb; ++rb; }
  return s.stage[(int64_t)rb * s.rows + rr];
}

// One listed (unmoved) row's sums over partners [j0, j1), every event at its
// proposed place; this thread's share.
template <int D>
__device__ __forceinline__ void listed_sums(const Step& s, int r, int j0, int j1, const double* tab, double (&ab)[2]) {
  double xr[D];
#pragma unroll
  for (int q = 0; q < D; ++q) xr[q] = s.x[(int64_t)r * D + q];
  const double tr = s.t[r];
  double a = 0.0, b = 0.0;
  for (int j = j0 + threadIdx.x; j < j1; j += kBlock) {
    if (j == r) continue;
    // k_mwg_rows flagged the moved rows with 2: only they search the list
    const int pos = s.flag[j] == 2 ? find_moved(s.idx, s.nmove, j) : -1;
    double xj[D];
#pragma unroll
    for (int q = 0; q < D; ++q) xj[q] = pos >= 0 ? s.xnew[(int64_t)pos * D + q] : s.x[(int64_t)j * D + q];
    double pa, pb;
    pair_ab<D>(s.m, xr, tr, xj, s.t[j], pa, pb, tab);
    a += pa;
    b += pb;
  }
  ab[0] = a * s.m.cbg_unit;
  ab[1] = b * s.m.cse_unit;
}

// The listed rows, split into (row, partner segment) tasks over a fixed grid, and
// (after them, one wave per row) the moved rows' chunk sums added in a fixed order.
// Workgroup 0 also writes the list and its length, which the decision kernel reads.
constexpr int kMergeRows = kBlock / 64;
template <int D>
__global__ void __launch_bounds__(kBlock) k_mwg_exact(Step s) {
  __shared__ double sh[2 * kBlock];
  __shared__ int s_scan[kBlock];
  __shared__ int s_wtot[kBlock / 64];
  __shared__ double s_exptab[kExpTab];   // 2^(j/kExpTab) for exp_tab
  const int tid = threadIdx.x;
  if ((int)blockIdx.x >= kExactGrid) {
    const int e = ((int)blockIdx.x - kExactGrid) * kMergeRows + (tid >> 6), lane = tid & 63;
    if (e >= s.nmove) return;
    double a = 0.0, b = 0.0;
    for (int c = lane; c < s.nchunk; c += 64) {
      a += s.mpart[((int64_t)c * s.nmove + e) * 2 + 0];
      b += s.mpart[((int64_t)c * s.nmove + e) * 2 + 1];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      a += __shfl_xor(a, o);
      b += __shfl_xor(b, o);
    }
    if (lane == 0) {
      s.mrow[(int64_t)e * 2 + 0] = a;
      s.mrow[(int64_t)e * 2 + 1] = b;
    }
    return;
  }
  int own, lo, hi;
  const Listed L = listed_rows(s, s_scan, s_wtot, own, lo, hi);
  if (blockIdx.x == 0) {
    int pos = s_scan[tid] - own;
    for (int b = lo; b < hi; ++b) {
      const int c = s.bcount[b];
      for (int k = 0; k < c; ++k) s.list[pos++] = s.stage[(int64_t)b * s.rows + k];
    }
    if (tid == 0) *s.nlisted = L.cnt;
  }
  if (L.cnt == 0) return;
  fill_exp_table(s_exptab);
  __syncthreads();
  const int segs = segs_for(L.cnt, s);
  const int seg = (s.n + segs - 1) / segs;
  for (int64_t task = blockIdx.x; task < (int64_t)L.cnt * segs; task += kExactGrid) {
    const int e = (int)(task / segs), sg = (int)(task % segs);
    double ab[2];
    listed_sums<D>(s, listed_row(s, L, e), sg * seg, min(s.n, sg * seg + seg), s_exptab, ab);
    block_sum_n(ab, sh);
    if (tid == 0) {
      s.part[((int64_t)e * segs + sg) * 2 + 0] = ab[0];
      s.part[((int64_t)e * segs + sg) * 2 + 1] = ab[1];
    }
  }
}

// Decision and update in one launch.  Every workgroup checks the moved block,
// takes the moved and the listed rows' sums and adds the log-rate changes in
// the same fixed order, so all of them reach the same total and the same
// decision; each then updates its own rows on accept, and workgroup 0 reports.
// The moved and listed rows' old log-rates come from k_mwg_rows' copy (a
// workgroup updating its rows' cached terms must not change what another one
// reads).  (A device-wide fence in every workgroup of
// the exact kernel, to decide in its last workgroup instead, would write back
// the L2 of each die, which costs more than a launch.)
template <int D>
__global__ void __launch_bounds__(kBlock) k_mwg_settle(Step s) {
  __shared__ double sh[2 * kBlock];
  __shared__ double s_na[kBlock], s_nb[kBlock], s_dl[kBlock];
  __shared__ int s_own[kBlock];
  __shared__ int s_bad;
  const int tid = threadIdx.x;
  const int base = blockIdx.x * kBlock;
  s_own[tid] = 0;
  if (tid == 0) s_bad = 0;
  __syncthreads();
  double acc = 0.0;   // this thread's part of the sum of log-rate changes
  auto settle_row = [&](int r, double a, double b) {
    const double dl = log(s.m.mu0 * a + s.m.theta * b) - s.dlog[r];
    acc += dl;
    if (r >= base && r < base + kBlock) {
      s_na[r - base] = a;
      s_nb[r - base] = b;
      s_dl[r - base] = dl;
      s_own[r - base] = 1;
    }
  };
  for (int k = tid; k < s.nmove; k += kBlock) {
    const int64_t j = s.idx[k];
    bool bad = j < 0 || j >= s.n || (k > 0 && s.idx[k - 1] >= j);
#pragma unroll
    for (int q = 0; q < D; ++q) bad = bad || !isfinite(s.xnew[(int64_t)k * D + q]);
    if (bad) atomicOr(&s_bad, 1);
    else settle_row((int)j, s.mrow[(int64_t)k * 2 + 0], s.mrow[(int64_t)k * 2 + 1]);
  }
  const int cnt = *s.nlisted;
  const int segs = segs_for(cnt, s);
  // G lanes per listed row (segs / 4, at most a wave): they add strided
  // segments, a butterfly within the group combines them (the same fixed
  // order every time).  Many listed rows (G small) run side by side.
  const int G = min(64, segs / 4);
  const int grp = tid / G, gl = tid % G;
  for (int e = grp; e < cnt; e += kBlock / G) {
    double a = 0.0, b = 0.0;
    for (int sg = gl; sg < segs; sg += G) {
      a += s.part[((int64_t)e * segs + sg) * 2 + 0];
      b += s.part[((int64_t)e * segs + sg) * 2 + 1];
    }
    for (int o = G / 2; o > 0; o >>= 1) {
      a += __shfl_xor(a, o);
      b += __shfl_xor(b, o);
    }
    if (gl == 0) settle_row(s.list[e], a, b);
  }
  for (int b = tid; b < s.nrb; b += kBlock) acc += s.bpart[b];
  const double tot = block_sum(acc, sh);   // also orders the LDS writes above
  const bool bad = s_bad != 0;
  const bool accept = !bad && tot > *s.thresh;
  if (blockIdx.x == 0 && tid == 0) {
    s.out3[0] = bad ? NAN : tot;
    s.out3[1] = accept ? 1.0 : 0.0;
    s.out3[2] = bad ? (double)HAWKES_EDATA : 0.0;
  }
  if (!accept) return;
  const int i = base + tid;
  if (i < s.nmove) {
    const int64_t j = s.idx[i];
#pragma unroll
    for (int q = 0; q < D; ++q) s.x[j * D + q] = s.xnew[(int64_t)i * D + q];
  }
  if (i >= s.n) return;
  double* tp = s.terms + (int64_t)i * 4;
  const bool own = s_own[tid] != 0;
  const double na = own ? s_na[tid] : s.new_a[i], nb = own ? s_nb[tid] : s.new_b[i];
  if (s.flag[i] == 0 && na == tp[0] && nb == tp[1]) return;
  const double lam1 = s.m.mu0 * na + s.m.theta * nb;
  tp[0] = na;
  tp[1] = nb;
  tp[2] = tp[2] + (own ? s_dl[tid] : s.dlog[i]);
  tp[3] = s.m.theta * nb / lam1;
}

// Two-launch steps.  Every workgroup merges the moved rows' chunk sums (32 lanes a row).
// Where no row is listed, which the counts of k_mwg_rows tell all workgroups alike, each
// decides and updates its own rows as in k_mwg_settle.  Else they split the listed rows
// into (row, partner segment) tasks, and the last one to finish adds the segments,
// decides and updates every row: only it writes, after all others have read.  (The
// device-wide fence that this takes writes back the L2 of each die, so it is left to steps
// that list a row.)  Which workgroup is the last changes no bit of the sums.
//
// Two launches against three, one moved event at N = 2,925: 8.7 us a step against 10.4 on
// the device, and 9.5 against 10.7 to 12.2 where the host's launches bound it.  With rows
// listed (the first event moved away from that many of the next day), three launches and
// two: N = 2,925 1 row 15.5 and 15.6, 30 19.8 and 17.5, 300 101 and 36; N = 8,192 10 rows
// 15.4 and 17.2, 300 100 and 60, 8,191 1,817 and 868.  (Every workgroup recomputing all
// listed rows, so that none needs a fence: 1 row 18, 30 214, 300 2,045; N = 8,192, 8,191 rows
// 104,000.)  128 workgroups: with 64 300 rows 49, with 256 1 row 18.2.
template <int D>
__global__ void __launch_bounds__(kBlock) k_mwg_settle_few(Step s) {
  constexpr int LM = kBlock / kManyMoved;   // lanes per moved row
  static_assert(LM <= 64, "a moved row's lanes are one wave's");
  __shared__ double sh[2 * kBlock];
  __shared__ double s_exptab[kExpTab];   // 2^(j/kExpTab) for exp_tab
  __shared__ double s_ma[kManyMoved], s_mb[kManyMoved], s_mdl[kManyMoved];
  __shared__ int s_scan[kBlock];
  __shared__ int s_wtot[kBlock / 64];
  __shared__ int s_bad, s_last;
  const int tid = threadIdx.x;
  if (tid == 0) s_bad = 0;
  // what the decision needs is read first, so that no load waits behind the barriers
  const double thresh = *s.thresh;
  double acc = 0.0;   // this thread's part of the sum of log-rate changes
  for (int b = tid; b < s.nrb; b += kBlock) acc += s.bpart[b];
  const int km = tid / LM;   // this thread's moved row
  double ma = 0.0, mb = 0.0;
  if (km < s.nmove)
    for (int c = tid % LM; c < s.nchunk; c += LM) {
      ma += s.mpart[((int64_t)c * s.nmove + km) * 2 + 0];
      mb += s.mpart[((int64_t)c * s.nmove + km) * 2 + 1];
    }
  int own, lo, hi;
  const Listed L = listed_rows(s, s_scan, s_wtot, own, lo, hi);   // (its barriers order s_bad)
  const bool listed = L.cnt > 0;
  const int first = listed ? 0 : blockIdx.x * kBlock, end = listed ? s.n : min(s.n, first + kBlock);
  if (first >= s.n) return;   // nothing listed and no rows of its own
#pragma unroll
  for (int o = LM / 2; o > 0; o >>= 1) {
    ma += __shfl_xor(ma, o);
    mb += __shfl_xor(mb, o);
  }
  if (km < s.nmove && tid % LM == 0) {
    const int64_t j = s.idx[km];
    bool bad = j < 0 || j >= s.n || (km > 0 && s.idx[km - 1] >= j);
#pragma unroll
    for (int q = 0; q < D; ++q) bad = bad || !isfinite(s.xnew[(int64_t)km * D + q]);
    if (bad) {
      atomicOr(&s_bad, 1);
    } else {
      s_ma[km] = ma;
      s_mb[km] = mb;
      s_mdl[km] = log(s.m.mu0 * ma + s.m.theta * mb) - s.dlog[j];
      acc += s_mdl[km];
    }
  }
  int segs = 1;
  while (segs < kFewSegs && L.cnt * segs * 2 <= kFewGrid && 2 * segs * kBlock <= s.n) segs *= 2;
  // each listed row's segments added by as many lanes, use(row, a, b, log-rate change) by the
  // first of them
  const auto for_listed = [&](auto use) {
    for (int e0 = 0; e0 < L.cnt; e0 += kBlock / segs) {
      const int e = e0 + tid / segs, sg = tid % segs;
      double a = 0.0, b = 0.0;
      if (e < L.cnt) {
        a = s.part[((int64_t)e * segs + sg) * 2 + 0];
        b = s.part[((int64_t)e * segs + sg) * 2 + 1];
      }
      for (int o = segs / 2; o > 0; o >>= 1) {
        a += __shfl_xor(a, o);
        b += __shfl_xor(b, o);
      }
      if (e < L.cnt && sg == 0) {
        const int r = listed_row(s, L, e);
        use(r, a, b, log(s.m.mu0 * a + s.m.theta * b) - s.dlog[r]);
      }
    }
  };
  if (listed) {
    fill_exp_table(s_exptab);
    __syncthreads();
    const int seg = (s.n + segs - 1) / segs;
    for (int task = blockIdx.x; task < L.cnt * segs; task += gridDim.x) {
      const int e = task / segs, j0 = task % segs * seg;
      double ab[2];
      listed_sums<D>(s, listed_row(s, L, e), j0, min(s.n, j0 + seg), s_exptab, ab);
      block_sum_n(ab, sh);
      if (tid == 0) {
        s.part[(int64_t)task * 2 + 0] = ab[0];
        s.part[(int64_t)task * 2 + 1] = ab[1];
      }
    }
    __syncthreads();   // all of this workgroup's reads are done
    if (tid == 0)
      s_last = __hip_atomic_fetch_add(&s.nlisted[1], 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1;
    __syncthreads();
    if (!s_last) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    for_listed([&](int, double, double, double dl) { acc += dl; });
  }
  const double tot = block_sum(acc, sh);   // also orders the LDS writes above
  const bool bad = s_bad != 0;
  const bool accept = !bad && tot > thresh;
  if (first == 0 && tid == 0) {
    s.out3[0] = bad ? NAN : tot;
    s.out3[1] = accept ? 1.0 : 0.0;
    s.out3[2] = bad ? (double)HAWKES_EDATA : 0.0;
  }
  if (!accept) return;
  const auto update = [&](int i, double na, double nb, double dl) {
    double* tp = s.terms + (int64_t)i * 4;
    tp[0] = na;
    tp[1] = nb;
    tp[2] = tp[2] + dl;
    tp[3] = s.m.theta * nb / (s.m.mu0 * na + s.m.theta * nb);
  };
  for (int i = first + tid; i < end; i += kBlock) {
    if (s.flag[i] != 0) continue;
    const double na = s.new_a[i], nb = s.new_b[i];
    if (na != s.terms[(int64_t)i * 4 + 0] || nb != s.terms[(int64_t)i * 4 + 1]) update(i, na, nb, s.dlog[i]);
  }
  for_listed(update);
  if (tid < s.nmove) {
    const int64_t j = s.idx[tid];
    if (j >= first && j < end) {
      update((int)j, s_ma[tid], s_mb[tid], s_mdl[tid]);
#pragma unroll
      for (int q = 0; q < D; ++q) s.x[j * D + q] = s.xnew[(int64_t)tid * D + q];
    }
  }
}

// Log-likelihood and its derivatives in mu0 and theta at new weights, every
// other parameter as when the terms were computed (one workgroup):
//   ell = sum_i log(mu0 a_i + theta b_i) - sum_i (mu0 C_i + theta E_i)
// with C_i the background's time integral and E_i = 1 - exp(-omega (T - t_i)).
__global__ void __launch_bounds__(kListThreads) k_reweight(const double* t, int n, Model m, double tau_t,
                                                             const double* terms, double* out3) {
  __shared__ double sh[3 * kListThreads];
  const double T = t[n - 1];
  double ll = 0.0, gm = 0.0, gt = 0.0;
  for (int i = threadIdx.x; i < n; i += kListThreads) {
    const double a = terms[(int64_t)i * 4 + 0], b = terms[(int64_t)i * 4 + 1];
    const double lam = m.mu0 * a + m.theta * b;
    const double ti = t[i];
    const double za = (T - ti) / tau_t, zb = -ti / tau_t;
    const double C = 0.5 * erfc(-za * 0.70710678118654752440) - 0.5 * erfc(-zb * 0.70710678118654752440);
    const double E = -expm1(-m.omega * (T - ti));
    ll += log(lam) - m.mu0 * C - m.theta * E;
    gm += a / lam - C;
    gt += b / lam - E;
  }
  double v[3] = {ll, gm, gt};
  block_sum_n(v, sh);
  if (threadIdx.x == 0)
    for (int k = 0; k < 3; ++k) out3[k] = v[k];
}

static Model make_model(const hawkes_params_t* p, int d) {
  const double two_pi = 6.283185307179586476925286766559;
  Model m;
  m.mu0 = p->mu;
  m.theta = p->theta;
  m.cbg_unit = std::pow(two_pi, -0.5 * (d + 1)) * std::pow(p->h, -d) / p->tau;
  m.cse_unit = p->omega * std::pow(two_pi, -0.5 * d) * std::pow(p->xi, -d);
  m.alpha = 0.5 / (p->h * p->h);
  m.beta = 0.5 / (p->tau * p->tau);
  m.gamma = 0.5 / (p->xi * p->xi);
  m.omega = p->omega;
  return m;
}

static size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

// Pairs of the buffer that moved and listed rows share.  (Less n / 32 where the counts of
// 64-row blocks take more than those of 256-row blocks: the workspace's size stays below
// 32 segments a row and 256-row blocks.)
static int64_t shared_pairs(int64_t n) { return kSeg * n - (n > 2048 ? n / 32 : 0); }

// Workspace pieces for n events, in order.
struct Pieces {
  size_t new_a, new_b, dlog, flag, bpart, bcount, stage, list, part, nlisted, total;
};
static Pieces pieces(int64_t n) {
  const size_t nrb = (size_t)((n + kBlock / kRowLanesMany - 1) / (kBlock / kRowLanesMany));
  Pieces p;
  size_t o = 0;
  auto take = [&](size_t bytes) { const size_t at = o; o = align256(o + bytes); return at; };
  p.new_a = take(sizeof(double) * (size_t)n);
  p.new_b = take(sizeof(double) * (size_t)n);
  p.dlog = take(sizeof(double) * (size_t)n);
  p.flag = take(sizeof(int) * (size_t)n);
  p.bpart = take(sizeof(double) * nrb);
  p.bcount = take(sizeof(int) * nrb);
  p.stage = take(sizeof(int) * (size_t)((n + kBlock - 1) / kBlock * kBlock));
  p.list = take(sizeof(int) * (size_t)n);
  p.part = take(sizeof(double) * 2 * (size_t)shared_pairs(n));
  p.nlisted = take(2 * sizeof(int));
  p.total = o;
  return p;
}

template <int D>
static void launch(const Step& s, hipStream_t st) {
  const int grid = s.nrb + s.nchunk * ((s.nmove + 63) / 64);
  const int nset = (s.n + kBlock - 1) / kBlock;
  if (s.nmove >= kManyMoved) k_mwg_rows<D, kRowLanesMany><<<grid, kBlock, 0, st>>>(s);
  else k_mwg_rows<D, 1><<<grid, kBlock, 0, st>>>(s);
  if (s.n <= kFewEvents && s.nmove < kManyMoved) {
    static_assert(kFewEvents <= kFewGrid * kBlock, "every row has a workgroup");
    k_mwg_settle_few<D><<<kFewGrid, kBlock, 0, st>>>(s);
    return;
  }
  k_mwg_exact<D><<<kExactGrid + (s.nmove + kMergeRows - 1) / kMergeRows, kBlock, 0, st>>>(s);
  k_mwg_settle<D><<<nset, kBlock, 0, st>>>(s);
}

}  // namespace mwg
}  // namespace hawkes

extern "C" {

size_t hawkes_mwg_workspace_bytes(int64_t n) {
  if (n < 2 || n > (int64_t(1) << 30)) return 0;
  return hawkes::mwg::pieces(n).total;
}

int hawkes_mwg_step(double* x, const double* t, int64_t n, int d, const hawkes_params_t* p, double* terms,
                    const int64_t* idx, const double* x_new, int64_t nmove, const double* log_thresh, void* ws,
                    size_t ws_bytes, void* stream, double* out3) {
  using namespace hawkes::mwg;
  if (!x || !t || !p || !terms || !idx || !x_new || !log_thresh || !ws || !out3) return HAWKES_EINVAL;
  if (d < 1 || d > hawkes::kMaxD || nmove < 1 || nmove > n) return HAWKES_EINVAL;
  const size_t need = hawkes_mwg_workspace_bytes(n);
  if (need == 0 || ws_bytes < need) return HAWKES_EINVAL;
  if (!hawkes::valid_params(p)) return HAWKES_EPARAM;
  const Pieces pc = pieces(n);
  char* w = static_cast<char*>(ws);
  Step s;
  s.m = make_model(p, d);
  s.x = x;
  s.t = t;
  s.n = (int)n;
  s.nmove = (int)nmove;
  s.rows = kBlock / (nmove >= kManyMoved ? kRowLanesMany : 1);
  s.nrb = (int)((n + s.rows - 1) / s.rows);
  // kBlock partners per chunk, or as many more as keep the chunk sums of all
  // moved rows within half of the shared buffer
  const int64_t most = std::max<int64_t>(1, (int64_t)(kSeg / 2) * n / nmove);
  s.chunk = kBlock * (int)((n + kBlock * most - 1) / (kBlock * most));
  s.nchunk = (int)((n + s.chunk - 1) / s.chunk);
  s.terms = terms;
  s.idx = idx;
  s.xnew = x_new;
  s.thresh = log_thresh;
  s.out3 = out3;
  s.new_a = reinterpret_cast<double*>(w + pc.new_a);
  s.new_b = reinterpret_cast<double*>(w + pc.new_b);
  s.dlog = reinterpret_cast<double*>(w + pc.dlog);
  s.flag = reinterpret_cast<int*>(w + pc.flag);
  s.bpart = reinterpret_cast<double*>(w + pc.bpart);
  s.bcount = reinterpret_cast<int*>(w + pc.bcount);
  s.stage = reinterpret_cast<int*>(w + pc.stage);
  s.list = reinterpret_cast<int*>(w + pc.list);
  s.mrow = reinterpret_cast<double*>(w + pc.part);
  s.mpart = s.mrow + 2 * nmove;
  s.part = s.mpart + 2 * nmove * s.nchunk;
  s.npart = shared_pairs(n) - nmove * (s.nchunk + 1);
  s.nlisted = reinterpret_cast<int*>(w + pc.nlisted);
  hipStream_t st = static_cast<hipStream_t>(stream);
  (void)hipGetLastError();
  switch (d) {
    case 1: launch<1>(s, st); break;
    case 2: launch<2>(s, st); break;
    case 3: launch<3>(s, st); break;
    case 4: launch<4>(s, st); break;
    case 5: launch<5>(s, st); break;
    case 6: launch<6>(s, st); break;
    case 7: launch<7>(s, st); break;
    case 8: launch<8>(s, st); break;
  }
  return hipGetLastError() == hipSuccess ? HAWKES_OK : HAWKES_EDEVICE;
}

int hawkes_loglik_reweight(const double* t, int64_t n, int d, const hawkes_params_t* p, const double* terms,
                           void* stream, double* out3) {
  using namespace hawkes::mwg;
  if (!t || !p || !terms || !out3 || n < 2 || n > (int64_t(1) << 30) || d < 1 || d > hawkes::kMaxD)
    return HAWKES_EINVAL;
  if (!hawkes::valid_params(p)) return HAWKES_EPARAM;
  (void)hipGetLastError();
  k_reweight<<<1, kListThreads, 0, static_cast<hipStream_t>(stream)>>>(t, (int)n, make_model(p, d), p->tau, terms,
                                                                          out3);
  return hipGetLastError() == hipSuccess ? HAWKES_OK : HAWKES_EDEVICE;
}

}  // extern "C"
