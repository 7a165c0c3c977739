// gfx950 kernels of the Hawkes log-likelihood + gradient hot path.
//
// Notation (Sec. 2.1 of arXiv 2010.02994): for the ordered pair (i, j) with
// j earlier in time, r2 = |x_i - x_j|^2 and dt = t_i - t_j >= 0.
//   background term (symmetric)   e_bg = exp(-r2/(2 tau_x^2) - dt^2/(2 tau_t^2)),  dt != 0
//   excitation term (j -> i)      e_se = exp(-omega dt - r2/(2 h^2)),              dt > 0
// The weighted pair terms are mu_ij = c_bg e_bg and xi_ij = c_se e_se.
//
// Pass 1 accumulates, per event, the six unweighted sums
//   K = sum e_bg, R = sum e_bg r2, U = sum e_bg dt^2, J = sum e_se, V = sum e_se r2, W = sum e_se dt
// (K, R, U receive the pair from both endpoints; J, V, W only at the later one).
// Pass 2 accumulates the location gradient of App. A, scattering each
// unordered pair's coefficient into both endpoints.
//
// Mixed precision: coordinates are float32 offsets from the data center, the
// exponent is formed in base 2 with a constant shift S (terms carry a factor
// 2^S), exp is v_exp_f32, and per-tile float32 partials fold into float64.
// Rows whose rate sits below the shifted window are recomputed in float64 by
// the fix-ups (fix_rows, k_reduce2), so no event loses range.
#pragma once
#include <type_traits>

#include "hawkes_common.hpp"

namespace hawkes {

template <int D, bool MIX> struct Traits;
template <int D> struct Traits<D, true> {
  using Real = float;
  using ColT = double;   // partial sums stored outside a wave
  static constexpr int RW = ((D + 2 + 3) / 4) * 4;  // record words: coords, t, aux, pad
  struct alignas(16) Rec { float v[RW]; };
};
template <int D> struct Traits<D, false> {
  using Real = double;
  using ColT = double;
  static constexpr int RW = ((D + 2 + 1) / 2) * 2;
  struct alignas(16) Rec { double v[RW]; };
};

// ------------------------------------------------------------------ helpers

#ifndef HK_FP64_UNROLL
#define HK_FP64_UNROLL 4   // column steps per loop trip in the float64 passes
#endif

// Pointers taken from a request descriptor are generic; casting them to the
// global address space lets the compiler emit global (not flat) memory
// instructions with scalar base addresses.
#define HK_GLOBAL __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ HK_GLOBAL T* glb(T* p) {
  return (HK_GLOBAL T*)p;
}
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Exact culling: which of the two pair terms (kBg, kSe) can be nonzero for some
// pair of the band's rows with this column tile.  A term whose pairs all lie
// further apart in time than its kp.cull distance is exactly zero in this
// pass's arithmetic, so leaving it out changes no bit of any sum.  Records are
// time-sorted, so the band's first row (t_row0, read once per work item) and
// the tile's last column (read from the tile's records already staged in LDS)
// bound every pair's time difference.  Mixed records hold times relative to
// their own tile's first event; there t_row0 is the band's first row relative
// to the column tile's first event.  Far tiles of a ten-year window mostly keep
// one term: N = 50,000 with a ten-day background bandwidth has both terms in 10 %
// of its tiles in mixed precision (20 % in float64), the excitation alone in 67 %
// (80 %), none in 23 % (0 %).
constexpr int kBg = 1, kSe = 2, kBothTerms = 3;
template <int D, bool MIX, typename Real, typename Rec>
__device__ __forceinline__ int tile_terms(Real t_row0, const Rec* tile_recs, int tile, const KParams& kp) {
  const int last = min(kp.n - 1, tile * kTile + kTile - 1) - tile * kTile;
  int m;
  if constexpr (MIX) {
    const float dt = (float)t_row0 - (float)tile_recs[last].v[D];
    m = (dt > kp.cull_bgf ? 0 : kBg) | (dt > kp.cull_sef ? 0 : kSe);
  } else {
    const double dt = (double)t_row0 - (double)tile_recs[last].v[D];
    m = (dt > kp.cull_bg ? 0 : kBg) | (dt > kp.cull_se ? 0 : kSe);
  }
  return uni(m);
}

// Mixed records: an event's time is stored relative to the first event of its
// own column tile of kTile events (so the float32 offsets span one tile's time
// range), and for each column tile the rows' times are re-expressed relative to
// that tile's first event in float64 and rounded once: a pair's time
// difference then carries an absolute rounding error of about 2^-24 times
// (|dt| + the tile's time span), whatever the length of the window.
__device__ __forceinline__ double tile_origin(const double* t, int tile) {
  return glb(t)[(int64_t)tile * kTile];
}

// Which request of a batched launch owns block `blk`: the last request whose
// first block (offsets are non-decreasing) is <= blk.  kind 0: pair-pass
// items, 1: per-event blocks, 2: pack blocks, 3: reduction blocks.
__device__ __forceinline__ int find_req(const ReqDesc* __restrict__ reqs, int nreq, int blk, int kind) {
  if (nreq == 1) return 0;
  int lo = 0, hi = nreq - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    const int b = kind == 0 ? reqs[mid].blk_items
                : kind == 1 ? reqs[mid].blk_ev
                : kind == 2 ? reqs[mid].blk_pad
                            : reqs[mid].blk_red;
    if (b <= blk) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// ------------------------------------------------------------ work items

// Inclusive scan over the wave's lanes (DPP row shifts and broadcasts).
__device__ __forceinline__ int wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
  return v;
}

// Work items of band b: runs of item_tiles(b) column tiles.
__device__ __forceinline__ int band_items(const KParams& kp, int b) {
  const int nt = (min(kp.n, (b + 1) * kBandRows) + kTile - 1) / kTile;
  const int Lb = item_tiles(b, kp.b_fine, kp.L);
  return (nt + Lb - 1) / Lb;
}

// Items run band-major from the last (longest) band to the first.  The prepare
// launch's waves write the table, 64 consecutive items each: a wave finds its
// first item's band by scanning the bands' counts, 64 at a time, and its lanes
// walk on from there.  (Every workgroup of the passes finding its own band
// this way, with no table, cost them 3 % at N = 50,000: two integer divisions
// and a scan per wave against one load.)
__device__ __forceinline__ void write_items(const ReqDesc& rq, int wave_id, int waves) {
  const KParams& kp = rq.kp;
  const int lane = threadIdx.x & 63;
  for (int it0 = wave_id * 64; it0 < kp.items; it0 += waves * 64) {
    int band = 0, before = it0;   // band of item it0, items before it in that band
    for (int p0 = 0; p0 < kp.nb; p0 += 64) {
      const int b = kp.nb - 1 - (p0 + lane);
      const int ch = b >= 0 ? band_items(kp, b) : 0;
      const int incl = wave_scan(ch);
      const unsigned long long past = __ballot(incl > before);
      if (past != 0) {
        const int l = __builtin_ctzll(past);
        before -= __builtin_amdgcn_readlane(incl, l) - __builtin_amdgcn_readlane(ch, l);
        band = kp.nb - 1 - (p0 + l);
        break;
      }
      before -= __builtin_amdgcn_readlane(incl, 63);
    }
    int chunk = before + lane;
    for (int n_b = band_items(kp, band); chunk >= n_b && band > 0; n_b = band_items(kp, band)) {
      chunk -= n_b;
      --band;
    }
    if (it0 + lane < kp.items) {
      glb(rq.items)[it0 + lane].x = band;
      glb(rq.items)[it0 + lane].y = chunk;
    }
  }
}

// First item of band b: the items of the bands after it.
__device__ __forceinline__ int band_first_item(const KParams& kp, int b) {
  const int lane = threadIdx.x & 63;
  int sum = 0;
  for (int c = b + 1 + lane; c < kp.nb; c += 64) sum += band_items(kp, c);
  return __builtin_amdgcn_readlane(wave_scan(sum), 63);
}

// ------------------------------------------------------------ prepare

// Validation, packed records and tie groups; one thread per padded event.
// The mixed path's float32 origin is the spatial midpoint of the first and
// last events (any origin inside the data's extent keeps the offsets within
// the range).  first[i] is the first index with t == t[i] (sorted input), so
// for j < i: t_j < t_i  <=>  j < first[i].  Padded rows get first = 0, which
// makes every pair with them inactive.  Each block leaves its own "bad data"
// word (k_reduce1 joins them: the rate pass between them reads nothing out of
// bounds whatever the data).
template <int D, bool MIX>
__device__ __forceinline__ void prep_event(const ReqDesc& rq, int blk) {
  using Tr = Traits<D, MIX>;
  using Real = typename Tr::Real;
  const int i = blk * kEvBlock + threadIdx.x;
  const int n = rq.kp.n;
  const auto x = glb(rq.x);
  const auto t = glb(rq.t);
  typename Tr::Rec rr;
#pragma unroll
  for (int k = 0; k < Tr::RW; ++k) rr.v[k] = Real(0);
  int f = 0;
  bool bad = false;
  if (i < n) {
    const double ti = t[i];
    const double tp = i > 0 ? t[i - 1] : -INFINITY;
    bad = !isfinite(ti) || ti < 0.0 || !(ti >= tp);
#pragma unroll
    for (int k = 0; k < D; ++k) {
      const double v = x[(int64_t)i * D + k];
      bad = bad || !isfinite(v);
      if constexpr (MIX) {
        const double c = 0.5 * (x[k] + x[(int64_t)(n - 1) * D + k]);
        rr.v[k] = Real((v - c) * rq.kp.inv_tx);
      } else {
        rr.v[k] = Real(v);
      }
    }
    // mixed: time relative to the first event of the event's column tile
    rr.v[D] = MIX ? Real((ti - t[(int64_t)(i / kTile) * kTile]) * rq.kp.inv_tt) : Real(ti);
    // first index with time ti: i itself unless the previous event ties
    // (then a lower_bound of ti in t[0..i], a chain of dependent loads that
    // only tied events pay)
    int lo = 0, hi = i;
    if (tp < ti) lo = i;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (t[mid] < ti) lo = mid + 1; else hi = mid;
    }
    f = lo;
  }
  {
    const auto dst = glb(static_cast<typename Tr::Rec*>(rq.rec));
#pragma unroll
    for (int q = 0; q < Tr::RW; ++q) dst[i].v[q] = rr.v[q];
  }
  glb(rq.first)[i] = f;
  glb(static_cast<Real*>(rq.ps))[i] = Real(0);
  write_items(rq, blk * (kEvBlock / 64) + (threadIdx.x >> 6), rq.kp.n_pad / 64);
  const int any = __syncthreads_or(bad ? 1 : 0);
  if (threadIdx.x == 0) {
    glb(rq.bad)[blk] = any;
    if (blk == 0) glb(rq.status)[kStFlagCount] = 0;
  }
}

template <int D, bool MIX>
__global__ void __launch_bounds__(kEvBlock) k_prep(const ReqDesc* __restrict__ reqs, int nreq) {
  const ReqDesc& rq = reqs[find_req(reqs, nreq, blockIdx.x, 2)];
  prep_event<D, MIX>(rq, blockIdx.x - rq.blk_pad);
}

// Single-request form: the descriptor arrives as a kernel argument and is
// written to device memory for the later kernels.
template <int D, bool MIX>
__global__ void __launch_bounds__(kEvBlock) k_prep_one(ReqDesc d, ReqDesc* __restrict__ dst) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *dst = d;
  prep_event<D, MIX>(d, blockIdx.x);
}

// ------------------------------------------------------------ pair passes

// Stage one tile of 64 records into LDS (16-byte chunks), NT threads.
template <typename Rec, int NT>
struct TileStage {
  static constexpr int kChunks = 64 * (int)sizeof(Rec) / 16;
  static constexpr int kPer = (kChunks + NT - 1) / NT;
  Chunk16 r[kPer];
  template <typename P>
  __device__ __forceinline__ void load(P src, int tile) {
    const HK_GLOBAL Chunk16* s = (const HK_GLOBAL Chunk16*)(src + (int64_t)tile * kTile);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int c = threadIdx.x + k * NT;
      if (c < kChunks) { r[k].a = s[c].a; r[k].b = s[c].b; r[k].c = s[c].c; r[k].d = s[c].d; }
    }
  }
  __device__ __forceinline__ void store(Rec* dst) {
    Chunk16* s = reinterpret_cast<Chunk16*>(dst);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int c = threadIdx.x + k * NT;
      if (c < kChunks) s[c] = r[k];
    }
  }
};

// Step groups (float64 passes).  A work item is a row band against a run of
// column tiles, and a tile is a chain of 64 steps per wave (a step: the lane's
// rows against one column each).  At small N there are few items, so the chip
// holds a wave or two per SIMD and the chain's latency, not its issue, is the
// pass's time.  SP step groups of kWaves waves then share each tile: group h
// takes the steps [64 h / SP, 64 (h + 1) / SP) of the same rows and columns,
// and the groups' row sums are added in group order in LDS, so the partials
// that leave the workgroup, and the reductions' work, stay those of one group.
// split_for (hawkes.hip) says when.
//
// Every wave keeps its own column slots (a slot that two waves added to would
// depend on their timing).  Unsplit passes double-buffer them (one barrier per
// tile); split ones, whose workgroups do one tile or two, keep one buffer and
// a second barrier, so that several workgroups fit a CU's LDS.
template <int SP, int NQ, int QR = 0>
struct PassLds {
  static constexpr int kBufs = SP > 1 ? 1 : 2;
  static constexpr int kColumns = kBufs * SP * kWaves * NQ * kTile;
  static constexpr int kRowsOut = SP > 1 ? kBandRows * QR : 0;
  // the groups' row sums reuse the column slots once these are written out
  static constexpr int kDoubles = kColumns > kRowsOut ? kColumns : kRowsOut;
};

// The column sums of a tile, fixed-order over the waves' slots, to the band's
// column partials; CLEAR leaves the slots at zero for the next tile.
template <int SP, int NQ, bool CLEAR, typename P>
__device__ __forceinline__ void store_columns(double* __restrict__ acc, P pcol, const KParams& kp, int band, int tile) {
  for (int e = threadIdx.x; e < NQ * kTile; e += SP * kThreads) {
    const int q = e >> 6, c = e & 63;
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < SP * kWaves; ++w) {
      sum += acc[(w * NQ + q) * kTile + c];
      if (CLEAR) acc[(w * NQ + q) * kTile + c] = 0.0;
    }
    pcol[((int64_t)band * NQ + q) * kp.n_pad + tile * kTile + c] = sum;
  }
}

// Adds the step groups' row sums in group order; group 0 ends with the totals.
// `own` is this thread's slot base (row of the band), v its QR x R values.
template <int SP, int QR>
__device__ __forceinline__ void add_groups(double (&v)[kRowsPerLane][QR], double* __restrict__ lds, int group) {
  const int own = (threadIdx.x & (kThreads - 1));
#pragma unroll
  for (int g = 1; g < SP; ++g) {
    __syncthreads();   // the slots' last readers are done
    if (group == g) {
#pragma unroll
      for (int r = 0; r < kRowsPerLane; ++r)
#pragma unroll
        for (int q = 0; q < QR; ++q) lds[(r * QR + q) * kThreads + own] = v[r][q];
    }
    __syncthreads();
    if (group == 0) {
#pragma unroll
      for (int r = 0; r < kRowsPerLane; ++r)
#pragma unroll
        for (int q = 0; q < QR; ++q) v[r][q] += lds[(r * QR + q) * kThreads + own];
    }
  }
}

// Pass 1: rates and the moments the parameter gradient needs.
template <int D, bool MIX>
struct Pass1Rows {
  using Real = typename Traits<D, MIX>::Real;
  static constexpr int R = kRowsPerLane;
  Real x[R][D], t[R];   // mixed: t is relative to the current column tile's first event
  int first[R];
  Real a[R][6];        // per-tile partials (float32 in mixed, the running sums in float64)
  double acc[R][6];    // float64 running sums (mixed path only)
};

// A pair that does not interact (MASK): its exponent's high word becomes that
// of a huge negative number, so the exp is 0 (one select instead of two).
__device__ __forceinline__ double masked_exponent(bool active, double z) {
  constexpr int kHuge = (int)0xfe37e43c;   // -1e300
  return __hiloint2double(active ? __double2hiint(z) : kHuge, __double2loint(z));
}

// RU: also accumulate the background moments R and U (see k_pass1_mixed).
template <int D, bool MASK, bool RU, int SP, int TERMS>
__device__ __forceinline__ void pass1_tile(Pass1Rows<D, false>& S, const typename Traits<D, false>::Rec* __restrict__ cols,
                                           double* __restrict__ acc_w, int tile_base, const KParams& kp,
                                           const double* __restrict__ tab, int k_begin) {
  constexpr int R = kRowsPerLane;
  const int lane = threadIdx.x & 63;
  const double cb = kp.alpha, ct = kp.beta, cg = kp.gamma, cw = kp.omega;
#pragma unroll SP > 1 ? 2 : HK_FP64_UNROLL
  for (int kk = 0; kk < 64 / SP; ++kk) {
    const int c = lane ^ (k_begin + kk);
    const auto col = cols[c];
    double cK, cR, cU;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      double r2 = 0;
#pragma unroll
      for (int q = 0; q < D; ++q) {
        const double dx = S.x[r][q] - col.v[q];
        r2 = q == 0 ? dx * dx : __builtin_fma(dx, dx, r2);
      }
      const double dt = S.t[r] - col.v[D];
      const double dt2 = dt * dt;
      // exponents as one product plus a fused multiply-add each
      double zb = -__builtin_fma(cb, r2, ct * dt2);
      double zs = -__builtin_fma(cg, r2, cw * dt);
      if (MASK) {
        const bool act = (tile_base + c) < S.first[r];
        zb = masked_exponent(act, zb);
        zs = masked_exponent(act, zs);
      }
      const double eb = TERMS & kBg ? exp_tab(zb, tab) : 0.0;
      const double es = TERMS & kSe ? exp_tab(zs, tab) : 0.0;
      // raw r2, dt^2 and dt moments
      if (TERMS & kBg) S.a[r][0] += eb;
      if (RU && (TERMS & kBg)) {
        S.a[r][1] = __builtin_fma(eb, r2, S.a[r][1]);
        S.a[r][2] = __builtin_fma(eb, dt2, S.a[r][2]);
      }
      if (TERMS & kSe) {
        S.a[r][3] += es;
        S.a[r][4] = __builtin_fma(es, r2, S.a[r][4]);
        S.a[r][5] = __builtin_fma(es, dt, S.a[r][5]);
      }
      // column contributions summed over this lane's rows
      cK = r == 0 ? eb : cK + eb;
      if (RU) {
        cR = r == 0 ? eb * r2 : __builtin_fma(eb, r2, cR);
        cU = r == 0 ? eb * dt2 : __builtin_fma(eb, dt2, cU);
      }
    }
    if (TERMS & kBg) atomicAdd(&acc_w[0 * 64 + c], cK);
    if (RU && (TERMS & kBg)) {
      atomicAdd(&acc_w[1 * 64 + c], cR);
      atomicAdd(&acc_w[2 * 64 + c], cU);
    }
  }
}

template <int D, bool RU, int SP, bool CULL>
__global__ void __launch_bounds__(SP* kThreads) __attribute__((amdgpu_waves_per_eu(SP > 1 ? 4 : 1))) k_pass1(const ReqDesc* __restrict__ reqs, int nreq) {
  using Rec = typename Traits<D, false>::Rec;
  using Real = double;
  constexpr int R = kRowsPerLane;
  constexpr int NQ = RU ? 3 : 1;   // column sums
  constexpr int QR = RU ? 6 : 4;   // row sums stored per item
  using Lds = PassLds<SP, NQ, QR>;
  __shared__ Rec s_rec[2][kTile];
  __shared__ double s_acc[Lds::kDoubles];
  __shared__ double s_exptab[kExpTab];   // 2^(j/kExpTab) for exp_tab
  const int blk = blockIdx.x;
  const int rid = find_req(reqs, nreq, blk, 0);
  const ReqDesc& rq = reqs[rid];
  fill_exp_table(s_exptab);   // the tiles' first barrier comes before its first use
  const KParams& kp = rq.kp;
  const auto rec = glb(static_cast<const Rec*>(rq.rec));
  const auto first = glb(rq.first);
  const auto pcol = glb(static_cast<double*>(rq.pcol));
  const int item = blk - rq.blk_items;
  const int band = uni(glb(rq.items)[item].x), chunk = uni(glb(rq.items)[item].y);
  const int slot = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int wave = slot % kWaves, group = slot / kWaves;   // rows, step group
  const int row_base = band * kBandRows;
  const int row_end = min(kp.n, row_base + kBandRows);
  const int nt_band = (row_end + kTile - 1) / kTile;
  const int Lb = item_tiles(band, kp.b_fine, kp.L);
  const int tile0 = chunk * Lb;
  const int tile1 = min(tile0 + Lb, nt_band);
  const bool partial_band = row_base + kBandRows > kp.n;
  const int first_min = uni(first[row_base]);
  const double t_row0 = CULL ? rec[row_base].v[D] : 0.0;   // the band's first row

  Pass1Rows<D, false> S;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int gi = row_base + wave * 64 * R + r * 64 + lane;
    Rec rr;
#pragma unroll
    for (int q = 0; q < (int)(sizeof(Rec) / sizeof(rr.v[0])); ++q) rr.v[q] = rec[gi].v[q];
#pragma unroll
    for (int q = 0; q < D; ++q) S.x[r][q] = rr.v[q];
    S.t[r] = rr.v[D];
    S.first[r] = first[gi];
#pragma unroll
    for (int q = 0; q < 6; ++q) { S.a[r][q] = Real(0); S.acc[r][q] = 0.0; }
  }
  for (int e = threadIdx.x; e < Lds::kColumns; e += SP * kThreads) s_acc[e] = 0.0;
  TileStage<Rec, SP * kThreads> stage;
  stage.load(rec, tile0);
  for (int tile = tile0; tile < tile1; ++tile) {
    const int buf = (tile - tile0) & 1;
    stage.store(&s_rec[buf][0]);
    __syncthreads();
    if (tile + 1 < tile1) stage.load(rec, tile + 1);
    double* acc = s_acc + (Lds::kBufs > 1 ? buf : 0) * (Lds::kColumns / Lds::kBufs);
    double* acc_w = acc + slot * NQ * kTile;
    // column sums of the previous tile
    if (SP == 1 && tile > tile0)
      store_columns<SP, NQ, true>(s_acc + (buf ^ 1) * (Lds::kColumns / Lds::kBufs), pcol, kp, band, tile - 1);
    const bool full = !partial_band && (tile + 1) * kTile <= first_min;
    // terms that can be nonzero (with none, the tile's column sums stay zero)
    const int terms = CULL ? tile_terms<D, false>(t_row0, &s_rec[buf][0], tile, kp) : kBothTerms;
    if (terms == 0) {
    } else if (!full) {
      pass1_tile<D, true, RU, SP, kBothTerms>(S, s_rec[buf], acc_w, tile * kTile, kp, s_exptab, group * (64 / SP));
    } else if (terms == kBothTerms) {
      pass1_tile<D, false, RU, SP, kBothTerms>(S, s_rec[buf], acc_w, tile * kTile, kp, s_exptab, group * (64 / SP));
    } else if constexpr (CULL) {
      if (terms == kSe)
        pass1_tile<D, false, RU, SP, kSe>(S, s_rec[buf], acc_w, tile * kTile, kp, s_exptab, group * (64 / SP));
      else
        pass1_tile<D, false, RU, SP, kBg>(S, s_rec[buf], acc_w, tile * kTile, kp, s_exptab, group * (64 / SP));
    }
    if constexpr (SP > 1) {
      __syncthreads();
      store_columns<SP, NQ, true>(s_acc, pcol, kp, band, tile);
    }
  }
  if constexpr (SP == 1) {
    __syncthreads();
    store_columns<SP, NQ, false>(s_acc + ((tile1 - 1 - tile0) & 1) * (Lds::kColumns / Lds::kBufs), pcol, kp, band,
                                 tile1 - 1);
  }
  double rows[R][QR];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int q = 0; q < QR; ++q) rows[r][q] = S.a[r][RU || q == 0 ? q : q + 2];   // without RU: K, J, V, W
  if constexpr (SP > 1) {
    add_groups<SP, QR>(rows, s_acc, group);
    if (group != 0) return;
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int lr = wave * 64 * R + r * 64 + lane;
#pragma unroll
    for (int q = 0; q < QR; ++q)
      glb(static_cast<double*>(rq.prow))[((int64_t)item * QR + q) * kBandRows + lr] = rows[r][q];
  }
}

// ------------------------------------------------ fix-ups and finalize blocks
//
// They need the rate pass's sums (k_reduce1) and nothing of the gradient pass,
// and the gradient pass needs nothing of them, so in a gradient call they are
// the first blocks of its launch: they fill the chip beside it, and the call's
// chain is five launches on one stream (prepare, rate pass, reduce, gradient
// pass, reduce) with no event between streams.  Calls without a gradient run
// them as a launch of their own (k_side).

// Sum over a 16-lane row, then over the wave, by DPP adds in a fixed order;
// lane 63 (row_last: lane 15 of each row) ends with the sum.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, ROWS, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, ROWS, 0xf, false);
  return v + __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
__device__ __forceinline__ double row_sum_last(double v) {
  v = dpp_add<0x111, 0xf>(v);
  v = dpp_add<0x112, 0xf>(v);
  v = dpp_add<0x114, 0xf>(v);
  return dpp_add<0x118, 0xf>(v);
}
__device__ __forceinline__ double wave_sum_last(double v) {
  v = row_sum_last(v);
  v = dpp_add<0x142, 0xa>(v);
  return dpp_add<0x143, 0xc>(v);
}

// Fixed-order sums of NV (<= 64) values over the workgroup: within each wave,
// then the waves' totals in wave order (lane q of wave 0 adds value q).  sh:
// NV doubles per wave.  Thread 0 gets the totals; the last barrier frees sh.
template <int NV>
__device__ __forceinline__ void group_sum(double (&v)[NV], double* sh) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = blockDim.x >> 6;
#pragma unroll
  for (int q = 0; q < NV; ++q) v[q] = wave_sum_last(v[q]);
  if (lane == 63)
#pragma unroll
    for (int q = 0; q < NV; ++q) sh[wave * NV + q] = v[q];
  __syncthreads();
  if (wave == 0) {
    if (lane < NV) {
      double tot = sh[lane];
      for (int w = 1; w < nw; ++w) tot += sh[w * NV + lane];
      sh[lane] = tot;   // a wave's LDS operations run in order
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int q = 0; q < NV; ++q) v[q] = sh[q];
  }
  __syncthreads();
}

// Calls without a gradient, whose flagged rows have the chip to themselves: workgroups for a
// request of nblk event blocks (up to four a CU), and partner segments per flagged row, as
// many as keep kFixPartners partners a segment (with one a thread, 119 rows at N = 3,000
// took 7 us more than whole rows) and the tasks within four rounds.  (By the request's
// own size, not the launch's: a request's sums are the same in any batch.)
__host__ __device__ inline int fix_grid(int nblk) {
  return 4 * nblk < kFixGrid ? kFixGrid : 4 * nblk > 8 * kFixGrid ? 8 * kFixGrid : 4 * nblk;
}
constexpr int kFixSeg = 16;        // at most
constexpr int kFixPartners = 2048;
constexpr int kFixSegStride = 8;   // doubles per segment: fixpart holds three a row whatever the count
__device__ __forceinline__ int fix_segs(int cnt, const KParams& kp) {
  const int64_t most = min((int64_t)4 * fix_grid(kp.nblk), (int64_t)3 * kp.n);
  int segs = 1;
  while (segs < kFixSeg && 2 * segs * kFixPartners <= kp.n && (int64_t)cnt * 2 * segs <= most) segs *= 2;
  return segs;
}

// Exact float64 recomputation of each flagged row i: the six row sums and (in
// gradient calls) the row's own side of the location gradient,
//   sum_j [mu_ij/tau_x^2 + (t_j < t_i) xi_ij/h^2] (x_j - x_i) / lambda_i.
// A task finds the largest log pair term m among its partners and sums terms
// times exp(-m), so no term that matters can underflow.
//
// Gradient calls: one workgroup per row.  What the last reduction reads of row f of
// the list, fixpart[f * kFixStride + q]: q < 6 the unweighted sums times exp(-m), 6: m,
// 7: log lambda_i, 8: t_i, 9 ..: x_i, 17 ..: the gradient vector.  (Rows split
// over 16 partner segments, merged by every workgroup of the last reduction, cost it
// 14 us at N = 50,000 with about 40 flagged rows; whole rows cost nothing there, and
// their 136 us a row and workgroup at that size hide behind the gradient pass, or behind
// most of it where culling makes that short: N = 50,000, a two-day bandwidth, one flagged
// row 309 us a call, none 289.)
//
// Calls without a gradient have no pass to hide behind: fix_segs segments of the partners
// a row, each a task of its own, fixpart[(f * segs + g) * 8 + q]: q < 6 the segment's sums,
// 6: its m (-infinity: no partner).  final_block merges them.  Log-likelihoods of
// N = 50,000 events with whole rows on 128 workgroups and with segments, us: one flagged
// row (float64) 1,904 and 1,769 (none: 1,746), 22 (mixed) 973 and 853, 2,500 (mixed) 3,010
// and 1,410, 49,000 (mixed) 41,000 and 12,000.
//
// The ordered list of flagged rows comes from k_reduce1's per-block counts
// and staged rows: every workgroup scans the counts (each thread over a chunk
// of consecutive blocks) and finds its tasks' rows from the scan; workgroup 0
// of each request also writes the list, each row's list position and the
// count, which the next kernel reads.
template <int D, bool GRAD>
__device__ __forceinline__ void fix_rows(const ReqDesc& rq, int bx, int nbx, double* pool) {
  if (uni(glb(rq.status)[kStData]) != 0) return;
  const KParams& kp = rq.kp;
  const int tid = threadIdx.x, nt = blockDim.x;
  int* s_scan = reinterpret_cast<int*>(pool);            // nt
  double* sh = pool + nt / 2;                            // (6 + D) per wave
  int* s_wtot = reinterpret_cast<int*>(sh);              // one per wave
  const int per = (kp.nsblk + nt - 1) / nt;
  const int lo = min(kp.nsblk, tid * per), hi = min(kp.nsblk, lo + per);
  int own = 0;
  for (int b = lo; b < hi; ++b) own += glb(rq.bcount)[b];
  int incl = wave_scan(own);
  if ((tid & 63) == 63) s_wtot[tid >> 6] = incl;
  __syncthreads();
  for (int w = 0; w < (tid >> 6); ++w) incl += s_wtot[w];
  s_scan[tid] = incl;
  __syncthreads();
  const int cnt = s_scan[nt - 1];
  if (bx == 0) {
    int pos = incl - own;
    for (int b = lo; b < hi; ++b) {
      const int c = glb(rq.bcount)[b];
      for (int k = 0; k < c; ++k) {
        const int i = glb(rq.bstage)[(int64_t)b * kRedEv + k];
        glb(rq.list)[pos] = i;
        glb(rq.listpos)[i] = pos;
        ++pos;
      }
    }
    if (tid == 0) glb(rq.status)[kStFlagCount] = cnt;
  }
  const auto x = glb(rq.x);
  const auto t = glb(rq.t);
  const double wb = kp.cbg * kp.itx2, ws = kp.cse * kp.ih2;
  const int segs = GRAD ? 1 : fix_segs(cnt, kp), seg = (kp.n + segs - 1) / segs;
  for (int task = bx; task < cnt * segs; task += nbx) {
    const int f = task / segs, j0 = task % segs * seg, j1 = min(kp.n, j0 + seg);
    // row f of the list: the first chunk whose inclusive count exceeds f,
    // then the block inside it
    int c0 = 0, c1 = nt - 1;
    while (c0 < c1) {
      const int mid = (c0 + c1) >> 1;
      if (s_scan[mid] > f) c1 = mid; else c0 = mid + 1;
    }
    int r = f - (c0 > 0 ? s_scan[c0 - 1] : 0);
    int b = c0 * per;
    for (int cb = glb(rq.bcount)[b]; r >= cb; cb = glb(rq.bcount)[b]) { r -= cb; ++b; }
    const int i = glb(rq.bstage)[(int64_t)b * kRedEv + r];
    double xi[D];
#pragma unroll
    for (int q = 0; q < D; ++q) xi[q] = x[(int64_t)i * D + q];
    const double ti = t[i];
    // each partner's place is read a step ahead, so its latency lies beside the previous
    // one's arithmetic (a row of 50,000 partners 165 -> 136 us)
    double xn[D], tn = 0.0;
    const auto read = [&](int j) {
      const int jc = min(j, kp.n - 1);
#pragma unroll
      for (int q = 0; q < D; ++q) xn[q] = x[(int64_t)jc * D + q];
      tn = t[jc];
    };
    double m = -INFINITY;
    read(j0 + tid);
    for (int j = j0 + tid; j < j1; j += nt) {
      double r2 = 0;
#pragma unroll
      for (int q = 0; q < D; ++q) { const double dx = xi[q] - xn[q]; r2 += dx * dx; }
      const double dt = ti - tn;
      read(j + nt);
      if (j == i) continue;
      if (dt != 0.0) m = fmax(m, kp.log_cbg - kp.alpha * r2 - kp.beta * dt * dt);
      if (dt > 0.0) m = fmax(m, kp.log_cse - kp.omega * dt - kp.gamma * r2);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o));
    if ((tid & 63) == 0) sh[tid >> 6] = m;
    __syncthreads();
    for (int w = 0; w < (nt >> 6); ++w) m = fmax(m, sh[w]);
    __syncthreads();
    const double msub = m > -INFINITY ? m : 0.0;
    constexpr int NA = GRAD ? 6 + D : 6;
    double a[NA];
#pragma unroll
    for (int q = 0; q < NA; ++q) a[q] = 0.0;
    read(j0 + tid);
    for (int j = j0 + tid; j < j1; j += nt) {
      double dx[D], r2 = 0;
#pragma unroll
      for (int q = 0; q < D; ++q) { dx[q] = xn[q] - xi[q]; r2 += dx[q] * dx[q]; }
      const double dt = ti - tn;
      read(j + nt);
      if (j == i) continue;
      double c = 0.0;
      if (dt != 0.0) {
        const double e = exp(-kp.alpha * r2 - kp.beta * dt * dt - msub);
        a[0] += e; a[1] += e * r2; a[2] += e * dt * dt;
        c = wb * e;
      }
      if (dt > 0.0) {
        const double e = exp(-kp.omega * dt - kp.gamma * r2 - msub);
        a[3] += e; a[4] += e * r2; a[5] += e * dt;
        c += ws * e;
      }
      if constexpr (GRAD)
#pragma unroll
        for (int q = 0; q < D; ++q) a[6 + q] += c * dx[q];
    }
    group_sum(a, sh);
    if (tid == 0) {
      const auto fp = glb(rq.fixpart) + (int64_t)task * (GRAD ? kFixStride : kFixSegStride);
#pragma unroll
      for (int q = 0; q < 6; ++q) fp[q] = a[q];
      fp[6] = GRAD ? msub : m;
      if constexpr (GRAD) {
        const double lt = kp.cbg * a[0] + kp.cse * a[3];
        fp[7] = log(lt) + msub;   // -inf: the rate is zero
        fp[8] = ti;
#pragma unroll
        for (int q = 0; q < D; ++q) {
          fp[9 + q] = xi[q];
          fp[17 + q] = a[6 + q] / lt;
        }
      }
    }
  }
}

__device__ __forceinline__ double std_normal_cdf(double z) { return 0.5 * erfc(-z * 0.70710678118654752440); }
__device__ __forceinline__ double std_normal_pdf(double z) { return 0.39894228040143267794 * exp(-0.5 * z * z); }

// One row's terms that carry 1/lambda: log lambda and the six parameter
// gradients' shares, from its unweighted sums times exp(-scale); v[7] counts
// a zero rate.  Returns lambda exp(-scale).
template <int D>
__device__ __forceinline__ double rate_terms(const KParams& kp, const double (&s)[6], double scale, double (&v)[8]) {
  const double lt = kp.cbg * s[0] + kp.cse * s[3];
  const double il = 1.0 / lt;
  v[0] += log(lt) + scale;
  v[1] += kp.cbg_unit * s[0] * il;
  v[2] += kp.cbg * (s[1] / (kp.tau_x * kp.tau_x * kp.tau_x) - D * s[0] / kp.tau_x) * il;
  v[3] += kp.cbg * (s[2] / (kp.tau_t * kp.tau_t * kp.tau_t) - s[0] / kp.tau_t) * il;
  v[4] += kp.cse_unit * s[3] * il;
  v[5] += kp.cse * (s[3] / kp.omega - s[5]) * il;
  v[6] += kp.cse * (s[4] / (kp.h * kp.h * kp.h) - D * s[3] / kp.h) * il;
  v[7] += lt > 0.0 ? 0.0 : 1.0;
  return lt;
}

// Per-event outputs: background rate per unit mu0, self-excitation rate per
// unit theta, log lambda, and the probability that the event was triggered by
// an earlier one (self-excitation share of the rate).
__device__ __forceinline__ void store_terms(const ReqDesc& rq, int i, const double (&s)[6], double lt, double scale) {
  if (rq.terms == nullptr) return;
  const KParams& kp = rq.kp;
  const auto tp = glb(rq.terms) + (int64_t)i * 4;
  tp[0] = s[0] > 0.0 ? exp(log(kp.cbg_unit * s[0]) + scale) : 0.0;
  tp[1] = s[3] > 0.0 ? exp(log(kp.cse_unit * s[3]) + scale) : 0.0;
  tp[2] = log(lt) + scale;
  tp[3] = kp.cse * s[3] / lt;
}

// Per event: the compensator's terms and, for rows the fix-ups do not take,
// log lambda and the parameter gradient's; per-block fixed-order sums.
template <int D>
__device__ __forceinline__ void final_events(const ReqDesc& rq, int lb, double* pool) {
  if (uni(glb(rq.status)[kStData]) != 0) return;
  const KParams& kp = rq.kp;
  const int i = lb * kEvBlock + threadIdx.x;
  double v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (threadIdx.x < kEvBlock && i < kp.n) {
    double s[6];
#pragma unroll
    for (int q = 0; q < 6; ++q) s[q] = glb(rq.sums)[(int64_t)i * 6 + q];
    const double T = rq.t[kp.n - 1], ti = rq.t[i];   // t_N: the last of the sorted times
    if (glb(rq.flags)[i] == 0) {
      const double lt = rate_terms<D>(kp, s, kp.sigma_main, v);
      store_terms(rq, i, s, lt, kp.sigma_main);
    }
    const double a = (T - ti) / kp.tau_t, b = -ti / kp.tau_t;
    const double cdf_diff = std_normal_cdf(a) - std_normal_cdf(b);
    const double decay = exp(-kp.omega * (T - ti));
    const double omd = -expm1(-kp.omega * (T - ti));
    const double dtau = -kp.mu0 / (kp.tau_t * kp.tau_t) * ((T - ti) * std_normal_pdf(a) + ti * std_normal_pdf(b));
    v[0] -= kp.mu0 * cdf_diff + kp.theta * omd;
    v[1] -= cdf_diff;
    v[3] -= dtau;
    v[4] -= omd;
    v[5] -= kp.theta * (T - ti) * decay;
  }
  group_sum(v, pool);
  if (threadIdx.x == 0)
#pragma unroll
    for (int q = 0; q < 8; ++q) glb(rq.bpart)[(int64_t)lb * 8 + q] = v[q];
}

// Blocks of a gradient pass that take the fix-ups and the finalize terms.
__host__ __device__ inline int side_blocks(int nreq, int ev_blocks) { return nreq * kFixGrid + ev_blocks; }

template <int D, bool GRAD>
__device__ __forceinline__ void side_block(const ReqDesc* __restrict__ reqs, int nreq, int ev_blocks, int fix_blocks,
                                           double* pool) {
  int b = blockIdx.x;
  if (b < ev_blocks) {
    const ReqDesc& rq = reqs[find_req(reqs, nreq, b, 1)];
    final_events<D>(rq, b - rq.blk_ev, pool);
    return;
  }
  b -= ev_blocks;
  fix_rows<D, GRAD>(reqs[b / fix_blocks], b % fix_blocks, fix_blocks, pool);
}

// The same blocks alone (calls without a gradient).
template <int D>
__global__ void __launch_bounds__(kEvBlock) k_side(const ReqDesc* __restrict__ reqs, int nreq, int ev_blocks) {
  __shared__ double s_pool[kEvBlock + (kEvBlock / 64) * (8 + D)];
  side_block<D, false>(reqs, nreq, ev_blocks, fix_grid(ev_blocks / nreq), s_pool);
}

// Pass 2: location gradient.  For the pair (i later, j earlier)
//   c_ij = mu_ij (1/lambda_i + 1/lambda_j)/tau_x^2 + xi_ij/(lambda_i h^2)
// and d ell/d x_i += c_ij (x_j - x_i), d ell/d x_j += c_ij (x_i - x_j)   (App. A).
// Per event: pb = c_bg 2^-S/(lambda~ tau_x^2) in the record's aux slot (the
// column side), ps = c_se 2^-S/(lambda~ h^2) for the row side; both are 0 for
// rows the fix-up kernels handle.
template <int D, bool MIX>
struct Pass2Rows {
  using Real = typename Traits<D, MIX>::Real;
  static constexpr int R = kRowsPerLane;
  Real x[R][D], t[R], pb[R], ps[R];   // mixed: t is relative to the current column tile's first event
  int first[R];
  Real g[R][D];
  Real mom[2];        // mixed: per-tile sums of w r^2 and w dt^2 (w = background pair weight)
  double momd[2];     // their float64 running sums
  double acc[R][D];
};

template <int D, bool MASK, int SP, int TERMS>
__device__ __forceinline__ void pass2_tile(Pass2Rows<D, false>& S, const typename Traits<D, false>::Rec* __restrict__ cols,
                                           double* __restrict__ acc_w, int tile_base, const KParams& kp,
                                           const double* __restrict__ tab, int k_begin) {
  constexpr int R = kRowsPerLane;
  const int lane = threadIdx.x & 63;
  const double cb = kp.alpha, ct = kp.beta, cg = kp.gamma, cw = kp.omega;
#pragma unroll SP > 1 ? 2 : HK_FP64_UNROLL
  for (int kk = 0; kk < 64 / SP; ++kk) {
    const int c = lane ^ (k_begin + kk);
    const auto col = cols[c];
    double cgr[D];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      double dx[D];
      double r2 = 0;
#pragma unroll
      for (int q = 0; q < D; ++q) {
        dx[q] = S.x[r][q] - col.v[q];
        r2 = q == 0 ? dx[q] * dx[q] : __builtin_fma(dx[q], dx[q], r2);
      }
      const double dt = S.t[r] - col.v[D];
      const double dt2 = dt * dt;
      // exponents as one product plus a fused multiply-add each
      double zb = -__builtin_fma(cb, r2, ct * dt2);
      double zs = -__builtin_fma(cg, r2, cw * dt);
      if (MASK) {
        const bool act = (tile_base + c) < S.first[r];
        zb = masked_exponent(act, zb);
        zs = masked_exponent(act, zs);
      }
      const double eb = TERMS & kBg ? exp_tab(zb, tab) : 0.0;
      const double es = TERMS & kSe ? exp_tab(zs, tab) : 0.0;
      // background weight of the pair with both endpoints' 1/lambda; its r^2
      // and dt^2 moments give the R and U terms of the tau_x and tau_t gradients
      double coef;
      if (TERMS & kBg) {
        const double wb = eb * (S.pb[r] + col.v[D + 1]);
        coef = TERMS & kSe ? __builtin_fma(es, S.ps[r], wb) : wb;
        S.mom[0] = __builtin_fma(wb, r2, S.mom[0]);
        S.mom[1] = __builtin_fma(wb, dt2, S.mom[1]);
      } else {
        coef = es * S.ps[r];
      }
#pragma unroll
      for (int q = 0; q < D; ++q) {
        S.g[r][q] = __builtin_fma(-coef, dx[q], S.g[r][q]);
        cgr[q] = r == 0 ? coef * dx[q] : __builtin_fma(coef, dx[q], cgr[q]);
      }
    }
#pragma unroll
    for (int q = 0; q < D; ++q) atomicAdd(&acc_w[q * 64 + c], cgr[q]);
  }
}

template <int D, int SP, bool CULL>
__global__ void __launch_bounds__(SP* kThreads) __attribute__((amdgpu_waves_per_eu(SP > 1 ? 4 : 1))) k_pass2(const ReqDesc* __restrict__ reqs, int nreq, int ev_blocks) {
  using Rec = typename Traits<D, false>::Rec;
  using Real = double;
  constexpr int R = kRowsPerLane;
  constexpr int NQ = D;
  constexpr int QR = D;
  using Lds = PassLds<SP, NQ, QR>;
  __shared__ Rec s_rec[2][kTile];
  __shared__ double s_acc[Lds::kDoubles];
  __shared__ double s_exptab[kExpTab];   // 2^(j/kExpTab) for exp_tab
  __shared__ double s_red[2 * SP * kWaves];
  // the fix-up and finalize blocks come first (their results are read by the
  // next kernel only); nothing in the pair pass depends on them
  const int blk = (int)blockIdx.x - side_blocks(nreq, ev_blocks);
  if (blk < 0) {
    side_block<D, true>(reqs, nreq, ev_blocks, kFixGrid, s_acc);
    return;
  }
  const int rid = find_req(reqs, nreq, blk, 0);
  const ReqDesc& rq = reqs[rid];
  fill_exp_table(s_exptab);   // the tiles' first barrier comes before its first use
  const KParams& kp = rq.kp;
  const auto rec = glb(static_cast<const Rec*>(rq.rec));
  const auto first = glb(rq.first);
  const auto pcol = glb(static_cast<double*>(rq.pcol));
  const int item = blk - rq.blk_items;
  const int band = uni(glb(rq.items)[item].x), chunk = uni(glb(rq.items)[item].y);
  const int slot = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int wave = slot % kWaves, group = slot / kWaves;   // rows, step group
  const int row_base = band * kBandRows;
  const int row_end = min(kp.n, row_base + kBandRows);
  const int nt_band = (row_end + kTile - 1) / kTile;
  const int Lb = item_tiles(band, kp.b_fine, kp.L);
  const int tile0 = chunk * Lb;
  const int tile1 = min(tile0 + Lb, nt_band);
  const bool partial_band = row_base + kBandRows > kp.n;
  const int first_min = uni(first[row_base]);
  const double t_row0 = CULL ? rec[row_base].v[D] : 0.0;   // the band's first row

  Pass2Rows<D, false> S;
  S.mom[0] = S.mom[1] = 0.0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int gi = row_base + wave * 64 * R + r * 64 + lane;
    Rec rr;
#pragma unroll
    for (int q = 0; q < (int)(sizeof(Rec) / sizeof(rr.v[0])); ++q) rr.v[q] = rec[gi].v[q];
#pragma unroll
    for (int q = 0; q < D; ++q) { S.x[r][q] = rr.v[q]; S.g[r][q] = Real(0);  }
    S.t[r] = rr.v[D];
    S.pb[r] = rr.v[D + 1];
    S.ps[r] = glb(static_cast<const Real*>(rq.ps))[gi];
    S.first[r] = first[gi];
  }
  for (int e = threadIdx.x; e < Lds::kColumns; e += SP * kThreads) s_acc[e] = 0.0;
  TileStage<Rec, SP * kThreads> stage;
  stage.load(rec, tile0);
  for (int tile = tile0; tile < tile1; ++tile) {
    const int buf = (tile - tile0) & 1;
    stage.store(&s_rec[buf][0]);
    __syncthreads();
    if (tile + 1 < tile1) stage.load(rec, tile + 1);
    double* acc = s_acc + (Lds::kBufs > 1 ? buf : 0) * (Lds::kColumns / Lds::kBufs);
    double* acc_w = acc + slot * NQ * kTile;
    // column sums of the previous tile
    if (SP == 1 && tile > tile0)
      store_columns<SP, NQ, true>(s_acc + (buf ^ 1) * (Lds::kColumns / Lds::kBufs), pcol, kp, band, tile - 1);
    const bool full = !partial_band && (tile + 1) * kTile <= first_min;
    // terms that can be nonzero (with none, the tile's column sums stay zero)
    const int terms = CULL ? tile_terms<D, false>(t_row0, &s_rec[buf][0], tile, kp) : kBothTerms;
    if (terms == 0) {
    } else if (!full) {
      pass2_tile<D, true, SP, kBothTerms>(S, s_rec[buf], acc_w, tile * kTile, kp, s_exptab, group * (64 / SP));
    } else if (terms == kBothTerms) {
      pass2_tile<D, false, SP, kBothTerms>(S, s_rec[buf], acc_w, tile * kTile, kp, s_exptab, group * (64 / SP));
    } else if constexpr (CULL) {
      if (terms == kSe)
        pass2_tile<D, false, SP, kSe>(S, s_rec[buf], acc_w, tile * kTile, kp, s_exptab, group * (64 / SP));
      else
        pass2_tile<D, false, SP, kBg>(S, s_rec[buf], acc_w, tile * kTile, kp, s_exptab, group * (64 / SP));
    }
    if constexpr (SP > 1) {
      __syncthreads();
      store_columns<SP, NQ, true>(s_acc, pcol, kp, band, tile);
    }
  }
  if constexpr (SP == 1) {
    __syncthreads();
    store_columns<SP, NQ, false>(s_acc + ((tile1 - 1 - tile0) & 1) * (Lds::kColumns / Lds::kBufs), pcol, kp, band,
                                 tile1 - 1);
  }
  // the item's two moment sums, fixed-order over the workgroup
  double mom[2] = {S.mom[0], S.mom[1]};
  group_sum(mom, s_red);
  if (threadIdx.x == 0) {
    glb(rq.mompart)[(int64_t)item * 2 + 0] = mom[0];
    glb(rq.mompart)[(int64_t)item * 2 + 1] = mom[1];
  }
  if constexpr (SP > 1) {
    add_groups<SP, QR>(S.g, s_acc, group);
    if (group != 0) return;
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int lr = wave * 64 * R + r * 64 + lane;
#pragma unroll
    for (int q = 0; q < D; ++q) glb(static_cast<double*>(rq.prow))[((int64_t)item * D + q) * kBandRows + lr] = S.g[r][q];
  }
}

// ------------------------------------------------ mixed-precision pair passes
//
// The float32 passes keep the symmetric (column) sums out of LDS atomics:
// at step k of a 64-column tile, lane l pairs its rows with column (l + k) mod 64,
// and the column accumulators rotate one lane per step with a DPP wave_rol:1
// fused into the add (acc <- acc[lane + 1] + contribution), so after step k
// lane l holds the partial sum of column (l + k) mod 64.  The tile's records
// sit in LDS twice in a row, so the column read is lds[lane + k] with a
// constant offset.
//
// Float32 sums are micro-partials of at most 32 terms, folded into float64:
// every kColSteps = 32 / kRowsPerLane steps (16 steps x 2 rows = 32 terms) each lane adds
// its rotating column accumulator, converted to float64, to its column's slot
// of the wave's float64 LDS row with an LDS add (lanes hold distinct columns
// and a wave's LDS operations run in program order, so each slot receives its
// four adds in a fixed order), and restarts it at zero; the row sums are
// folded into their float64 accumulators every kRowFold = 32 steps.
// Everything stored outside the wave is float64.
constexpr int kColSteps = 32 / kRowsPerLane;
// Exponent of a pair that does not interact, selected after the exponents are formed: the
// scales mG and mW may be infinite in float32 (tau_x/h beyond 2e19, omega tau_t beyond
// 2e38), and infinity times the zero distance or time difference of an event with itself
// would make an exponent that starts at -infinity NaN.
constexpr float kNoPair = -INFINITY;
constexpr float kHalfLog2e = (float)(0.5 * 1.4426950408889634074);   // mA = mB

// A constant of the pair loop in a vector register.  A float32 operation with
// a scalar-register operand issues at half the rate of one on vector registers
// or literals (the peaks microbenchmark: 61 against 112 lanes per CU and clock for
// a multiply, 59 against 114 for a fused multiply-add), and the exponents take four
// such operations per pair.
__device__ __forceinline__ float in_vgpr(float v) {
  asm("" : "+v"(v));
  return v;
}
constexpr int kRowFold = 32;
static_assert(kColSteps * kRowsPerLane <= 32 && kRowFold <= 32 && kRowFold % kColSteps == 0 && 64 % kRowFold == 0,
              "float32 micro-partials hold at most 32 terms");

__device__ __forceinline__ float rol1(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x134, 0xf, 0xf, false));
}

template <int D, bool MASK, bool RU, int TERMS>
__device__ __forceinline__ void pass1_tile_mixed(Pass1Rows<D, true>& S, const typename Traits<D, true>::Rec* __restrict__ cols,
                                                 double* __restrict__ acc_w, int tile_base, const KParams& kp) {
  constexpr int R = kRowsPerLane;
  const int lane = threadIdx.x & 63;
  const float mW = in_vgpr(kp.mW), mG = in_vgpr(kp.mG), sh = in_vgpr(kp.S);
  const typename Traits<D, true>::Rec* __restrict__ my = cols + lane;
  // The exponents of kRateExpSteps consecutive steps are formed first and
  // their exps issued back to back, so no exp result is consumed by the very
  // next instruction; the steps are then accumulated in order.
  constexpr int KS = kRateExpSteps;
  static_assert(kColSteps % KS == 0, "exp groups must not straddle a flush");
  constexpr int UO = HK_RATE_UNROLL >= kRowFold ? HK_RATE_UNROLL / kRowFold : 1;
  constexpr int UC = HK_RATE_UNROLL >= kRowFold ? kRowFold / kColSteps : 1;
#pragma unroll UO
  for (int k2 = 0; k2 < 64; k2 += kRowFold) {
#pragma unroll UC
  for (int kc = 0; kc < kRowFold; kc += kColSteps) {
    const int k1 = k2 + kc;
    float aK = 0.f, aR = 0.f, aU = 0.f;
#pragma unroll
    for (int kk = 0; kk < kColSteps; kk += KS) {
      const int k0 = k1 + kk;
      float r2v[KS][R], dtv[KS][R], ebv[KS][R], esv[KS][R];
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const auto col = my[k0 + s];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          float r2 = 0.f;
#pragma unroll
          for (int q = 0; q < D; ++q) {
            const float dx = S.x[r][q] - col.v[q];
            r2 = q == 0 ? dx * dx : dx * dx + r2;
          }
          const float dt = S.t[r] - col.v[D];
          r2v[s][r] = r2;
          dtv[s][r] = dt;
          const bool act = !MASK || (tile_base + ((lane + k0 + s) & 63)) < S.first[r];
          const float zb = __builtin_fmaf(-kHalfLog2e, dt * dt, __builtin_fmaf(-kHalfLog2e, r2, sh));
          const float zs = __builtin_fmaf(-mW, dt, __builtin_fmaf(-mG, r2, sh));
          ebv[s][r] = act ? zb : kNoPair;
          esv[s][r] = act ? zs : kNoPair;
        }
      }
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if (TERMS & kBg) ebv[s][r] = __builtin_amdgcn_exp2f(ebv[s][r]);
          if (TERMS & kSe) esv[s][r] = __builtin_amdgcn_exp2f(esv[s][r]);
        }
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        float cK, cR, cU;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const float r2 = r2v[s][r], dt = dtv[s][r], dt2 = dt * dt;
          const float eb = ebv[s][r], es = esv[s][r];
          if (TERMS & kBg) S.a[r][0] += eb;
          if (RU && (TERMS & kBg)) {
            S.a[r][1] = eb * r2 + S.a[r][1];
            S.a[r][2] = eb * dt2 + S.a[r][2];
          }
          if (TERMS & kSe) {
            S.a[r][3] += es;
            S.a[r][4] = es * r2 + S.a[r][4];
            S.a[r][5] = es * dt + S.a[r][5];
          }
          // column contributions summed over this lane's rows (no "+ 0": a
          // signed zero keeps the compiler from folding it)
          cK = r == 0 ? eb : cK + eb;
          if (RU) {
            cR = r == 0 ? eb * r2 : eb * r2 + cR;
            cU = r == 0 ? eb * dt2 : eb * dt2 + cU;
          }
        }
        if (TERMS & kBg) aK = rol1(aK) + cK;
        if (RU && (TERMS & kBg)) {
          aR = rol1(aR) + cR;
          aU = rol1(aU) + cU;
        }
      }
    }
    // column flush: this lane now holds column (lane + k1 + kColSteps - 1) mod 64
    const int c = (lane + k1 + kColSteps - 1) & 63;
    if (TERMS & kBg) atomicAdd(&acc_w[0 * 64 + c], (double)aK);
    if (RU && (TERMS & kBg)) { atomicAdd(&acc_w[1 * 64 + c], (double)aR); atomicAdd(&acc_w[2 * 64 + c], (double)aU); }
  }
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      if (!RU && (q == 1 || q == 2)) continue;
      if (!(TERMS & (q < 3 ? kBg : kSe))) continue;
      S.acc[r][q] += (double)S.a[r][q];
      S.a[r][q] = 0.f;
    }
  }
}

// RU: also accumulate the background moments R = sum e r^2 and U = sum e dt^2
// (six row sums, three column sums).  Without RU (gradient calls) the rate
// pass keeps K, J, V, W (four row sums, one column sum) and the gradient pass
// forms the two moments' contributions to the parameter gradient instead.
template <int D, bool RU, bool CULL>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(rate_waves(D, RU)))) k_pass1_mixed(const ReqDesc* __restrict__ reqs, int nreq) {
  using Rec = typename Traits<D, true>::Rec;
  using Real = float;
  constexpr int R = kRowsPerLane;
  constexpr int NQ = RU ? 3 : 1;   // column sums
  constexpr int QR = RU ? 6 : 4;   // row sums stored per item
  using Lds = PassLds<1, NQ>;
  __shared__ Rec s_rec[2][2 * kTile];
  __shared__ double s_trow[R * kThreads];   // the rows' event times
  __shared__ double s_acc[Lds::kDoubles];
  const int blk = blockIdx.x;
  const int rid = find_req(reqs, nreq, blk, 0);
  const ReqDesc& rq = reqs[rid];
  const KParams& kp = rq.kp;
  const auto rec = glb(static_cast<const Rec*>(rq.rec));
  const auto first = glb(rq.first);
  const auto pcol = glb(static_cast<double*>(rq.pcol));
  const int item = blk - rq.blk_items;
  const int band = uni(glb(rq.items)[item].x), chunk = uni(glb(rq.items)[item].y);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int row_base = band * kBandRows;
  const int row_end = min(kp.n, row_base + kBandRows);
  const int nt_band = (row_end + kTile - 1) / kTile;
  const int Lb = item_tiles(band, kp.b_fine, kp.L);
  const int tile0 = chunk * Lb;
  const int tile1 = min(tile0 + Lb, nt_band);
  const bool partial_band = row_base + kBandRows > kp.n;
  const int first_min = uni(first[row_base]);
  const double t_row0 = CULL ? glb(rq.t)[row_base] : 0.0;   // the band's first row

  Pass1Rows<D, true> S;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int gi = row_base + wave * 64 * R + r * 64 + lane;
    Rec rr;
#pragma unroll
    for (int q = 0; q < (int)(sizeof(Rec) / sizeof(rr.v[0])); ++q) rr.v[q] = rec[gi].v[q];
#pragma unroll
    for (int q = 0; q < D; ++q) S.x[r][q] = rr.v[q];
    s_trow[r * kThreads + threadIdx.x] = glb(rq.t)[gi < kp.n ? gi : kp.n - 1];   // own slots: no barrier
    S.first[r] = first[gi];
#pragma unroll
    for (int q = 0; q < 6; ++q) { S.a[r][q] = Real(0); S.acc[r][q] = 0.0; }
  }
  TileStage<Rec, kThreads> stage;
  stage.load(rec, tile0);
  for (int tile = tile0; tile < tile1; ++tile) {
    const int buf = (tile - tile0) & 1;
    stage.store(&s_rec[buf][0]);
    stage.store(&s_rec[buf][kTile]);
    __syncthreads();
    if (tile + 1 < tile1) stage.load(rec, tile + 1);
    double* acc_w = s_acc + (buf * kWaves + wave) * NQ * kTile;
    // column sums of the previous tile
    if (tile > tile0)
      store_columns<1, NQ, false>(s_acc + (buf ^ 1) * kWaves * NQ * kTile, pcol, kp, band, tile - 1);
    const bool full = !partial_band && (tile + 1) * kTile <= first_min;
    // the wave's float64 column slots start at zero (a culled tile adds
    // exactly zero and leaves them so)
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc_w[q * kTile + lane] = 0.0;
    // row times relative to this column tile's first event
    const double t_tile = tile_origin(rq.t, tile);
#pragma unroll
    for (int r = 0; r < R; ++r) S.t[r] = (float)((s_trow[r * kThreads + threadIdx.x] - t_tile) * kp.inv_tt);
    // terms that can be nonzero (with none, the tile's column sums stay zero)
    const int terms = CULL ? tile_terms<D, true>((float)((t_row0 - t_tile) * kp.inv_tt), &s_rec[buf][0], tile, kp) : kBothTerms;
    if (terms == 0) {
    } else if (!full) {
      pass1_tile_mixed<D, true, RU, kBothTerms>(S, s_rec[buf], acc_w, tile * kTile, kp);
    } else if (terms == kBothTerms) {
      pass1_tile_mixed<D, false, RU, kBothTerms>(S, s_rec[buf], acc_w, tile * kTile, kp);
    } else if constexpr (CULL) {
      if (terms == kSe)
        pass1_tile_mixed<D, false, RU, kSe>(S, s_rec[buf], acc_w, tile * kTile, kp);
      else
        pass1_tile_mixed<D, false, RU, kBg>(S, s_rec[buf], acc_w, tile * kTile, kp);
    }
  }
  __syncthreads();
  store_columns<1, NQ, false>(s_acc + ((tile1 - 1 - tile0) & 1) * kWaves * NQ * kTile, pcol, kp, band, tile1 - 1);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int lr = wave * 64 * R + r * 64 + lane;
#pragma unroll
    for (int q = 0; q < QR; ++q) {
      const int src = RU || q == 0 ? q : q + 2;   // without RU: K, J, V, W
      glb(static_cast<double*>(rq.prow))[((int64_t)item * QR + q) * kBandRows + lr] = S.acc[r][src];
    }
  }
}

template <int D, bool MASK, int TERMS>
__device__ __forceinline__ void pass2_tile_mixed(Pass2Rows<D, true>& S, const typename Traits<D, true>::Rec* __restrict__ cols,
                                                 double* __restrict__ acc_w, int tile_base, const KParams& kp) {
  constexpr int R = kRowsPerLane;
  const int lane = threadIdx.x & 63;
  const float mW = in_vgpr(kp.mW), mG = in_vgpr(kp.mG), sh = in_vgpr(kp.S);
  const typename Traits<D, true>::Rec* __restrict__ my = cols + lane;
  // exponents of kGradExpSteps steps first, exps back to back, then the
  // steps in order (as in the rate pass)
  constexpr int KS = kGradExpSteps;
  static_assert(kColSteps % KS == 0, "exp groups must not straddle a flush");
  constexpr int UO = HK_GRAD_UNROLL >= kRowFold ? HK_GRAD_UNROLL / kRowFold : 1;
  constexpr int UC = HK_GRAD_UNROLL >= kRowFold ? kRowFold / kColSteps : 1;
#pragma unroll UO
  for (int k2 = 0; k2 < 64; k2 += kRowFold) {
#pragma unroll UC
  for (int kc = 0; kc < kRowFold; kc += kColSteps) {
    const int k1 = k2 + kc;
    float ag[D];
#pragma unroll
    for (int q = 0; q < D; ++q) ag[q] = 0.f;
#pragma unroll
    for (int kk = 0; kk < kColSteps; kk += KS) {
      const int k0 = k1 + kk;
      float dx[KS][R][D], r2[KS][R], dt[KS][R], eb[KS][R], es[KS][R], pbj[KS];
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const auto col = my[k0 + s];
        pbj[s] = col.v[D + 1];
#pragma unroll
        for (int r = 0; r < R; ++r) {
#pragma unroll
          for (int q = 0; q < D; ++q) {
            dx[s][r][q] = S.x[r][q] - col.v[q];
            r2[s][r] = q == 0 ? dx[s][r][q] * dx[s][r][q] : dx[s][r][q] * dx[s][r][q] + r2[s][r];
          }
          dt[s][r] = S.t[r] - col.v[D];
          const bool act = !MASK || (tile_base + ((lane + k0 + s) & 63)) < S.first[r];
          const float zb = __builtin_fmaf(-kHalfLog2e, dt[s][r] * dt[s][r], __builtin_fmaf(-kHalfLog2e, r2[s][r], sh));
          const float zs = __builtin_fmaf(-mW, dt[s][r], __builtin_fmaf(-mG, r2[s][r], sh));
          eb[s][r] = act ? zb : kNoPair;
          es[s][r] = act ? zs : kNoPair;
        }
      }
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if (TERMS & kBg) eb[s][r] = __builtin_amdgcn_exp2f(eb[s][r]);
          if (TERMS & kSe) es[s][r] = __builtin_amdgcn_exp2f(es[s][r]);
        }
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        float cgr[D];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const float ebr = eb[s][r], esr = es[s][r];
          // background weight of the pair with both endpoints' 1/lambda; its
          // r^2 and dt^2 moments give the rate pass's R and U terms of the
          // tau_x and tau_t gradients
          float coef;
          if (TERMS & kBg) {
            const float wb = ebr * (S.pb[r] + pbj[s]);
            coef = TERMS & kSe ? esr * S.ps[r] + wb : wb;
            S.mom[0] = wb * r2[s][r] + S.mom[0];
            S.mom[1] = wb * (dt[s][r] * dt[s][r]) + S.mom[1];
          } else {
            coef = esr * S.ps[r];
          }
#pragma unroll
          for (int q = 0; q < D; ++q) {
            S.g[r][q] = -coef * dx[s][r][q] + S.g[r][q];
            cgr[q] = r == 0 ? coef * dx[s][r][q] : coef * dx[s][r][q] + cgr[q];
          }
        }
#pragma unroll
        for (int q = 0; q < D; ++q) ag[q] = rol1(ag[q]) + cgr[q];
      }
    }
    // column flush: this lane now holds column (lane + k1 + kColSteps - 1) mod 64
    const int c = (lane + k1 + kColSteps - 1) & 63;
#pragma unroll
    for (int q = 0; q < D; ++q) atomicAdd(&acc_w[q * 64 + c], (double)ag[q]);
    // the moments hold 2 rows x kColSteps terms: fold them at every flush
    if (TERMS & kBg) {
      S.momd[0] += (double)S.mom[0];
      S.momd[1] += (double)S.mom[1];
      S.mom[0] = S.mom[1] = 0.f;
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int q = 0; q < D; ++q) { S.acc[r][q] += (double)S.g[r][q]; S.g[r][q] = 0.f; }
  }
}

template <int D, bool CULL>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(grad_waves(D)))) k_pass2_mixed(const ReqDesc* __restrict__ reqs, int nreq, int ev_blocks) {
  using Rec = typename Traits<D, true>::Rec;
  using Real = float;
  constexpr int R = kRowsPerLane;
  constexpr int NQ = D;
  using Lds = PassLds<1, NQ>;
  __shared__ Rec s_rec[2][2 * kTile];
  __shared__ double s_trow[R * kThreads];   // the rows' event times
  __shared__ double s_acc[Lds::kDoubles];
  __shared__ double s_red[2 * kWaves];
  // the fix-up and finalize blocks come first (their results are read by the
  // next kernel only); nothing in the pair pass depends on them
  const int blk = (int)blockIdx.x - side_blocks(nreq, ev_blocks);
  if (blk < 0) {
    side_block<D, true>(reqs, nreq, ev_blocks, kFixGrid, s_acc);
    return;
  }
  const int rid = find_req(reqs, nreq, blk, 0);
  const ReqDesc& rq = reqs[rid];
  const KParams& kp = rq.kp;
  const auto rec = glb(static_cast<const Rec*>(rq.rec));
  const auto first = glb(rq.first);
  const auto pcol = glb(static_cast<double*>(rq.pcol));
  const int item = blk - rq.blk_items;
  const int band = uni(glb(rq.items)[item].x), chunk = uni(glb(rq.items)[item].y);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int row_base = band * kBandRows;
  const int row_end = min(kp.n, row_base + kBandRows);
  const int nt_band = (row_end + kTile - 1) / kTile;
  const int Lb = item_tiles(band, kp.b_fine, kp.L);
  const int tile0 = chunk * Lb;
  const int tile1 = min(tile0 + Lb, nt_band);
  const bool partial_band = row_base + kBandRows > kp.n;
  const int first_min = uni(first[row_base]);
  const double t_row0 = CULL ? glb(rq.t)[row_base] : 0.0;   // the band's first row

  Pass2Rows<D, true> S;
  S.mom[0] = S.mom[1] = 0.f;
  S.momd[0] = S.momd[1] = 0.0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int gi = row_base + wave * 64 * R + r * 64 + lane;
    Rec rr;
#pragma unroll
    for (int q = 0; q < (int)(sizeof(Rec) / sizeof(rr.v[0])); ++q) rr.v[q] = rec[gi].v[q];
#pragma unroll
    for (int q = 0; q < D; ++q) { S.x[r][q] = rr.v[q]; S.g[r][q] = Real(0); S.acc[r][q] = 0.0; }
    s_trow[r * kThreads + threadIdx.x] = glb(rq.t)[gi < kp.n ? gi : kp.n - 1];   // own slots: no barrier
    S.pb[r] = rr.v[D + 1];
    S.ps[r] = glb(static_cast<const Real*>(rq.ps))[gi];
    S.first[r] = first[gi];
  }
  TileStage<Rec, kThreads> stage;
  stage.load(rec, tile0);
  for (int tile = tile0; tile < tile1; ++tile) {
    const int buf = (tile - tile0) & 1;
    stage.store(&s_rec[buf][0]);
    stage.store(&s_rec[buf][kTile]);
    __syncthreads();
    if (tile + 1 < tile1) stage.load(rec, tile + 1);
    double* acc_w = s_acc + (buf * kWaves + wave) * NQ * kTile;
    // column sums of the previous tile
    if (tile > tile0)
      store_columns<1, NQ, false>(s_acc + (buf ^ 1) * kWaves * NQ * kTile, pcol, kp, band, tile - 1);
    const bool full = !partial_band && (tile + 1) * kTile <= first_min;
    // the wave's float64 column slots start at zero (a culled tile adds
    // exactly zero and leaves them so)
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc_w[q * kTile + lane] = 0.0;
    // row times relative to this column tile's first event
    const double t_tile = tile_origin(rq.t, tile);
#pragma unroll
    for (int r = 0; r < R; ++r) S.t[r] = (float)((s_trow[r * kThreads + threadIdx.x] - t_tile) * kp.inv_tt);
    // terms that can be nonzero (with none, the tile's column sums stay zero)
    const int terms = CULL ? tile_terms<D, true>((float)((t_row0 - t_tile) * kp.inv_tt), &s_rec[buf][0], tile, kp) : kBothTerms;
    if (terms == 0) {
    } else if (!full) {
      pass2_tile_mixed<D, true, kBothTerms>(S, s_rec[buf], acc_w, tile * kTile, kp);
    } else if (terms == kBothTerms) {
      pass2_tile_mixed<D, false, kBothTerms>(S, s_rec[buf], acc_w, tile * kTile, kp);
    } else if constexpr (CULL) {
      if (terms == kSe)
        pass2_tile_mixed<D, false, kSe>(S, s_rec[buf], acc_w, tile * kTile, kp);
      else
        pass2_tile_mixed<D, false, kBg>(S, s_rec[buf], acc_w, tile * kTile, kp);
    }
  }
  __syncthreads();
  store_columns<1, NQ, false>(s_acc + ((tile1 - 1 - tile0) & 1) * kWaves * NQ * kTile, pcol, kp, band, tile1 - 1);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int lr = wave * 64 * R + r * 64 + lane;
#pragma unroll
    for (int q = 0; q < D; ++q)
      glb(static_cast<double*>(rq.prow))[((int64_t)item * D + q) * kBandRows + lr] = S.acc[r][q];
  }
  // the item's two moment sums, fixed-order over the workgroup
  double mom[2] = {S.momd[0], S.momd[1]};
  group_sum(mom, s_red);
  if (threadIdx.x == 0) {
    glb(rq.mompart)[(int64_t)item * 2 + 0] = mom[0];
    glb(rq.mompart)[(int64_t)item * 2 + 1] = mom[1];
  }
}

// ------------------------------------------------------------ reductions

// Per event: fixed-order sum of the row partials (this band's items) and the
// column partials (bands from this one to the last), conversion to the raw
// sums K, R, U, J, V, W (times exp(sigma)), the recompute flag, and the
// pass-2 factors (1/lambda scaled to the main pass's terms; 0 for flagged rows,
// whose pairs the float64 fix-ups take).  Pass 2 needs nothing later than this
// kernel, so it can run while the fix-ups and the finalize kernels do.
//
// A workgroup takes kRedEv consecutive events (one band, since kRedEv divides
// kBandRows), one per lane, in each of kRedWaves waves: wave w sums the items
// c = w, w + kRedWaves, ... and the bands I = b + w, b + w + kRedWaves, ..., so
// every load instruction reads one contiguous row of kRedEv float64 partials;
// the waves' sums meet in LDS and wave 0 adds them in wave order (a fixed
// order: results do not depend on timing).  Flagged rows of each workgroup are
// staged in index order for fix_rows.

static_assert(kRedEv == 64 && kBandRows % kRedEv == 0, "a reduction workgroup is one wave of events inside one band");

template <int D, bool MIX>
__global__ void __launch_bounds__(kRedThreads) k_reduce1(const ReqDesc* __restrict__ reqs, int nreq) {
  using ColT = double;   // partials are float64 in both precisions
  using Real = typename Traits<D, MIX>::Real;
  using Rec = typename Traits<D, MIX>::Rec;
  __shared__ double s_part[kRedWaves][6][kRedEv];
  const int rid = find_req(reqs, nreq, blockIdx.x, 3);
  const ReqDesc& rq = reqs[rid];
  const KParams& kp = rq.kp;
  const int lb = blockIdx.x - rq.blk_red;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (lb == 0) {   // the request's first workgroup joins the data checks
    int bad = 0;
    for (int k = threadIdx.x; k < kp.n_pad / kEvBlock; k += kRedThreads) bad |= glb(rq.bad)[k];
    bad = __syncthreads_or(bad);
    if (threadIdx.x == 0) glb(rq.status)[kStData] = bad != 0 ? 1 : 0;
  }
  const int i0 = lb * kRedEv;
  const int i = i0 + lane;   // >= n only in the last band's padding (read, never written)
  const int b = i0 / kBandRows, lr = i % kBandRows;
  const IPair bi{band_first_item(kp, b), band_items(kp, b)};
  const auto prow = glb(static_cast<const ColT*>(rq.prow));
  const auto pcol = glb(static_cast<const ColT*>(rq.pcol));
  double s[6] = {0, 0, 0, 0, 0, 0};
  if (kp.ru1) {
#pragma unroll 2
    for (int c = wave; c < bi.y; c += kRedWaves) {
      const auto p = prow + (int64_t)(bi.x + c) * 6 * kBandRows + lr;
#pragma unroll
      for (int q = 0; q < 6; ++q) s[q] += p[(int64_t)q * kBandRows];
    }
#pragma unroll 2
    for (int I = b + wave; I < kp.nb; I += kRedWaves) {
      const auto p = pcol + (int64_t)I * 3 * kp.n_pad + i;
#pragma unroll
      for (int q = 0; q < 3; ++q) s[q] += p[(int64_t)q * kp.n_pad];
    }
  } else {
    // rate pass without the background moments: rows K, J, V, W, column K
#pragma unroll 2
    for (int c = wave; c < bi.y; c += kRedWaves) {
      const auto p = prow + (int64_t)(bi.x + c) * 4 * kBandRows + lr;
      s[0] += p[0];
#pragma unroll
      for (int q = 1; q < 4; ++q) s[q + 2] += p[(int64_t)q * kBandRows];
    }
#pragma unroll 4
    for (int I = b + wave; I < kp.nb; I += kRedWaves) s[0] += pcol[(int64_t)I * kp.n_pad + i];
  }
#pragma unroll
  for (int q = 0; q < 6; ++q) s_part[wave][q][lane] = s[q];
  __syncthreads();
  if (wave != 0) return;
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    double v = s_part[0][q][lane];
#pragma unroll
    for (int w = 1; w < kRedWaves; ++w) v += s_part[w][q][lane];
    s[q] = v;
  }
  bool flag = false;
  if (i < kp.n) {
    if (MIX) {   // moments were accumulated in bandwidth units
      s[1] *= kp.tau_x * kp.tau_x;
      s[2] *= kp.tau_t * kp.tau_t;
      s[4] *= kp.tau_x * kp.tau_x;
      s[5] *= kp.tau_t;
    }
    const double lam = kp.cbg * s[0] + kp.cse * s[3];
    flag = !(lam >= kp.cmax * exp2(kp.flag_floor));
#pragma unroll
    for (int q = 0; q < 6; ++q) glb(rq.sums)[(int64_t)i * 6 + q] = s[q];
    glb(rq.flags)[i] = flag ? 1 : 0;
    // mixed: coordinates are in units of tau_x, so one factor tau_x moves in
    const double il = flag ? 0.0 : 1.0 / lam;
    const double pb = MIX ? kp.cbg * kp.inv_tx * il : kp.cbg * kp.itx2 * il;
    const double ps = MIX ? kp.cse * kp.tau_x * kp.ih2 * il : kp.cse * kp.ih2 * il;
    glb(static_cast<Rec*>(rq.rec))[i].v[D + 1] = (Real)pb;
    glb(static_cast<Real*>(rq.ps))[i] = (Real)ps;
  }
  // stage this workgroup's flagged rows in index order (one wave ballot)
  const unsigned long long m = __ballot(flag);
  if (flag) glb(rq.bstage)[(int64_t)lb * kRedEv + __popcll(m & ((1ull << lane) - 1ull))] = i;
  if (lane == 0) glb(rq.bcount)[lb] = __popcll(m);
}

// ell, the six parameter gradients and the status of one request: the
// finalize blocks' sums, the flagged rows' terms and (gradient calls) the
// gradient pass's two moment sums, all in a fixed order.
// out8 = [ell, 6 gradients, status].  kRedThreads threads.
template <int D, bool MIX, bool GRAD>
__device__ __forceinline__ void final_block(const ReqDesc& rq, double* pool) {
  const KParams& kp = rq.kp;
  const int tid = threadIdx.x;
  const bool bad = uni(glb(rq.status)[kStData]) != 0;
  double v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  double mom[2] = {0, 0};
  if (!bad) {
    for (int b = tid; b < kp.nblk; b += kRedThreads)
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] += glb(rq.bpart)[(int64_t)b * 8 + q];
    if (!kp.ru1) {
      // the background moments' terms of d ell/d tau_x and d ell/d tau_t, from
      // the gradient pass's item sums: sum over pairs of
      // w r'^2 = sum_n c_bg R_n / (tau_x^3 lambda_n) and w dt'^2 tau_x / tau_t =
      // sum_n c_bg U_n / (tau_t^3 lambda_n) over the unflagged rows (flagged
      // rows carry their exact R and U from the fix-up instead)
      for (int it = tid; it < kp.items; it += kRedThreads) {
        mom[0] += glb(rq.mompart)[(int64_t)it * 2 + 0];
        mom[1] += glb(rq.mompart)[(int64_t)it * 2 + 1];
      }
    }
    const int cnt = glb(rq.status)[kStFlagCount];
    const int segs = GRAD ? 1 : fix_segs(cnt, kp);
    for (int f = tid; f < cnt; f += kRedThreads) {
      double s[6], scale;
      if constexpr (GRAD) {
        const auto fp = glb(rq.fixpart) + (int64_t)f * kFixStride;
#pragma unroll
        for (int q = 0; q < 6; ++q) s[q] = fp[q];
        scale = fp[6];
      } else {
        const auto fp = glb(rq.fixpart) + (int64_t)f * segs * kFixSegStride;
        double m = -INFINITY;
        for (int g = 0; g < segs; ++g) m = fmax(m, fp[g * kFixSegStride + 6]);
#pragma unroll
        for (int q = 0; q < 6; ++q) s[q] = 0.0;
        for (int g = 0; g < segs && m > -INFINITY; ++g) {
          const double mg = fp[g * kFixSegStride + 6];
          if (!(mg > -INFINITY)) continue;
          const double w = exp(mg - m);
#pragma unroll
          for (int q = 0; q < 6; ++q) s[q] += fp[g * kFixSegStride + q] * w;
        }
        scale = m > -INFINITY ? m : 0.0;
      }
      const double lt = rate_terms<D>(kp, s, scale, v);
      store_terms(rq, glb(rq.list)[f], s, lt, scale);
    }
  }
  // mixed sums are in bandwidth units and carry 1/tau_x, float64 ones 1/tau_x^2
  v[2] += MIX ? mom[0] : mom[0] / kp.tau_x;
  v[3] += MIX ? mom[1] * kp.tau_x / kp.tau_t : mom[1] * (kp.tau_x * kp.tau_x / (kp.tau_t * kp.tau_t * kp.tau_t));
  group_sum(v, pool);
  if (tid == 0) {
    double o[8];
    if (bad || v[7] > 0.0) {
      o[0] = bad ? NAN : -INFINITY;
      for (int q = 1; q < 7; ++q) o[q] = NAN;
      o[7] = bad ? -3.0 : -4.0;   // HAWKES_EDATA, HAWKES_EZERORATE
    } else {
      for (int q = 0; q < 7; ++q) o[q] = v[q];
      o[7] = 0.0;
    }
    for (int q = 0; q < 8; ++q) {
      glb(rq.out8)[q] = o[q];
      if (rq.out_host) rq.out_host[q] = o[q];
    }
  }
}

template <int D, bool MIX>
__global__ void __launch_bounds__(kRedThreads) k_final(const ReqDesc* __restrict__ reqs) {
  __shared__ double s_pool[kRedWaves * 8];
  final_block<D, MIX, false>(reqs[blockIdx.x], s_pool);
}

// grad_x = row partials + column partials + fix-up terms, in a fixed order
// (workgroups, waves and the LDS meeting as in k_reduce1); the first nreq
// workgroups take final_block instead.
//
// Fix-up terms.  For a flagged row j and any event i the j-side coefficient
// c = mu_ij/(lambda_j tau_x^2) + [t_i < t_j] xi_ji/(lambda_j h^2) is formed in
// float64 as exp(log-term - log lambda_j): every event adds c (x_j - x_i) over
// the flagged rows (kFixChunk at a time in LDS, every kRedWaves-th of them per
// wave), and a flagged row adds its own vector.
constexpr int kFixChunk = 256;

template <int D, bool MIX>
__global__ void __launch_bounds__(kRedThreads) k_reduce2(const ReqDesc* __restrict__ reqs, int nreq) {
  constexpr int kMeet = kRedWaves * D * kRedEv, kFlagged = kFixChunk * (D + 2);
  __shared__ double s_pool[kMeet > kFlagged ? kMeet : kFlagged];
  if ((int)blockIdx.x < nreq) {
    final_block<D, MIX, true>(reqs[blockIdx.x], s_pool);
    return;
  }
  const int blk = blockIdx.x - nreq;
  const ReqDesc& rq = reqs[find_req(reqs, nreq, blk, 3)];
  const KParams& kp = rq.kp;
  if (uni(glb(rq.status)[kStData]) != 0 || rq.grad_x == nullptr) return;
  const int lb = blk - rq.blk_red;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i0 = lb * kRedEv;
  const int i = i0 + lane;   // >= n only in the last band's padding (read, never written)
  const int cnt = uni(glb(rq.status)[kStFlagCount]);
  const int b = i0 / kBandRows, lr = i % kBandRows;
  const IPair bi{band_first_item(kp, b), band_items(kp, b)};
  const auto prow = glb(static_cast<const double*>(rq.prow));
  const auto pcol = glb(static_cast<const double*>(rq.pcol));
  double s[D];
#pragma unroll
  for (int q = 0; q < D; ++q) s[q] = 0.0;
#pragma unroll 2
  for (int c = wave; c < bi.y; c += kRedWaves) {
    const auto p = prow + (int64_t)(bi.x + c) * D * kBandRows + lr;
#pragma unroll
    for (int q = 0; q < D; ++q) s[q] += p[(int64_t)q * kBandRows];
  }
#pragma unroll 2
  for (int I = b + wave; I < kp.nb; I += kRedWaves) {
    const auto p = pcol + (int64_t)I * D * kp.n_pad + i;
#pragma unroll
    for (int q = 0; q < D; ++q) s[q] += p[(int64_t)q * kp.n_pad];
  }
  int zero = 0;
  if (cnt > 0) {
    const int ic = min(i, kp.n - 1);
    double xi[D];
#pragma unroll
    for (int q = 0; q < D; ++q) xi[q] = glb(rq.x)[(int64_t)ic * D + q];
    const double ti = glb(rq.t)[ic];
    for (int f0 = 0; f0 < cnt; f0 += kFixChunk) {
      const int fn = min(kFixChunk, cnt - f0);
      __syncthreads();
      for (int e = threadIdx.x; e < fn * (D + 2); e += kRedThreads) {
        const double v = glb(rq.fixpart)[(int64_t)(f0 + e / (D + 2)) * kFixStride + 7 + e % (D + 2)];
        if (e % (D + 2) == 0) zero |= v > -INFINITY ? 0 : 1;
        s_pool[e] = v;   // log lambda_j, t_j, x_j
      }
      __syncthreads();
      for (int k = wave; k < fn; k += kRedWaves) {
        const double* e = s_pool + k * (D + 2);
        double dx[D], r2 = 0;
#pragma unroll
        for (int q = 0; q < D; ++q) { dx[q] = e[2 + q] - xi[q]; r2 += dx[q] * dx[q]; }
        const double dt = e[1] - ti;   // > 0 when the flagged row is the later event
        const double Lj = e[0];
        double c = 0.0;   // the pair of a row with itself has dt = 0
        if (dt != 0.0) c += exp(kp.log_cbg - kp.alpha * r2 - kp.beta * dt * dt - Lj) * kp.itx2;
        if (dt > 0.0) c += exp(kp.log_cse - kp.omega * dt - kp.gamma * r2 - Lj) * kp.ih2;
#pragma unroll
        for (int q = 0; q < D; ++q) s[q] += c * dx[q];
      }
    }
    zero = __syncthreads_or(zero);
  }
  double* s_part = s_pool;   // [wave][q][event]
#pragma unroll
  for (int q = 0; q < D; ++q) s_part[(wave * D + q) * kRedEv + lane] = s[q];
  __syncthreads();
  if (wave != 0 || i >= kp.n) return;
#pragma unroll
  for (int q = 0; q < D; ++q) {
    double v = s_part[q * kRedEv + lane];
#pragma unroll
    for (int w = 1; w < kRedWaves; ++w) v += s_part[(w * D + q) * kRedEv + lane];
    s[q] = v;
  }
  if (cnt > 0 && glb(rq.flags)[i] != 0) {
#pragma unroll
    for (int q = 0; q < D; ++q) s[q] += glb(rq.fixpart)[(int64_t)glb(rq.listpos)[i] * kFixStride + 17 + q];
  }
#pragma unroll
  for (int q = 0; q < D; ++q) glb(rq.grad_x)[(int64_t)i * D + q] = zero ? NAN : s[q];   // NaN: some rate is zero
}

}  // namespace hawkes
