// libhawkes: the launch sequence of one batch and its kernels, for the one
// dimension HK_D (this file is compiled once per dimension, so that the
// dimensions' kernels build in parallel).
#include <hip/hip_runtime.h>

#include "hawkes_internal.hpp"
#include "hawkes_kernels.hpp"

#ifndef HK_D
#error "compile with -DHK_D=<dimension>"
#endif

namespace hawkes {

// The phases over every request of a batch (all with the same D, precision and
// step groups).  reqs: device array of descriptors; g: grid sizes.
// one != nullptr: a single request whose descriptor the first kernel writes
// to reqs[0].
template <int D, bool MIX, int SP, bool CULL>
static bool launch_phases(const ReqDesc* reqs, int nreq, const BatchGrid& g, bool grad, hipStream_t s,
                          const ReqDesc* one) {
  mark_stage(s, 0);
  if (one) k_prep_one<D, MIX><<<g.pad_blocks, kEvBlock, 0, s>>>(*one, const_cast<ReqDesc*>(reqs));
  else k_prep<D, MIX><<<g.pad_blocks, kEvBlock, 0, s>>>(reqs, nreq);
  mark_stage(s, 1);
  mark_stage(s, 2);
  if constexpr (MIX) {
    if (grad) k_pass1_mixed<D, false, CULL><<<g.items, kThreads, 0, s>>>(reqs, nreq);
    else k_pass1_mixed<D, true, CULL><<<g.items, kThreads, 0, s>>>(reqs, nreq);
  } else {
    if (grad) k_pass1<D, false, SP, CULL><<<g.items, SP * kThreads, 0, s>>>(reqs, nreq);
    else k_pass1<D, true, SP, CULL><<<g.items, SP * kThreads, 0, s>>>(reqs, nreq);
  }
  mark_stage(s, 3);
  k_reduce1<D, MIX><<<g.red_blocks, kRedThreads, 0, s>>>(reqs, nreq);
  mark_stage(s, 4);
  const int side = side_blocks(nreq, g.ev_blocks);
  if (!grad) {
    k_side<D><<<g.ev_blocks + nreq * fix_grid(g.ev_blocks / nreq), kEvBlock, 0, s>>>(reqs, nreq, g.ev_blocks);
    for (int k = 5; k <= 7; ++k) mark_stage(s, k);
    k_final<D, MIX><<<nreq, kRedThreads, 0, s>>>(reqs);
    mark_stage(s, 8);
    return true;
  }
  mark_stage(s, 5);
  mark_stage(s, 6);
  if constexpr (MIX) k_pass2_mixed<D, CULL><<<side + g.items, kThreads, 0, s>>>(reqs, nreq, g.ev_blocks);
  else k_pass2<D, SP, CULL><<<side + g.items, SP * kThreads, 0, s>>>(reqs, nreq, g.ev_blocks);
  mark_stage(s, 7);
  mark_stage(s, 8);
  k_reduce2<D, MIX><<<nreq + g.red_blocks, kRedThreads, 0, s>>>(reqs, nreq);
  mark_stage(s, 9);
  return true;
}

template <int D, bool CULL>
static bool launch_cull(int mixed, int split, const ReqDesc* reqs, int nreq, const BatchGrid& g, bool grad,
                        hipStream_t s, const ReqDesc* one) {
  if (mixed) return launch_phases<D, true, 1, CULL>(reqs, nreq, g, grad, s, one);
  if constexpr (D <= kMaxSplitD)
    if (split == 2) return launch_phases<D, false, 2, CULL>(reqs, nreq, g, grad, s, one);
  return split == 1 && launch_phases<D, false, 1, CULL>(reqs, nreq, g, grad, s, one);
}

template <int D>
bool launch_d(int mixed, int cull, int split, const ReqDesc* reqs, int nreq, const BatchGrid& g, bool grad,
              hipStream_t s, const ReqDesc* one) {
  return cull ? launch_cull<D, true>(mixed, split, reqs, nreq, g, grad, s, one)
              : launch_cull<D, false>(mixed, split, reqs, nreq, g, grad, s, one);
}
template bool launch_d<HK_D>(int, int, int, const ReqDesc*, int, const BatchGrid&, bool, hipStream_t, const ReqDesc*);

}  // namespace hawkes
