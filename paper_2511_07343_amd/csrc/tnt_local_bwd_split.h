// Pointers and sizes shared by the three backward passes of the fixed-size local kernels.
#pragma once

#include "tnt_kernels.h"
#include "tnt_local_record.h"

namespace tnt {

// Compute units whose workgroups the walk of the adjoint may count on to be resident
// together (one workgroup per CU): the size of its grid where slices exchange data.
constexpr int WALK_CUS = 256;
// its workgroups draw their roles from this many counters, each in a line of its own
constexpr int WALK_LANES = 8, TICKET_STRIDE = 32;
constexpr int WALK_TICKETS = 2 * WALK_LANES * TICKET_STRIDE;

struct SplitPtrs {
  void* brec;               // CT   [units * nch][r.bc.n]  backward records
  float* brec_f;            // fp32 [units * nch][r.bf.n]
  float* dks;               // fp32 [units * nch][slices][Cp * d]  the walk's part of dk, per slice
  unsigned long long* xch;  // [groups][2][slices][Cp * d]  the slices' partial Rbar: value (low
                            // half) and tag (high half)
  unsigned* tickets;        // [2][WALK_LANES] of a cache line each: workgroups started, by the walk of
                            // the last chunks and of the others
  int units;
  int n0, nc;               // passes A and B: the chunks n0 .. n0 + nc - 1 of every unit
  int groups;               // walk: groups of `slices` workgroups, unit u on group u % groups
};

// the walk of the carried adjoint (pass B); false: not built for these sizes
bool launch_local_bwd_walk(const LocalBwdArgs& a, const SplitPtrs& P, hipStream_t st, hipError_t* err);

}  // namespace tnt
