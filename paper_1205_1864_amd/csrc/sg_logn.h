// Block solve of the lognormal path in one launch (k_logn.hip), shared by its
// host driver and kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace sgk {

struct LognSolveArgs {
  const int *rptr, *rcol;  // stored blocks of every chaos row, ascending columns, numbered in this order
  const double* C;
  const double* Dinv;
  int n_e, P;
  int lo, nr;      // chaos columns of the sub-block
  const double* B;
  double* X;
  long stride;     // from one system's B and X to the next
  int G, lpr, rows;  // blocks per system, lanes per operator row, rows per block (set by the launch)
  double rtol;
  int maxit;
  unsigned long long* ex;   // exchange, 3 n nr places (systems of several blocks)
  int *first, *last;        // [P] stored blocks of the sub-block per chaos row
  unsigned long long* its;  // CG iterations, added to
  unsigned long long* status;  // set if a bounded wait expired
  unsigned long long* told;    // the same in host memory
  long spins;               // polls of an exchange before a wait expires
};

// CG on `nsys` systems (see logn_solve_kernel) from X = 0; *done = false if the
// system does not fit the kernel, and nothing was launched.
hipError_t launch_logn_solve(const LognSolveArgs& args, int nsys, hipStream_t s, bool* done);

}  // namespace sgk
