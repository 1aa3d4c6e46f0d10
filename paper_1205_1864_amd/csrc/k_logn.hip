// Kernels of the lognormal-coefficient SG operator (Section 6, second set of
// experiments): the coefficient is expanded in Hermite chaos to twice the
// solution's degree, so every chaos block couples and the operator is
//   Y_a = sum_b K(c_ab) U_b,  c_ab(e) = sum_i E[psi_i psi_a psi_b] k_i(e),
// with K(c) the Q1 stiffness of the element field c (eq. (global-matrix-block)).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "sg_device.h"
#include "sg_internal.h"
#include "sg_logn.h"

namespace sgk {

// c_ab(e) for every stored block: one thread per (element, block slot),
// summing the block's (term, triple product) list in a fixed order.
__global__ void __launch_bounds__(256) logn_blocks_kernel(const long* __restrict__ ptr, const int* __restrict__ term,
                                                          const double* __restrict__ g,
                                                          const double* __restrict__ kc, int ne2, int nslots,
                                                          double* __restrict__ C) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= ne2) return;
  for (int s = blockIdx.y; s < nslots; s += gridDim.y) {
    double acc = 0.0;
    for (long j = ptr[s]; j < ptr[s + 1]; ++j) acc += g[j] * kc[(long)term[j] * ne2 + e];
    C[(long)s * ne2 + e] = acc;
  }
}

// Y[:, a] = sum over the stored blocks (a, b) of K(c_ab) U[:, b]: one thread
// per (interior node, chaos row a). The Q1 element matrix of the unit
// coefficient is (4 on the diagonal, -1 along an edge, -2 across) / 6; nodes
// on the boundary carry zero. The node's 3 x 3 neighbourhood offsets and
// boundary masks are fixed per thread, so every load of a block is
// unconditional (a neighbour off the grid reads the node itself, masked to 0).
__global__ void __launch_bounds__(256) logn_matvec_kernel(const int* __restrict__ rptr, const int* __restrict__ rcol,
                                                          const int* __restrict__ rslot,
                                                          const double* __restrict__ C,
                                                          const double* __restrict__ U, int n_e, long n,
                                                          double* __restrict__ Y) {
  const long xi = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const int a = blockIdx.y;
  if (xi >= n) return;
  const int nx = n_e - 1;
  const int ix = (int)(xi % nx) + 1, iy = (int)(xi / nx) + 1;  // grid node, 1..n_e-1
  const long ne2 = (long)n_e * n_e;
  long off[3][3];
  double msk[3][3];
#pragma unroll
  for (int dy = 0; dy < 3; ++dy)
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) {
      const int gx = ix + dx - 1, gy = iy + dy - 1;
      const bool in = gx >= 1 && gx <= nx && gy >= 1 && gy <= nx;
      off[dy][dx] = in ? (long)(gy - 1) * nx + (gx - 1) : xi;
      msk[dy][dx] = in ? 1.0 : 0.0;
    }
  // elements below-left, below-right, above-left, above-right of the node
  const long e00 = (long)(iy - 1) * n_e + (ix - 1);
  double y = 0.0;
  for (int r = rptr[a]; r < rptr[a + 1]; ++r) {
    const double* __restrict__ u = U + (long)rcol[r] * n;
    const double* __restrict__ c = C + (long)rslot[r] * ne2;
    double v[3][3];
#pragma unroll
    for (int dy = 0; dy < 3; ++dy)
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) v[dy][dx] = u[off[dy][dx]] * msk[dy][dx];
    const double c00 = c[e00], c01 = c[e00 + 1], c10 = c[e00 + n_e], c11 = c[e00 + n_e + 1];
    const double uc = 4.0 * v[1][1];
    // element (ey, ex) with the node at one corner: edge neighbours (ox, iy),
    // (ix, oy) and the opposite corner (ox, oy)
    y += c00 * (uc - v[1][0] - v[0][1] - 2.0 * v[0][0]);
    y += c01 * (uc - v[1][2] - v[0][1] - 2.0 * v[0][2]);
    y += c10 * (uc - v[1][0] - v[2][1] - 2.0 * v[2][0]);
    y += c11 * (uc - v[1][2] - v[2][1] - 2.0 * v[2][2]);
  }
  Y[(long)a * n + xi] = y * (1.0 / 6.0);
}

// Sub-block of the operator for the hierarchical preconditioner: rows
// row0..row0+nrows-1 and columns col0..col1-1 of A (eq. (global-matrix-hierarchy)).
// X holds the columns col0.. (ld n); mode 0: Y = A_sub X; mode 1: Y = R - A_sub X
// (R may be Y). Same element form and summation order as logn_matvec_kernel.
__global__ void __launch_bounds__(256) logn_apply_kernel(const int* __restrict__ rptr, const int* __restrict__ rcol,
                                                         const int* __restrict__ rslot,
                                                         const double* __restrict__ C,
                                                         const double* __restrict__ X, int n_e, long n, int row0,
                                                         int col0, int col1, int mode, const double* R, double* Y) {
  const long xi = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const int a = row0 + (int)blockIdx.y;
  if (xi >= n) return;
  const int nx = n_e - 1;
  const int ix = (int)(xi % nx) + 1, iy = (int)(xi / nx) + 1;
  const long ne2 = (long)n_e * n_e;
  long off[3][3];
  double msk[3][3];
#pragma unroll
  for (int dy = 0; dy < 3; ++dy)
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) {
      const int gx = ix + dx - 1, gy = iy + dy - 1;
      const bool in = gx >= 1 && gx <= nx && gy >= 1 && gy <= nx;
      off[dy][dx] = in ? (long)(gy - 1) * nx + (gx - 1) : xi;
      msk[dy][dx] = in ? 1.0 : 0.0;
    }
  const long e00 = (long)(iy - 1) * n_e + (ix - 1);
  double y = 0.0;
  for (int r = rptr[a]; r < rptr[a + 1]; ++r) {
    const int b = rcol[r];
    if (b < col0 || b >= col1) continue;
    const double* __restrict__ u = X + (long)(b - col0) * n;
    const double* __restrict__ c = C + (long)rslot[r] * ne2;
    double v[3][3];
#pragma unroll
    for (int dy = 0; dy < 3; ++dy)
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) v[dy][dx] = u[off[dy][dx]] * msk[dy][dx];
    const double c00 = c[e00], c01 = c[e00 + 1], c10 = c[e00 + n_e], c11 = c[e00 + n_e + 1];
    const double uc = 4.0 * v[1][1];
    y += c00 * (uc - v[1][0] - v[0][1] - 2.0 * v[0][0]);
    y += c01 * (uc - v[1][2] - v[0][1] - 2.0 * v[0][2]);
    y += c10 * (uc - v[1][0] - v[2][1] - 2.0 * v[2][0]);
    y += c11 * (uc - v[1][2] - v[2][1] - 2.0 * v[2][2]);
  }
  y *= (1.0 / 6.0);
  const long o = (long)(a - row0) * n + xi;
  Y[o] = mode ? R[o] - y : y;
}

// Y[:, j] = K(c) X[:, j] for ncols columns with one element field c (the
// mean coefficient: the blocks of the mean-based preconditioner).
__global__ void __launch_bounds__(256) logn_mean_apply_kernel(const double* __restrict__ c,
                                                              const double* __restrict__ X, int n_e, long n,
                                                              double* __restrict__ Y) {
  const long xi = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const int j = blockIdx.y;
  if (xi >= n) return;
  const int nx = n_e - 1;
  const int ix = (int)(xi % nx) + 1, iy = (int)(xi / nx) + 1;
  const double* __restrict__ u = X + (long)j * n;
  double v[3][3];
#pragma unroll
  for (int dy = 0; dy < 3; ++dy)
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) {
      const int gx = ix + dx - 1, gy = iy + dy - 1;
      const bool in = gx >= 1 && gx <= nx && gy >= 1 && gy <= nx;
      v[dy][dx] = u[in ? (long)(gy - 1) * nx + (gx - 1) : xi] * (in ? 1.0 : 0.0);
    }
  const long e00 = (long)(iy - 1) * n_e + (ix - 1);
  const double c00 = c[e00], c01 = c[e00 + 1], c10 = c[e00 + n_e], c11 = c[e00 + n_e + 1];
  const double uc = 4.0 * v[1][1];
  double y = c00 * (uc - v[1][0] - v[0][1] - 2.0 * v[0][0]);
  y += c01 * (uc - v[1][2] - v[0][1] - 2.0 * v[0][2]);
  y += c10 * (uc - v[1][0] - v[2][1] - 2.0 * v[2][0]);
  y += c11 * (uc - v[1][2] - v[2][1] - 2.0 * v[2][2]);
  Y[(long)j * n + xi] = y * (1.0 / 6.0);
}

// Inverse diagonal of A (Jacobi scaling of the level-block solves): the
// (a, a) block's stencil centre, (4/6) times the sum of c_aa over the four
// elements around the node.
__global__ void __launch_bounds__(256) logn_invdiag_kernel(const int* __restrict__ rptr, const int* __restrict__ rcol,
                                                           const int* __restrict__ rslot,
                                                           const double* __restrict__ C, int n_e, long n,
                                                           double* __restrict__ Dinv) {
  const long xi = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const int a = blockIdx.y;
  if (xi >= n) return;
  const int nx = n_e - 1;
  const int ix = (int)(xi % nx) + 1, iy = (int)(xi / nx) + 1;
  const long e00 = (long)(iy - 1) * n_e + (ix - 1);
  double d = 0.0;
  for (int r = rptr[a]; r < rptr[a + 1]; ++r) {
    if (rcol[r] != a) continue;
    const double* c = C + (long)rslot[r] * n_e * n_e;
    d = (4.0 / 6.0) * (c[e00] + c[e00 + 1] + c[e00 + n_e] + c[e00 + n_e + 1]);
  }
  Dinv[(long)a * n + xi] = d > 0.0 ? 1.0 / d : 0.0;
}

// Partial dot products: block b sums a strided range in a fixed order, then a
// fixed LDS tree; the host adds the partials in index order.
__global__ void __launch_bounds__(256) logn_dot_kernel(const double* __restrict__ x, const double* __restrict__ y,
                                                       long len, double* __restrict__ part) {
  __shared__ double sm[256];
  double acc = 0.0;
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < len; i += (long)gridDim.x * blockDim.x)
    acc += x[i] * y[i];
  sm[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sm[threadIdx.x] += sm[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = sm[0];
}

// y = a x + b y (b = 0 overwrites y), or y = d * x elementwise with d of
// period dn (mode 1).
__global__ void __launch_bounds__(256) logn_axpby_kernel(long len, double a, const double* __restrict__ x, double b,
                                                         double* __restrict__ y, int mode,
                                                         const double* __restrict__ d, long dn) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < len; i += (long)gridDim.x * blockDim.x) {
    if (mode == 1) {
      y[i] = d[i % dn] * x[i];
    } else {
      y[i] = b == 0.0 ? a * x[i] : a * x[i] + b * y[i];
    }
  }
}

// One fused level-solve CG update over a grid-stride range (the grid and
// stride of logn_dot_kernel, so the partial sums have the same order):
//   x += alpha p;  r -= alpha q;  z = d r (d of period dn);
//   partials of r.r into part[0..] and of r.z into part[gridDim.x..].
__global__ void __launch_bounds__(256) logn_cg_update_kernel(long len, double alpha, const double* __restrict__ p,
                                                             const double* __restrict__ q, double* __restrict__ x,
                                                             double* __restrict__ r, const double* __restrict__ d,
                                                             long dn, double* __restrict__ z,
                                                             double* __restrict__ part) {
  __shared__ double sm[2][256];
  double a1 = 0.0, a2 = 0.0;
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < len; i += (long)gridDim.x * blockDim.x) {
    x[i] = alpha * p[i] + 1.0 * x[i];
    const double ri = -alpha * q[i] + 1.0 * r[i];
    r[i] = ri;
    const double zi = d[i % dn] * ri;
    z[i] = zi;
    a1 += ri * ri;
    a2 += ri * zi;
  }
  sm[0][threadIdx.x] = a1;
  sm[1][threadIdx.x] = a2;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      sm[0][threadIdx.x] += sm[0][threadIdx.x + w];
      sm[1][threadIdx.x] += sm[1][threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[blockIdx.x] = sm[0][0];
    part[gridDim.x + blockIdx.x] = sm[1][0];
  }
}

namespace {

// Sums of two values per thread over a block of NT threads, the same bits in every thread.
template <int NT>
__device__ __forceinline__ void block_sum2(double& a, double& b, double (*red)[2]) {
  a = wave_sum(a);
  b = wave_sum(b);
  if constexpr (NT == 64) {
    __syncthreads();
    return;
  }
  static_assert(NT == 64 || NT == 512, "eight waves or one");
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6][0] = a;
    red[threadIdx.x >> 6][1] = b;
  }
  __syncthreads();
  // lane 2 w + i (of each 16) holds sum i of wave w
  double t = red[(threadIdx.x >> 1) & 7][threadIdx.x & 1];
  t += dpp_f64<0x128>(t);  // row_ror:8
  t += dpp_f64<0x124>(t);  // row_ror:4
  t += dpp_f64<0x122>(t);  // row_ror:2
  a = lane_f64(t, 0);
  b = lane_f64(t, 1);
}

}  // namespace

// Jacobi-preconditioned CG on a diagonal sub-block of A (chaos columns lo ..
// lo + nr - 1), all iterations in one launch; several systems with the same
// block run side by side (one block each).
// The G blocks of a system each own the operator rows of a contiguous share.
// Every block keeps all of r (registers) and p (LDS, with zeros around each
// column's grid so that a row's neighbours need no masks) and repeats the vector
// work and the sums, so an iteration needs one exchange: each block publishes its
// rows of q = A p and takes everyone's. A place of the exchange is empty until its
// value is there; three buffers take turns, and a block clears its rows of one
// exchange after the next is complete (then every block has read them).
// lpr lanes share an operator row; with TREG > 0 a lane keeps the element
// coefficients of its (at most TREG) tasks in registers for the whole solve, so
// the loop reads no memory but the exchange (and the inverse diagonal beside more than
// 8 unknowns a thread); its tasks are the blocks of one row or, where a row has one
// block, several rows. As many are held as leave the registers unspilled: six beside 8
// unknowns a thread, two beside 20 (with ten, 189 spilled registers made an iteration
// of 16 x 16, N = 4, degree 4 11.5 us against 10.3, of two columns of 69^2 16.0 against
// 10.3), none beside 38, where r and q alone spill (290 registers; 81 x 81, N = 2,
// degree 2 25.8 us an iteration). Thread t holds the vector elements i = NT k + t; x_i
// is kept by the block that k falls to (k % G, at most one k per block when G >= VPT),
// or, if a block has several, in memory.
// The stored blocks are numbered in the order of the rows' lists.
// An iteration is a chain of latencies, not a stream: the exchange (one store and
// its way to the others, about 2 us), two block sums and the tasks. 10 x 10, N = 4,
// degree 4 (2835 unknowns of the top level): 63 us per iteration as four kernels
// and two host round trips, 5.2 us here with 24 to 64 blocks (26 us with one block,
// 8.4 with 8); 16 x 16: 10.3 us with 32 blocks, 67 with one.
// A wait that expires (blocks of this launch held back by other work on the device)
// sets the status, and in later launches the waves that find it set give up at their
// first wait. Another block may set it while a block starts, so its waves may differ in
// what they find: whether a block leaves is settled for all of it between two barriers.
template <int NT, int VPT, int TREG>
__global__ void __launch_bounds__(NT, 1) logn_solve_kernel(LognSolveArgs A) {
  constexpr bool REG = TREG > 0;
  constexpr bool SMALL = VPT <= 8;  // x and the inverse diagonal in registers too
  extern __shared__ double lds[];
  __shared__ double red[2][NT / 64][2];
  __shared__ int dead;
  const int tid = threadIdx.x;
  const long limit = __builtin_amdgcn_readfirstlane((int)agent_load(A.status)) != 0 ? 0 : A.spins;
  const int sys = blockIdx.x / A.G, g = blockIdx.x - sys * A.G;
  const int nx = A.n_e - 1, n = nx * nx, len = n * A.nr;
  const int RS = nx + 1, CS = RS * RS;  // row and column strides of the padded p
  const int psize = A.nr * CS + RS + 2;
  double* P = lds;           // padded p
  double* Qs = lds + psize;  // q of a system of one block
  const double* B = A.B + (long)sys * A.stride;
  double* X = A.X + (long)sys * A.stride;
  const double* dinv = A.Dinv + (long)A.lo * n;
  if (tid == 0) dead = 0;
  for (int i = tid; i < psize; i += NT) P[i] = 0.0;
  double r[VPT], d[SMALL ? VPT : 1], x[SMALL ? VPT : 1];
  unsigned pk[(VPT + 1) / 2];  // places of the elements in the padded p, two to a word
  auto pos = [&](int k) { return (int)((pk[k >> 1] >> (16 * (k & 1))) & 0xFFFFu); };
  double bb = 0.0, rz = 0.0;
#pragma unroll
  for (int k = 0; k < VPT; ++k) {
    const int i = k * NT + tid;
    unsigned o = 0;
    r[k] = 0.0;
    if constexpr (SMALL) {
      x[k] = 0.0;
      d[k] = 0.0;
    }
    if (i < len) {
      const int b = i / n, node = i - b * n, iy = node / nx, ix = node - iy * nx;
      o = 1 + RS + b * CS + iy * RS + ix;
      r[k] = B[i];
      const double di = dinv[i];
      if constexpr (SMALL) d[k] = di;
      bb += r[k] * r[k];
      rz += r[k] * (di * r[k]);
    }
    pk[k >> 1] = (k & 1) ? pk[k >> 1] | (o << 16) : o;
  }
  double x1 = 0.0;  // !SMALL, G >= VPT: the element k = g
  // this lane's operator rows: row0 + pass * rpp, blocks sub, sub + lpr, ..
  const int rpp = NT / A.lpr, sub = tid & (A.lpr - 1);
  const int row_end = min(len, (g + 1) * A.rows);
  const int row0 = g * A.rows + tid / A.lpr;
  const int ntj = (A.nr + A.lpr - 1) / A.lpr;
  auto centre = [&](int b, int node) {
    const int iy = node / nx;
    return 1 + RS + b * CS + iy * RS + node - iy * nx;
  };
  double c[REG ? TREG : 1][4];
  int pc[REG ? TREG : 1];
  if constexpr (REG) {
#pragma unroll
    for (int t = 0; t < TREG; ++t) {
      pc[t] = 1 + RS;
      c[t][0] = c[t][1] = c[t][2] = c[t][3] = 0.0;
      const int row = ntj == 1 ? row0 + t * rpp : row0;
      if (row >= row_end || (ntj > 1 && t >= ntj)) continue;
      const int a = A.lo + row / n, node = row % n;
      // first stored block of operator row a with a column in the sub-block
      int first = A.rptr[a], last = A.rptr[a + 1];
      for (int hi = last; first < hi;) {
        const int mid = (first + hi) >> 1;
        if (A.rcol[mid] < A.lo) first = mid + 1;
        else hi = mid;
      }
      const int e = first + (ntj == 1 ? 0 : t * A.lpr) + sub;
      if (e >= last || A.rcol[e] >= A.lo + A.nr) continue;
      const double* ck = A.C + (long)e * A.n_e * A.n_e + node / nx * A.n_e + node % nx;
      pc[t] = centre(A.rcol[e] - A.lo, node);
      c[t][0] = ck[0];
      c[t][1] = ck[1];
      c[t][2] = ck[A.n_e];
      c[t][3] = ck[A.n_e + 1];
    }
  }
  // q at the node whose padded p has its centre at P[o], element coefficients around it
  auto node_value = [&](int o, double c00, double c01, double c10, double c11) {
    const double* q = P + o;
    const double uc = 4.0 * q[0], w = q[-1], e = q[1], s = q[-RS], nn = q[RS];
    return c00 * (uc - w - s - 2.0 * q[-RS - 1]) + c01 * (uc - e - s - 2.0 * q[-RS + 1]) +
           c10 * (uc - w - nn - 2.0 * q[RS - 1]) + c11 * (uc - e - nn - 2.0 * q[RS + 1]);
  };
  __syncthreads();
  block_sum2<NT>(bb, rz, red[0]);
  int it = 0;
  if (bb != 0.0) {
#pragma unroll
    for (int k = 0; k < VPT; ++k)
      if (k * NT + tid < len) P[pos(k)] = (SMALL ? d[SMALL ? k : 0] : dinv[k * NT + tid]) * r[k];  // p = z
  }
  const bool x_mem = !SMALL && A.G < VPT;
  if (x_mem)
    for (int i = tid + NT * g; i < len; i += NT * A.G) X[i] = 0.0;
  __syncthreads();
  if (bb != 0.0)
    while (it < A.maxit) {
      unsigned long long* ex = A.ex + (long)(it % 3) * len;
      unsigned long long* old = A.ex + (long)((it + 2) % 3) * len;
      int me = tid;
      asm volatile("" : "+v"(me));  // the addresses below are not kept across iterations
      // this block's rows of q = A p
      auto publish = [&](int row, double v) {
        for (int w = A.lpr >> 1; w > 0; w >>= 1) v += __shfl_xor(v, w);
        v *= 1.0 / 6.0;
        if (sub == 0 && row < row_end) {
          if (A.G == 1) {
            Qs[row] = v;
          } else {
            __builtin_amdgcn_s_waitcnt(0);  // this thread's clearing stores are done
            agent_store(ex + row, publishable(v));
          }
        }
      };
      if constexpr (REG) {
        double v = 0.0;
#pragma unroll
        for (int t = 0; t < TREG; ++t) {
          const double w = node_value(pc[t], c[t][0], c[t][1], c[t][2], c[t][3]);
          if (ntj == 1) publish(row0 + t * rpp, w);
          else v += w;  // zero coefficients past the row's blocks
        }
        if (ntj > 1) publish(row0, v);
      } else {
        for (int row = row0; row - tid / A.lpr < row_end; row += rpp) {
          double v = 0.0;
          if (row < row_end) {
            const int a = A.lo + row / n, node = row % n;
            const int e0 = node / nx * A.n_e + node % nx;
            const int o = centre(0, node);
            // the row's stored blocks; those past the sub-block add nothing
            const int first = A.first[a], last = A.last[a];
#pragma unroll 4
            for (int e = first + sub; e < last; e += A.lpr) {
              const double* ck = A.C + (long)e * A.n_e * A.n_e + e0;
              v += node_value(o + (A.rcol[e] - A.lo) * CS, ck[0], ck[1], ck[A.n_e], ck[A.n_e + 1]);
            }
          }
          publish(row, v);
        }
      }
      // everyone's q
      double q[VPT];
      double pq = 0.0, unused = 0.0;
      if (A.G == 1) {
        __syncthreads();
#pragma unroll
        for (int k = 0; k < VPT; ++k) q[k] = k * NT + me < len ? Qs[k * NT + me] : 0.0;
      } else {
#pragma unroll
        for (int k = 0; k < VPT; ++k)
          q[k] = k * NT + me < len ? __longlong_as_double((long long)agent_load(ex + k * NT + me)) : 0.0;
        auto empty = [&](int k) { return (unsigned long long)__double_as_longlong(q[k]) == kEmpty; };
        for (long spins = 0;; ++spins) {
          bool miss = false;
#pragma unroll
          for (int k = 0; k < VPT; ++k) miss |= empty(k);
          if (!__any(miss)) break;
          if (spins >= limit) {
            dead = 1;  // the block leaves as a whole after its next barrier
            break;
          }
          // the missing ones again, all on their way together
#pragma unroll
          for (int k = 0; k < VPT; ++k)
            if (empty(k)) q[k] = __longlong_as_double((long long)agent_load(ex + k * NT + me));
        }
      }
#pragma unroll
      for (int k = 0; k < VPT; ++k)
        if (k * NT + me < len) pq += P[pos(k)] * q[k];
      block_sum2<NT>(pq, unused, red[1]);
      if (A.G > 1) {
        if (dead) {
          if (tid == 0) {
            agent_store(A.status, 1ull);
            __hip_atomic_store(A.told, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
          }
          break;
        }
        if (it > 0 && sub == 0)
          for (int row = row0; row < row_end; row += rpp) agent_store(old + row, kEmpty);
      }
      if (!(pq > 0.0) || !isfinite(pq)) break;
      const double alpha = rz / pq;
      double rr = 0.0, rzn = 0.0;
#pragma unroll
      for (int k = 0; k < VPT; ++k) {
        const int i = k * NT + me;
        if (i < len) {
          if constexpr (SMALL) {
            x[k] = fma(alpha, P[pos(k)], x[k]);
          } else if (x_mem) {
            if (k % A.G == g) X[i] = fma(alpha, P[pos(k)], X[i]);
          } else if (k == g) {
            x1 = fma(alpha, P[pos(k)], x1);
          }
          r[k] = fma(-alpha, q[k], r[k]);
          rr += r[k] * r[k];
          rzn += r[k] * ((SMALL ? d[SMALL ? k : 0] : dinv[i]) * r[k]);
        }
      }
      block_sum2<NT>(rr, rzn, red[0]);
      ++it;
      if (rr <= A.rtol * A.rtol * bb) break;
      const double beta = rzn / rz;
      rz = rzn;
#pragma unroll
      for (int k = 0; k < VPT; ++k)
        if (k * NT + me < len)
          P[pos(k)] = fma(beta, P[pos(k)], (SMALL ? d[SMALL ? k : 0] : dinv[k * NT + me]) * r[k]);
      __syncthreads();
    }
#pragma unroll
  for (int k = 0; k < VPT; ++k) {
    const int i = k * NT + tid;
    if (i >= len) continue;
    if constexpr (SMALL) {
      if (k % A.G == g) X[i] = x[k];
    } else if (!x_mem && k == g) {
      X[i] = x1;
    }
  }
  if (g == 0 && tid == 0 && it > 0) atomicAdd(A.its, (unsigned long long)it);
}

// Range of the stored blocks of every chaos row with a column in lo .. hi - 1.
__global__ void logn_range_kernel(const int* rptr, const int* rcol, int P, int lo, int hi, int* first, int* last) {
  for (int a = threadIdx.x; a < P; a += blockDim.x)
    for (int side = 0; side < 2; ++side) {
      int l = rptr[a], h = rptr[a + 1];
      while (l < h) {
        const int mid = (l + h) >> 1;
        if (rcol[mid] < (side ? hi : lo)) l = mid + 1;
        else h = mid;
      }
      (side ? last : first)[a] = l;
    }
}

__global__ void logn_clear_kernel(unsigned long long* ex, long n) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) ex[i] = kEmpty;
}

// Launch shape of a system of len = n nr unknowns: threads, blocks, lanes per row
// and rows per block with the least estimated time of an iteration. A block's
// tasks (a row and one of its blocks, per lane) take about 0.15 us each with their
// coefficients in registers, 0.3 us without, the exchange of more than one block
// 2 us. At most 64 blocks, so that the waiting blocks of the launches that the
// hardware queues of a process can run at once (four) all fit on the device; where
// more wait on each other, the bounded waits end it.
// Systems of at most 256 unknowns run on one wave, whose sums need no barrier.
bool logn_solve_shape(int n_e, int nr, int nsys, LognSolveArgs& A, int& nt, int& vpt, int& treg, size_t& lds_bytes) {
  const long nx = n_e - 1, n = nx * nx, len = n * nr;
  const long psize = nr * (nx + 1) * (nx + 1) + nx + 3;
  constexpr long lds_max = 160 * 1024 - 1024;
  if (len > 38L * 512 || psize * 8 > lds_max) return false;
  nt = len <= 256 ? 64 : 512;
  vpt = nt == 64 ? 4 : len <= 2 * 512 ? 2 : len <= 8 * 512 ? 8 : len <= 20 * 512 ? 20 : 38;
  const int held = vpt <= 8 ? 6 : vpt == 20 ? 2 : 0;  // tasks whose coefficients the kernel can hold
  double best = 1e300;
  for (int G : {1, 2, 4, 8, 16, 24, 32, 48, 64}) {
    if (G > 1 && (G > len || nsys > 1 || nt == 64)) break;  // several systems take one block each
    if (G == 1 && (psize + len) * 8 > lds_max) continue;
    const long rows = (len + G - 1) / G;
    int lpr = 1;
    while (lpr < 16 && 2 * lpr <= nr && rows * 2 * lpr <= nt) lpr *= 2;
    const long passes = (rows + nt / lpr - 1) / (nt / lpr);
    const long ntj = (nr + lpr - 1) / lpr;
    const bool in_regs = ntj == 1 ? passes <= held : passes == 1 && ntj <= held;
    const double cost = (in_regs ? 0.15 : 0.3) * passes * ntj + (G > 1 ? 2.0 : 0.0);
    if (cost < best) {
      best = cost;
      A.G = (int)((len + rows - 1) / rows);  // no block without rows: its reads would not be waited for
      A.lpr = lpr;
      A.rows = (int)rows;
      treg = in_regs ? held : 0;
    }
  }
  if (best > 1e299) return false;
  lds_bytes = 8 * (size_t)(psize + (A.G == 1 ? len : 0));
  return true;
}

hipError_t launch_logn_solve(const LognSolveArgs& args, int nsys, hipStream_t s, bool* done) {
  LognSolveArgs A = args;
  int nt = 0, vpt = 0, treg = 0;
  size_t lds_bytes = 0;
  *done = logn_solve_shape(A.n_e, A.nr, nsys, A, nt, vpt, treg, lds_bytes);
  if (!*done) return hipSuccess;
  const long len = (long)(A.n_e - 1) * (A.n_e - 1) * A.nr;
  if (A.G > 1) hipLaunchKernelGGL(logn_clear_kernel, dim3(32), dim3(256), 0, s, A.ex, 3 * len);
  if (treg == 0)
    hipLaunchKernelGGL(logn_range_kernel, dim3(1), dim3(256), 0, s, A.rptr, A.rcol, A.P, A.lo, A.lo + A.nr, A.first,
                       A.last);
  auto launch = [&](auto kfn) {
    if (lds_bytes > 64 * 1024) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kfn),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kfn, dim3((unsigned)(nsys * A.G)), dim3(nt), lds_bytes, s, A);
    return hipGetLastError();
  };
  if (nt == 64) return treg ? launch(logn_solve_kernel<64, 4, 6>) : launch(logn_solve_kernel<64, 4, 0>);
  if (treg == 6) return vpt == 2 ? launch(logn_solve_kernel<512, 2, 6>) : launch(logn_solve_kernel<512, 8, 6>);
  if (treg == 2) return launch(logn_solve_kernel<512, 20, 2>);
  return vpt == 2    ? launch(logn_solve_kernel<512, 2, 0>)
         : vpt == 8  ? launch(logn_solve_kernel<512, 8, 0>)
         : vpt == 20 ? launch(logn_solve_kernel<512, 20, 0>)
                     : launch(logn_solve_kernel<512, 38, 0>);
}

void launch_logn_cg_update(long len, double alpha, const double* p, const double* q, double* x, double* r,
                           const double* d, long dn, double* z, double* part, int nblocks, hipStream_t s) {
  hipLaunchKernelGGL(logn_cg_update_kernel, dim3(nblocks), dim3(256), 0, s, len, alpha, p, q, x, r, d,
                     dn > 0 ? dn : len, z, part);
}

void launch_logn_apply(const int* rptr, const int* rcol, const int* rslot, const double* C, const double* X,
                       int n_e, long n, int row0, int nrows, int col0, int col1, int mode, const double* R, double* Y,
                       hipStream_t s) {
  if (n <= 0 || nrows <= 0) return;
  hipLaunchKernelGGL(logn_apply_kernel, dim3((unsigned)((n + 255) / 256), nrows), dim3(256), 0, s, rptr, rcol, rslot,
                     C, X, n_e, n, row0, col0, col1, mode, R, Y);
}

void launch_logn_invdiag(const int* rptr, const int* rcol, const int* rslot, const double* C, int n_e, long n, int P,
                         double* Dinv, hipStream_t s) {
  if (n <= 0 || P <= 0) return;
  hipLaunchKernelGGL(logn_invdiag_kernel, dim3((unsigned)((n + 255) / 256), P), dim3(256), 0, s, rptr, rcol, rslot, C,
                     n_e, n, Dinv);
}

void launch_logn_dot(const double* x, const double* y, long len, double* part, int nblocks, hipStream_t s) {
  hipLaunchKernelGGL(logn_dot_kernel, dim3(nblocks), dim3(256), 0, s, x, y, len, part);
}

void launch_logn_axpby(long len, double a, const double* x, double b, double* y, int mode, const double* d,
                       long dn, hipStream_t s) {
  if (len <= 0) return;
  const long nb = std::min<long>((len + 255) / 256, 4096);
  hipLaunchKernelGGL(logn_axpby_kernel, dim3((unsigned)nb), dim3(256), 0, s, len, a, x, b, y, mode, d,
                     dn > 0 ? dn : len);
}

void launch_logn_mean_apply(const double* c, const double* X, int n_e, long n, int ncols, double* Y, hipStream_t s) {
  if (n <= 0 || ncols <= 0) return;
  hipLaunchKernelGGL(logn_mean_apply_kernel, dim3((unsigned)((n + 255) / 256), ncols), dim3(256), 0, s, c, X, n_e, n,
                     Y);
}

void launch_logn_blocks(const long* ptr, const int* term, const double* g, const double* kc, int ne2, int nslots,
                        double* C, hipStream_t s) {
  if (nslots <= 0) return;
  const int gy = nslots < 65535 ? nslots : 65535;
  hipLaunchKernelGGL(logn_blocks_kernel, dim3((ne2 + 255) / 256, gy), dim3(256), 0, s, ptr, term, g, kc, ne2, nslots,
                     C);
}

void launch_logn_matvec(const int* rptr, const int* rcol, const int* rslot, const double* C, const double* U,
                        int n_e, long n, int P, double* Y, hipStream_t s) {
  if (n <= 0 || P <= 0) return;
  hipLaunchKernelGGL(logn_matvec_kernel, dim3((unsigned)((n + 255) / 256), P), dim3(256), 0, s, rptr, rcol, rslot,
                     C, U, n_e, n, Y);
}

}  // namespace sgk
