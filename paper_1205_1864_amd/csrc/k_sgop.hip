// SG block operator: the MAT-VEC of the stochastic Galerkin matrix (Remark
// after eq. (global-matrix-block)) and the coupling products B_l, C_l of
// Algorithm 1, applied without forming any matrix.
//
// For chaos row a the kernel evaluates
//   out[a] = rcoef * rsrc[a] + diag * K_Lap in[a]
//            + sgn * sum_{(k, b, g) in lists(a)} g * K_k in[b]
// where K_k = sum_e a_k(e) K^e is the Q1 stiffness of the piecewise-constant
// coefficient a_k. At node i the element form is
//   (K_k u)_i = 1/6 sum_{e ni i} a_k(e) (4 u_i - u_adj1 - u_adj2 - 2 u_opp)
// over the four elements sharing i (the Q1 element matrix of a square).
#include "sg_internal.h"
#include "sg_device.h"

namespace sgk {

namespace {

// Strip kernel. A wave takes a strip of up to 62 node columns (lanes 1..width;
// the lanes beside them hold the neighbouring columns) by YN node rows for one
// chaos row, and gathers, per Galerkin neighbour, the node values of the rows
// around the strip and the coefficients of the element rows between them: one
// load per row and lane, the horizontal neighbours by lane shifts. The
// neighbour list is uniform in a block, and every load of a neighbour is
// unconditional (a place outside the grid reads the nearest one inside, and the
// value is replaced by zero), so that all of them are in flight together.
//
// Bound by latency where a launch is small and by the L1 data path on large
// grids (2.75 loads of 8 bytes per node and neighbour at YN = 4, about 2 ps per
// node and neighbour). Measured (FP64, caches warm): the full operator at 16^2,
// M = 4, p = 2 119 -> 7 us and at 75^2, M = 5, p = 3 73 -> 9 us, the top level's
// coupling products there 65 / 121 -> 8 / 8 us and at 256^2, M = 10, p = 3 115 /
// 187 -> 77 / 100 us; before, one wave marched 16 rows, a chain of loads per row.
// The same kernel without lane shifts (three loads per row) took 104 / 113 us
// there, and 8 rows a wave 78 / 107 us.
// That march read a large level once and a bit, so towards the lower level of many
// terms it was ahead by a little on large grids: M = 8, p = 3, level 3 to 2 / 2 to 3,
// 384^2 88 / 189 us against 96 / 119 now, 512^2 177 / 319 against 186 / 246 (both
// directions are needed in an action). Stacking a block's waves in y instead of in x
// gained nothing there (98 / 119 and 190 / 264 us).
constexpr int kStripThreads = 256;

// out0 and out1 receive the parts of the lower and the upper node row of an
// element row: elements left (l) and right (r) of the column, node values W, C, E
// of the lower (0) and upper (1) row.
template <typename T>
__device__ __forceinline__ void element_row(T l, T r, T W0, T C0, T E0, T W1, T C1, T E1, T& out0, T& out1) {
  const T a0 = T(4) * C0 - C1, a1 = T(4) * C1 - C0;
  out0 += l * (a0 - W0 - T(2) * W1) + r * (a0 - E0 - T(2) * E1);
  out1 += l * (a1 - W1 - T(2) * W0) + r * (a1 - E1 - T(2) * E0);
}

template <typename T, int YN>
__global__ void __launch_bounds__(kStripThreads) sgop_strip_kernel(const SgOpArgs<T> A, int tiles, int strips,
                                                                   int width) {
  if (A.active && ld_uniform(A.active, 0) == 0) return;
  // blocks of an XCD (b mod 8) go through the rows of one node tile before the
  // next, so that the tile's columns are read from memory once
  int row, tile;
  if (tiles >= 16) {
    const int xcd = blockIdx.x % 8, j = blockIdx.x / 8;
    row = j % A.nrows;
    tile = xcd + 8 * (j / A.nrows);
    if (tile >= tiles) return;
  } else {
    row = blockIdx.x / tiles;
    tile = blockIdx.x % tiles;
  }
  row += A.row0;
  const int nx = A.nx, ne = A.n_e;
  const int lane = threadIdx.x & 63;
  const int w = tile * (kStripThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int iy0 = w / strips * YN;
  if (iy0 >= nx) return;
  const int ix = w % strips * width + lane - 1;
  const bool mine = lane >= 1 && lane <= width && ix < nx;
  const int cx = min(max(ix, 0), nx - 1), ex = min(max(ix, 0), nx);
  // node rows iy0 - 1 .. iy0 + YN, element rows iy0 .. iy0 + YN
  bool on[YN + 2];
  int off[YN + 2], eoff[YN + 1];
#pragma unroll
  for (int j = 0; j < YN + 2; ++j) {
    const int y = iy0 - 1 + j;
    const bool in_y = y >= 0 && y < nx;
    off[j] = (in_y ? y : iy0) * nx + cx;
    on[j] = in_y && cx == ix;
  }
#pragma unroll
  for (int j = 0; j < YN + 1; ++j) eoff[j] = min(iy0 + j, nx) * ne + ex;
  T sum[YN + 2];
#pragma unroll
  for (int j = 0; j < YN + 2; ++j) sum[j] = T(0);
  auto add = [&](const T* col, const T* ak, T g) {
    T W[YN + 2], C[YN + 2], E[YN + 2], l[YN + 1], r[YN + 1];
#pragma unroll
    for (int j = 0; j < YN + 2; ++j) C[j] = col[off[j]];
#pragma unroll
    for (int j = 0; j < YN + 1; ++j) l[j] = ak ? ak[eoff[j]] : T(1);
#pragma unroll
    for (int j = 0; j < YN + 2; ++j) {
      C[j] = on[j] ? C[j] : T(0);
      W[j] = from_prev(C[j]);
      E[j] = from_next(C[j]);
      if (j <= YN) r[j] = from_next(l[j]);
    }
#pragma unroll
    for (int j = 0; j < YN + 1; ++j)
      element_row(g * l[j], g * r[j], W[j], C[j], E[j], W[j + 1], C[j + 1], E[j + 1], sum[j], sum[j + 1]);
  };
  for (int pass = 0; pass < 2; ++pass) {
    if (!(pass == 0 ? A.use_lower : A.use_upper)) continue;
    const int* ptr = pass == 0 ? A.lists.lo_ptr : A.lists.up_ptr;
    const int* ent = pass == 0 ? A.lists.lo_ent : A.lists.up_ent;
    const T* gv = pass == 0 ? A.lists.lo_g : A.lists.up_g;
    const int e1 = ld_uniform(ptr, row + 1);
    for (int e = ld_uniform(ptr, row); e < e1; ++e) {
      const int pk = ld_uniform(ent, e);
      add(A.in + (long)(pk & 0xFFFFF) * A.n, A.a + (long)((pk >> 20) - 1) * ne * ne, A.sgn * ld_uniform(gv, e));
    }
  }
  if (A.diag != T(0)) add(A.in + (long)row * A.n, nullptr, A.diag);
  T* out = A.out + (long)row * A.n;
  const T* rs = A.rsrc ? A.rsrc + (long)row * A.n : nullptr;
#pragma unroll
  for (int j = 0; j < YN; ++j)
    if (mine && iy0 + j < nx) {
      T v = sum[j + 1] / T(6);
      if (rs) v += A.rcoef * rs[off[j + 1]];
      out[off[j + 1]] = v;
    }
}

template <typename T, int YN>
void launch_strip(const SgOpArgs<T>& args, int strips, int width, hipStream_t s) {
  const long waves = (long)strips * ((args.nx + YN - 1) / YN);
  const int tiles = (int)((waves + kStripThreads / 64 - 1) / (kStripThreads / 64));
  const long blocks = (tiles >= 16 ? 8L * ((tiles + 7) / 8) : tiles) * args.nrows;
  hipLaunchKernelGGL((sgop_strip_kernel<T, YN>), dim3((unsigned)blocks), dim3(kStripThreads), 0, s, args, tiles, strips,
                     width);
}

}  // namespace

// ---------------------------------------------------------------------------
// Row-staged full operator (FP64). A block (one per CU: the staged rows take
// most of the LDS) works through pieces of kStageOut node columns by TY node
// rows. For each element row e of a piece (between node rows e - 1 and e) it
// holds node rows e - 1 and e of every chaos column, and the coefficients of
// element row e, in LDS; the next row is loaded into registers while the
// current one is used. Each half wave owns a list of output columns a; for
// every term (b, k, g) of a (b = a: k = 0 and g = 1 with coefficient theta0;
// b = a -+ e_k: the Galerkin weight g of G_k) it forms, lane by lane,
//   R0 += g c_k(right element) U_b(e - 1),  R1 += g c_k(right element) U_b(e),
//   L0 += g c_k(left element) U_b(e - 1),   L1 += g c_k(left element) U_b(e),
// the corner values of sum_terms c g U_b on the element right of the node
// (BL = R0, TL = R1; BR and TR are the next lane's L0, L1). The element matrix
// of the Q1 Laplacian (times 6: 4 on the diagonal, -1 along the edges, -2
// across) turns them into the element's contributions to its four corners,
// which complete node row e - 1 and start node row e of output a.
// ---------------------------------------------------------------------------
size_t stage_lds_bytes(int P, int M, int nterms, int nslots) {
  if (P < 1 || P >= 0xFFFF || M < 0 || M > 255 || nterms < 0 || nterms > 0xFFFF || nslots < 1) return 0;
  if ((long)P * kStageLanes > (long)kStagePre * kStageWaves * 64) return 0;
  if ((M + 1) * kStageLanes > kStageWaves * 64) return 0;
  // node rows [P][32 lanes][2 parities], coefficients [M + 1][32], terms, slots
  const size_t b = sizeof(double) * ((size_t)P * 2 * kStageLanes + (size_t)(M + 1) * kStageLanes) +
                   sizeof(StageTerm) * (size_t)nterms + sizeof(StageSlot) * (size_t)nslots;
  return b <= 160 * 1024 ? b : 0;
}

namespace {

// One element row e of a piece: node rows e - 1 (parity 1 - PE) and e (parity PE)
// and the coefficients of element row e are in LDS; the next node row (parity
// 1 - PE) and coefficient row are loaded meanwhile and stored after the step's
// reads. Completes output node row e - 1 (if e > y0) and starts row e.
template <int PE>
__device__ __forceinline__ void stage_step(const SgOpArgs<double>& A, const StageJob& J, double* Ub, double* Cb,
                                           const StageTerm* Tl, const StageSlot* Sl, int e, int y0, int y1, int x0,
                                           int s_begin, int s_end, double (&Yc)[kStageSlots]) {
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31;
  const int nx = A.nx, n_e = A.n_e;
  const long n = A.n;
  const int P = J.P, MC = J.M + 1;
  const bool more = e < y1;
  // the next rows into registers: thread tid stages lane tid % 32 of chaos
  // columns tid / 32 + 32 j (32-bit offsets: the host enables this kernel only
  // for n P < 2^31)
  const int sb = tid >> 5, sx = x0 - 1 + (tid & 31);
  double nv[kStagePre];
  double nc = 0.0;
  if (more) {
    const int gy = e + 1;
    const bool ok = gy < nx && sx >= 0 && sx < nx;
    const unsigned base = (unsigned)sb * (unsigned)n + (unsigned)(gy * nx + sx);
    const unsigned step = 32u * (unsigned)n;
#pragma unroll
    for (int j = 0; j < kStagePre; ++j) nv[j] = (ok && sb + 32 * j < P) ? A.in[base + (unsigned)j * step] : 0.0;
    if (tid < MC * kStageLanes) {
      const int k = tid >> 5, ex = x0 + (tid & 31);
      if (ex < n_e) nc = k == 0 ? A.diag : A.a[(long)(k - 1) * n_e * n_e + (long)gy * n_e + ex];
    }
  }
  const double2* Ul = reinterpret_cast<const double2*>(Ub) + l32;  // (node row parity 0, parity 1)
  const double* Cl = Cb + l32;                                      // right element of the lane's node
  const unsigned hb = (lane >> 5) * 16u, hk = (lane >> 5) * 8u;
  const int gx = x0 - 1 + l32;
  const double scale = 1.0 / 6.0, theta0 = A.diag;
  auto accumulate = [&](double g, const double2& uv, double cr, double& R0, double& R1, double& L0, double& L1) {
    const double u0 = PE ? uv.x : uv.y, u1 = PE ? uv.y : uv.x;  // node rows e - 1, e
    const double gr = g * cr, gl = from_prev(gr);                 // the left element is the previous lane's right one
    R0 = fma(gr, u0, R0);
    R1 = fma(gr, u1, R1);
    L0 = fma(gl, u0, L0);
    L1 = fma(gl, u1, L1);
  };
  // a term's staged values: U_b at node rows e - 1 and e (one 16-byte read) and
  // the coefficient of k on the right element
  auto term_vals = [&](const uint4& q, double2& uv, double& cr, double& g) {
    const unsigned b = (q.x >> hb) & 0xFFFFu, k = (q.y >> hk) & 0xFFu;
    uv = Ul[b * kStageLanes];
    cr = Cl[k * kStageLanes];
    g = __hiloint2double((int)q.w, (int)q.z);
  };
#pragma unroll
  for (int s = 0; s < kStageSlots; ++s) {
    const int si = s_begin + s;
    if (si < s_end) {
      const uint2 sv = *reinterpret_cast<const uint2*>(Sl + si);
      const int t0 = __builtin_amdgcn_readfirstlane((int)(sv.y & 0xFFFFu));
      const int nt = __builtin_amdgcn_readfirstlane((int)(sv.y >> 16));
      const unsigned oh = (sv.x >> hb) & 0xFFFFu;
      const int out = oh == 0xFFFFu ? -1 : (int)oh;
      // the mean term: coefficient theta0 on both elements, weight 1
      const double2 ud = Ul[(out >= 0 ? out : (int)(sv.x & 0xFFFFu)) * kStageLanes];
      const double d0 = theta0 * (PE ? ud.x : ud.y), d1 = theta0 * (PE ? ud.y : ud.x);
      double R0 = d0, R1 = d1, L0 = d0, L1 = d1;
      const uint4* tq = reinterpret_cast<const uint4*>(Tl + t0);
      int t = 0;
      // two terms at a time: every LDS read of both goes out before the arithmetic
      for (; t + 1 < nt; t += 2) {
        const uint4 qa = tq[t], qb = tq[t + 1];
        double2 ua, ub;
        double ca, cb, ga, gb;
        term_vals(qa, ua, ca, ga);
        term_vals(qb, ub, cb, gb);
        accumulate(ga, ua, ca, R0, R1, L0, L1);
        accumulate(gb, ub, cb, R0, R1, L0, L1);
      }
      if (t < nt) {
        double2 ua;
        double ca, ga;
        term_vals(tq[t], ua, ca, ga);
        accumulate(ga, ua, ca, R0, R1, L0, L1);
      }
      const double BL = R0, TL = R1, BR = from_next(L0), TR = from_next(L1);
      const double S = (BL + BR) + (TR + TL);
      const double oBL = 5.0 * BL - S - TR;
      const double oBR = 5.0 * BR - S - TL;
      const double oTR = 5.0 * TR - S - BL;
      const double oTL = 5.0 * TL - S - BR;
      const double bot = oBL + from_prev(oBR);  // node row e - 1
      const double top = oTL + from_prev(oTR);  // node row e
      if (e > y0 && out >= 0 && l32 >= 1 && l32 <= kStageOut && gx < nx)
        A.out[(unsigned)out * (unsigned)n + (unsigned)((e - 1) * nx + gx)] = scale * (Yc[s] + bot);
      Yc[s] = top;
    }
  }
  __syncthreads();  // every read of node row e - 1 and of element row e is done
  if (more) {
    double* dst = Ub + (sb * kStageLanes + (tid & 31)) * 2 + (1 - PE);
#pragma unroll
    for (int j = 0; j < kStagePre; ++j)
      if (sb + 32 * j < P) dst[j * 32 * (2 * kStageLanes)] = nv[j];
    if (tid < MC * kStageLanes) Cb[tid] = nc;
  }
  __syncthreads();
}

__global__ void __launch_bounds__(kStageWaves * 64) sgop_stage_kernel(const SgOpArgs<double> A, const StageJob J) {
  if (A.active && ld_uniform(A.active, 0) == 0) return;
  extern __shared__ double stage_lds[];
  const int P = J.P, MC = J.M + 1;
  double* Ub = stage_lds;                              // [P][32][2]: node rows by parity
  double* Cb = Ub + P * 2 * kStageLanes;               // [M + 1][32]: coefficients of the current element row
  StageTerm* Tl = reinterpret_cast<StageTerm*>(Cb + MC * kStageLanes);
  StageSlot* Sl = reinterpret_cast<StageSlot*>(Tl + J.nterms);
  const int tid = threadIdx.x;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nx = A.nx, n_e = A.n_e;
  const long n = A.n;
  const int s_begin = ld_uniform(J.wslot, wv), s_end = ld_uniform(J.wslot, wv + 1);
  // the term and slot tables into LDS (16 and 8 bytes per entry)
  for (int i = tid; i < J.nterms; i += kStageWaves * 64)
    reinterpret_cast<uint4*>(Tl)[i] = reinterpret_cast<const uint4*>(J.terms)[i];
  for (int i = tid; i < J.nslots; i += kStageWaves * 64)
    reinterpret_cast<uint2*>(Sl)[i] = reinterpret_cast<const uint2*>(J.slots)[i];
  // pieces of this block's XCD (block b runs on XCD b mod 8), a contiguous band
  const int xcd = blockIdx.x % 8, bslot = blockIdx.x / 8;
  const int nb = ((int)gridDim.x - xcd + 7) / 8;
  const long npieces = (long)J.nyseg * J.nseg;
  const long p0 = npieces * xcd / 8, p1 = npieces * (xcd + 1) / 8;
  for (long pc = p0 + bslot; pc < p1; pc += nb) {
    const int yseg = (int)(pc / J.nseg), seg = (int)(pc % J.nseg);
    const int x0 = seg * kStageOut;     // first output node column
    const int y0 = yseg * J.TY;
    const int y1 = min(nx, y0 + J.TY);  // output node rows [y0, y1)
    // prologue: node rows y0 - 1 and y0, coefficients of element row y0
    for (int r = 0; r < 2; ++r) {
      const int gy = y0 - 1 + r, par = (y0 + 1 + r) & 1;
      const int sb = tid >> 5, sx = x0 - 1 + (tid & 31);
      const bool ok = gy >= 0 && gy < nx && sx >= 0 && sx < nx;
      const unsigned base = (unsigned)sb * (unsigned)n + (unsigned)(gy * nx + sx);
      double* dst = Ub + (sb * kStageLanes + (tid & 31)) * 2 + par;
      for (int j = 0; j < kStagePre; ++j)
        if (sb + 32 * j < P) dst[j * 32 * (2 * kStageLanes)] = ok ? A.in[base + (unsigned)j * 32u * (unsigned)n] : 0.0;
    }
    if (tid < MC * kStageLanes) {
      const int k = tid >> 5, ex = x0 + (tid & 31);
      double c = 0.0;
      if (ex < n_e) c = k == 0 ? A.diag : A.a[(long)(k - 1) * n_e * n_e + (long)y0 * n_e + ex];
      Cb[tid] = c;
    }
    __syncthreads();
    double Yc[kStageSlots];
#pragma unroll
    for (int s = 0; s < kStageSlots; ++s) Yc[s] = 0.0;
    for (int e = y0; e <= y1; ++e) {
      if (e & 1) stage_step<1>(A, J, Ub, Cb, Tl, Sl, e, y0, y1, x0, s_begin, s_end, Yc);
      else stage_step<0>(A, J, Ub, Cb, Tl, Sl, e, y0, y1, x0, s_begin, s_end, Yc);
    }
  }
}

}  // namespace

void launch_stage(const SgOpArgs<double>& args, const StageJob& job, hipStream_t s) {
  const size_t lds = stage_lds_bytes(job.P, job.M, job.nterms, job.nslots);
  if (lds == 0) return;
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(sgop_stage_kernel),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  int dev = 0, ncu = 1;
  (void)hipGetDevice(&dev);
  (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
  const long npieces = (long)job.nyseg * job.nseg;
  long grid = ncu;
  if (grid > npieces) grid = npieces;
  grid = (grid + 7) / 8 * 8;
  hipLaunchKernelGGL(sgop_stage_kernel, dim3((unsigned)grid), dim3(kStageWaves * 64), lds, s, args, job);
}

// Rows per wave (rows = 0): 4, which read 1.5 node rows and 1.25 element rows per
// row, or 2 where a launch would have fewer than eight waves per compute unit
// (the full operator at 32^2, M = 8, p = 3: 1320 waves of 4 rows 10 us, of 2 rows 8;
// at 64^2, 5280 waves of 4 rows 15 us, of 2 rows 17). Products with upper neighbours
// only, which read the larger level, take 6 from some 6000 waves of 6 on (FP64, us with
// 4 / 6 rows, level 3 to 2: 512^2, M = 8, 27 900 waves 182 / 174; 384^2, 16 100 96 / 93;
// 256^2, M = 10, 11 800 89 / 88; level 2 to 1 there, 2150 waves 34 / 36). The other
// direction does not gain (512^2, M = 8, level 2 to 3: 243 / 249).
template <typename T>
void launch_sgop(const SgOpArgs<T>& args, int rows, hipStream_t s) {
  if (args.nrows <= 0) return;
  const int strips = (args.nx + 61) / 62, width = (args.nx + strips - 1) / strips;
  auto waves = [&](int r) { return (long)strips * ((args.nx + r - 1) / r) * args.nrows; };
  if (rows == 0) rows = waves(4) < 2048 ? 2 : args.use_upper && !args.use_lower && waves(6) >= 6000 ? 6 : 4;
  if (rows <= 2) launch_strip<T, 2>(args, strips, width, s);
  else if (rows <= 4) launch_strip<T, 4>(args, strips, width, s);
  else if (rows <= 6) launch_strip<T, 6>(args, strips, width, s);
  else launch_strip<T, 8>(args, strips, width, s);
}

template void launch_sgop<double>(const SgOpArgs<double>&, int, hipStream_t);
template void launch_sgop<float>(const SgOpArgs<float>&, int, hipStream_t);

}  // namespace sgk
