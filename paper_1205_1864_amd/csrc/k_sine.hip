// Inner PCG in the sine basis: transforms to and from the basis and the
// iteration on the transformed columns.
//
// A solve is five launches (one for columns of up to 64 rows): right-hand side -> [x pass] -> [y pass] -> spectral
// right-hand side -> iteration -> spectral solution -> [y pass] -> [x pass].
// A pass is a product with sine matrices of a quarter (or half) of the length on
// folded data (FP64 or FP32 matrix instructions).
//
// Why: on the grid an iteration of degree d sweeps a column d times with halos
// and meets two column-wide synchronisations; here it is a dozen operations per
// pair of modes on values that never leave the registers. Measured at 256^2,
// degree 16, FP64: 220 white-noise columns to 1e-4 (34 iterations) 15.7 ms on banded
// tiles, 0.66 ms here; the benchmark's whole solve 230 -> 18 ms; 28 columns of 100^2
// unknowns at degree 8 730 -> 102 us.
#include <algorithm>

#include "sg_internal.h"
#include "sg_device.h"

namespace sgk {

namespace {

constexpr long kSpinLimit = 1L << 26;  // bounded waits: a stuck group aborts the launch
constexpr int kSumWidth = 4;           // sums exchanged at once by the blocks of a group

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

// 16 x 16 x 4 matrix instruction. Lane l holds A[l % 16][l / 16] and
// B[l / 16][l % 16]; register r of the result is D[row(l, r)][l % 16].
template <typename T>
struct Mac;
template <>
struct Mac<double> {
  using V = d4;
  __device__ static __forceinline__ V mac(double a, double b, V c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  __device__ static __forceinline__ int row(int lane, int r) { return (lane >> 4) + 4 * r; }
};
template <>
struct Mac<float> {
  using V = f4;
  __device__ static __forceinline__ V mac(float a, float b, V c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  __device__ static __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};

// Lengths of the products of a transform over n_e = nx + 1 intervals, in their
// order: two (odd and even wave numbers), or four (H = n_e / 2):
//   0: odd k at odd places, k < ceil(H / 2)    1: odd k at even places
//   2: k = 2, 6, 10, ..                         3: k = 4, 8, 12, ..
struct Fold {
  int N, H, h1, ho, he;
  bool four;
  __host__ __device__ Fold(int nx, int parts)
      : N(nx + 1), H(N / 2), h1(H / 2), ho((nx + 1) / 2), he(nx / 2), four(parts == 4) {}
  __host__ __device__ int len(int p) const {
    if (!four) return p ? he : ho;
    return p == 0 ? H - h1 : p == 3 ? H - h1 - 1 : h1;
  }
  // space index (from 1) and wave number behind entry (j, k) of part p
  __device__ int place(int p, int j) const { return !four || p >= 2 ? j + 1 : 2 * j + 1 + p; }
  __device__ int wave(int p, int k) const {
    if (!four) return 2 * k + 1 + p;
    return p < 2 ? 2 * k + 1 : 4 * k + 2 * (p - 1);
  }
  // wave number of spectral index a
  __device__ int wave_number(int a) const {
    if (a < ho) return 2 * a + 1;
    if (!four) return 2 * (a - ho) + 2;
    return a - H < h1 ? wave(2, a - H) : wave(3, a - H - h1);
  }
  // items of the input, up to four entries each
  __device__ int items(bool inv) const { return sine_items(N - 1, four ? 4 : 2, inv); }
  // entries (from 0) of item i; those that the item does not have repeat others
  template <bool INV>
  __device__ __forceinline__ void entries(int i, int (&e)[4]) const {
    if (!four) {
      const int m = min(i + (ho + 1) / 2, ho - 1);
      e[0] = i;
      e[1] = INV ? min(ho + i, N - 2) : N - 2 - i;
      e[2] = m;
      e[3] = INV ? min(ho + m, N - 2) : N - 2 - m;
    } else if (INV) {
      e[0] = i;
      e[1] = H - 1 - i;
      e[2] = H + i;
      e[3] = min(H + h1 + i, N - 2);
    } else {
      e[0] = i;
      e[1] = N - 2 - i;
      e[2] = H - 2 - i;
      e[3] = H + i;
    }
  }
  // item i with its entries' values x into the parts; get(e) for the entry in the middle
  template <bool INV, typename T, typename G, typename P>
  __device__ __forceinline__ void fold(int i, const T (&x)[4], G get, P put) const {
    if (!four) {
      auto two = [&](int k, T u, T v) {
        put(0, k, INV || k >= he ? u : u + v);
        if (k < he) put(1, k, INV ? v : u - v);
      };
      two(i, x[0], x[1]);
      if (i + (ho + 1) / 2 < ho) two(i + (ho + 1) / 2, x[2], x[3]);
    } else if (INV) {
      if (i < h1) {
        put(0, i, x[0] + x[1]);
        put(1, i, x[0] - x[1]);
        put(2, i, x[2]);
      } else {
        put(0, i, x[0]);
      }
      if (i < H - h1 - 1) put(3, i, x[3]);
    } else {
      const int j = i + 1, m = H - j;  // places
      const T v = x[0] - x[1];
      put(1 - (j & 1), i >> 1, x[0] + x[1]);
      if (m == j) {
        put(2, i, v);
      } else {
        const T w = x[2] - x[3];
        put(1 - (m & 1), (m - 1) >> 1, x[2] + x[3]);
        put(2, i, v + w);
        put(3, i, v - w);
      }
      if (j == h1) put(1 - (H & 1), (H - 1) >> 1, get(H - 1));
    }
  }
  // the entries of the result that item i's places in the parts, get(p, k), make up
  // (the items of the opposite direction's input)
  template <bool INV, typename G, typename P>
  __device__ __forceinline__ void unfold(int i, G get, P put) const {
    if (!four) {
      auto two = [&](int k) {
        const auto u = get(0, k);
        if (k >= he) {
          put(k, u);
        } else {
          const auto v = get(1, k);
          put(k, INV ? u + v : u);
          put(INV ? N - 2 - k : ho + k, INV ? u - v : v);
        }
      };
      two(i);
      if (i + (ho + 1) / 2 < ho) two(i + (ho + 1) / 2);
    } else if (!INV) {
      const auto u = get(0, i);
      if (i < h1) {
        const auto v = get(1, i);
        put(i, u + v);
        put(H - 1 - i, u - v);
        put(H + i, get(2, i));
      } else {
        put(i, u);
      }
      if (i < H - h1 - 1) put(H + h1 + i, get(3, i));
    } else {
      const int j = i + 1, m = H - j;  // places
      const auto u = get(1 - (j & 1), i >> 1), p = get(2, i);
      if (m == j) {
        put(i, u + p);
        put(N - 2 - i, u - p);
      } else {
        const auto q = get(3, i), t = get(1 - (m & 1), (m - 1) >> 1);
        const auto v = p + q, w = p - q;
        put(i, u + v);
        put(N - 2 - i, u - v);
        put(m - 1, t + w);
        put(H + i, t - w);
      }
      if (j == h1) put(H - 1, get(1 - (H & 1), (H - 1) >> 1));
    }
  }
};

// ---------------------------------------------------------------------------
// Tables
// ---------------------------------------------------------------------------

template <typename T>
__global__ void sine_pack_kernel(SineSizes z, int n_e, T* pack) {
  // pack order: forward parts, inverse parts
  const long total = 2 * z.parts * z.pack;
  const int steps = 4 * z.nq;
  const double scale = sqrt(2.0 / n_e);
  const Fold F(z.nx, z.parts);
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < total; i += (long)gridDim.x * blockDim.x) {
    const int which = (int)(i / z.pack);
    const long o = i % z.pack;
    const int lane = (int)(o % 64);
    const int step = (int)(o / 64 % steps), tile = (int)(o / 64 / steps);
    const int p = which % z.parts;
    int j = 4 * step + lane / 16, k = 16 * tile + lane % 16;  // place and wave within the part
    if (which >= z.parts) {
      const int u = j;
      j = k;
      k = u;
    }
    double v = 0.0;
    if (j < F.len(p) && k < F.len(p)) {
      const long m = (long)F.place(p, j) * F.wave(p, k) % (2L * n_e);
      v = scale * sinpi((double)m / n_e);
    }
    pack[i] = (T)v;
  }
}

__global__ void sine_tile_kernel(SineSizes z, int4* tiles) {
  const int nte = (z.he + 15) / 16;
  const long tri0 = (long)z.nt * (z.nt + 1) / 2, tri1 = (long)nte * (nte + 1) / 2;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < z.ntiles; i += (long)gridDim.x * blockDim.x) {
    int4 d = {0, 0, 0, 0};
    if (i < tri0 + tri1) {
      const bool even = i >= tri0;
      const int len = even ? nte : z.nt;
      long q = even ? i - tri0 : i;
      int I = 0;
      while (q >= len - I) q -= len - I++;
      const int J = I + (int)q, base = even ? z.ho : 0, end = even ? z.nx : z.ho;
      d = {base + 16 * I, base + 16 * J, end, end};
    } else if (i < tri0 + tri1 + (long)z.nt * nte) {
      const long q = i - tri0 - tri1;
      d = {16 * (int)(q / nte), z.ho + 16 * (int)(q % nte), z.ho, z.nx};
    }
    tiles[i] = d;
  }
}

// Row and column of a slot of a tile, and whether it holds a mode pair.
__device__ __forceinline__ bool slot_place(const int4& d, int in_tile, int& a, int& b) {
  a = d.x + (in_tile >> 4);
  b = d.y + (in_tile & 15);
  return a < d.z && b < d.w && a <= b;
}

__global__ void sine_slot_kernel(SineSizes z, SineConsts c, const int4* tiles, double* t, double* ipi) {
  const Fold F(z.nx, z.parts);
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < z.slots; i += (long)gridDim.x * blockDim.x) {
    int a, b;
    double tv = 0.0, iv = 0.0;
    if (slot_place(tiles[i / 256], (int)(i % 256), a, b)) {
      // eigenvalue of D^-1 K_0, (8 - 2 c_i - 2 c_j - 4 c_i c_j) / 8 with
      // c = cos(k pi / n_e), written through 1 - c = 2 sin^2(k pi / 2 n_e)
      const double si = sinpi(F.wave_number(a) / (2.0 * c.n_e)), sj = sinpi(F.wave_number(b) / (2.0 * c.n_e));
      const double ui = 2.0 * si * si, uj = 2.0 * sj * sj;
      const double mu = (6.0 * (ui + uj) - 4.0 * ui * uj) / 8.0;
      double S = 1.0 / c.diag, W = S * c.inv_theta, Z = W;
      for (int j = 1; j < c.degree; ++j) {
        S -= mu * W;
        W = c.chebA[j] * W + c.chebB[j] * S;
        Z += W;
      }
      tv = mu * c.diag * Z;
      iv = 1.0 / Z;
    }
    t[i] = tv;
    ipi[i] = iv;
  }
}

// ---------------------------------------------------------------------------
// Transform passes
// ---------------------------------------------------------------------------

constexpr int kPassThreads = 1024;

// What the first pass of a solve clears for the iteration that follows on the
// stream: the exchange places and tickets of its groups, and the status word.
struct SineReset {
  unsigned long long* ex;
  int nex;
  unsigned* tickets;
  int ntickets;
  int* status;  // null: nothing to clear
};

// Columns of several problems: the arrays of a ragged launch (listed columns
// only) and the tables of every problem.
enum { COL_B = 0, COL_X = 1, COL_S = 2, COL_S0 = 3, COL_W = 4 };
template <typename T>
struct SineRagged {
  PcgCols<T> cols;
  const SineTables<T>* tabs;
  __device__ __forceinline__ T* column(int which, int o) const {
    switch (which) {
      case COL_B: return const_cast<T*>(ld_uniform(cols.b, o));
      case COL_X: return ld_uniform(cols.x, o);
      case COL_S: return ld_uniform(cols.r0, o);
      case COL_S0: return ld_uniform(cols.r1, o);
      default: return ld_uniform(cols.z, o);
    }
  }
};

// Strip of block b of n: neighbours in an array go to one XCD (blocks are dealt to
// the eight in turn), whose L2 then holds the cache lines that they share.
__device__ __forceinline__ int xcd_block(int b, int n) {
  const int x = b & 7, q = n >> 3, r = n & 7;
  return x * q + min(x, r) + (b >> 3);
}

// The products of a block: item = a tile of 16 outputs of a pair of parts, IT items
// per wave of NB operand tiles each. The sine matrices come from L2, W steps at
// a time while the last W are multiplied; the first are on their way while the
// block folds its data.
template <typename T, int NB, int IT>
struct Products {
  using V = typename Mac<T>::V;
  int nq, pairs, items, wave, nw;
  const T* pack;
  static constexpr int W = 4;
  T w0[W], w1[W];

  __device__ __forceinline__ Products(int parts, int nq_, const T* pk)
      : nq(nq_),
        pairs(parts / 2),
        items(nq_ * (parts / 2)),
        wave(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)),
        nw(blockDim.x >> 6),
        pack(pk) {
    load(wave < items ? wave : 0, 0, threadIdx.x & 63, w0, w1);
  }
  __device__ __forceinline__ void load(int item, int chunk, int lane, T (&a)[W], T (&b)[W]) const {
    const T* f = pack + ((2 * (item % pairs) * nq + item / pairs) * nq * 4 + chunk * W) * 64;
    const T* g = f + nq * nq * 256;
#pragma unroll
    for (int k = 0; k < W; ++k) {
      a[k] = f[64 * k + lane];
      b[k] = g[64 * k + lane];
    }
  }
  // `tile` multiplies operand tile i of a part at step k, `result` takes the
  // products once every wave has read its operands
  template <typename L, typename S>
  __device__ __forceinline__ void run(L tile, S result) {
    const int lane = threadIdx.x & 63;
    V acc[IT][2][NB];
#pragma unroll
    for (int t = 0; t < IT; ++t)
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        acc[t][0][i] = V{0, 0, 0, 0};
        acc[t][1][i] = V{0, 0, 0, 0};
      }
#pragma unroll
    for (int t = 0; t < IT; ++t) {
      const int item = wave + t * nw;
      if (item >= items) continue;
      const int chunks = 4 / W * nq;
      const int p = 2 * (item % pairs);
      for (int c = 0; c < chunks; ++c) {
        T n0[W], n1[W];
        const bool last = c + 1 == chunks;
        load(last && IT > 1 && item + nw < items ? item + nw : item, last ? 0 : c + 1, lane, n0, n1);
#pragma unroll
        for (int k = 0; k < W; ++k)
#pragma unroll
          for (int i = 0; i < NB; ++i) {
            acc[t][0][i] = tile(w0[k], p, i, W * c + k, acc[t][0][i]);
            acc[t][1][i] = tile(w1[k], p + 1, i, W * c + k, acc[t][1][i]);
          }
#pragma unroll
        for (int k = 0; k < W; ++k) {
          w0[k] = n0[k];
          w1[k] = n1[k];
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < IT; ++t) {
      const int item = wave + t * nw;
      if (item >= items) continue;
      const int p = 2 * (item % pairs), ct = item / pairs;
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          result(p, ct, i, r, acc[t][0][i][r]);
          result(p + 1, ct, i, r, acc[t][1][i][r]);
        }
    }
    __syncthreads();
  }
};

// The passes are bound by memory and the matrix cores in turn (a block's loads,
// products and stores follow each other; two blocks fit a compute unit up to n_e =
// 256, one above). 220 columns of 255^2: 62 us a pass in FP64 (3.7 TB/s; 44 us for a
// copy, 28 us for the products alone), 35 us in FP32; 120 columns of 511^2: 245 us
// (97 us and 122 us). With two products per transform, unfolding from the registers
// and 128-byte stores it was 120 to 130, 60 to 80 and 610 us. A block's index
// arithmetic counts: with one element per step of the unfolding loop 255^2 took 75
// to 95 us. Blocks that load their next strip during the products gained nothing
// (75 to 95 us): the table's entries, asked for after it, return after it.
//
// Pass along x: a block folds 16 RT rows of nx values into the parts in LDS,
// multiplies them by the sine matrices from the right and unfolds the products,
// which take the operands' place.
// RAGGED: the launch covers columns of several problems, `strips` blocks each
// (as many as the largest grid needs; the blocks past a column's rows end).
template <typename T, bool INV, int RT, int IT, bool RAGGED>
__global__ __launch_bounds__(kPassThreads) void sine_x_kernel(SineTables<T> tab, const T* in, T* out, long rows,
                                                              SineReset reset, SineRagged<T> C, int from, int to,
                                                              int strips) {
  using M = Mac<T>;
  using V = typename M::V;
  extern __shared__ unsigned char smem[];
  if (!INV && blockIdx.x == 0 && reset.status) {
    for (int i = threadIdx.x; i < reset.nex; i += blockDim.x) reset.ex[i] = kEmpty;
    for (int i = threadIdx.x; i < reset.ntickets; i += blockDim.x) reset.tickets[i] = 0u;
    if (threadIdx.x == 0) *reset.status = 0;
  }
  long strip = RAGGED ? blockIdx.x : xcd_block(blockIdx.x, gridDim.x);
  if constexpr (RAGGED) {
    const int i = blockIdx.x / strips;
    if (i >= ld_uniform(C.cols.nact, 0)) return;
    const int o = ld_uniform(C.cols.act, i);
    strip -= (long)i * strips;
    tab = C.tabs[ld_uniform(C.cols.prob, o)];
    if (strip * 16 * RT >= tab.nx) return;
    rows = tab.nx;
    in = C.column(from, o);
    out = C.column(to, o);
  }
  const int nx = tab.nx, parts = tab.parts, nq = tab.nq, hq = 16 * nq;
  constexpr int R = 16 * RT, PAD = 16 / sizeof(T);  // rows of an operand fall into different LDS banks
  const int ld = hq + PAD;
  T* Q = reinterpret_cast<T*>(smem);  // [parts][R][ld], each part half the banks further
  auto base = [&](int p) { return p * (R * ld + 128 / (int)sizeof(T)); };
  const Fold F(nx, parts);
  const int t = threadIdx.x, lane = t & 63;
  // this thread's u-th place in (rows x items): as many lanes to a row as it has items, in powers of two
  auto mine = [&](int items, int u, int& r, int& i) {
    const int llog = sine_lane_log(items);
    const int rstep = blockDim.x >> llog, rper = max(1, R / rstep), chunk = u / rper;
    r = (t >> llog) + (u - chunk * rper) * rstep;
    i = (t & ((1 << llog) - 1)) + (chunk << llog);
    return r < R && i < items;
  };
  const long r0 = strip * R;
  Products<T, RT, IT> products(parts, nq, INV ? tab.inv : tab.fwd);
  {
    T x[kPassBatch][4];
    const int items = F.items(INV);
    auto source = [&](int r) { return in + min(r0 + r, rows - 1) * nx; };  // rows past the end are not stored
#pragma unroll
    for (int u = 0; u < kPassBatch; ++u) {
      int r, i, e[4];
      if (!mine(items, u, r, i)) continue;
      F.template entries<INV>(i, e);
      const T* src = source(r);
#pragma unroll
      for (int k = 0; k < 4; ++k) x[u][k] = src[e[k]];
    }
    for (int r = t >> 4; r < R; r += blockDim.x >> 4)
      for (int p = 0; p < parts; ++p)
        for (int j = F.len(p) + (t & 15); j < hq; j += 16) Q[base(p) + r * ld + j] = T(0);
#pragma unroll
    for (int u = 0; u < kPassBatch; ++u) {
      int r, i;
      if (!mine(items, u, r, i)) continue;
      F.template fold<INV>(
          i, x[u], [&](int m) { return source(r)[m]; }, [&](int p, int j, T v) { Q[base(p) + r * ld + j] = v; });
    }
  }
  __syncthreads();
  const T* q = Q + (lane & 15) * ld + (lane >> 4);
  products.run([&](T w, int p, int i, int k, V a) { return M::mac(q[base(p) + 16 * i * ld + 4 * k], w, a); },
               [&](int p, int ct, int i, int r, T v) {
                 Q[base(p) + (16 * i + M::row(lane, r)) * ld + 16 * ct + (lane & 15)] = v;
               });
  const int outs = F.items(!INV);
#pragma unroll
  for (int u = 0; u < kPassBatch; ++u) {
    int r, i;
    if (!mine(outs, u, r, i) || r0 + r >= rows) continue;
    T* dst = out + (r0 + r) * nx;
    const T* g = Q + r * ld;
    F.template unfold<INV>(
        i, [&](int p, int k) { return g[base(p) + k]; }, [&](int e, T v) { dst[e] = v; });
  }
}

// Pass along y of one column's nx x nx array: a block takes CW = 16 CT array
// columns, folds their rows into the parts in LDS, multiplies by the sine
// matrices from the left and unfolds the products. With 32 columns the two halves
// of every other row (pair of rows in FP32) are exchanged, so that the four rows
// of a matrix operand fall into different LDS banks.
template <typename T, bool INV, int CT, int IT, bool RAGGED>
__global__ __launch_bounds__(kPassThreads) void sine_y_kernel(SineTables<T> tab, const T* in, T* out, long n,
                                                              SineRagged<T> C, int from, int to, int strips) {
  using M = Mac<T>;
  using V = typename M::V;
  extern __shared__ unsigned char smem[];
  int strip = RAGGED ? blockIdx.x : xcd_block(blockIdx.x, gridDim.x);
  const int col = strip / strips;
  strip -= col * strips;
  if constexpr (RAGGED) {
    if (col >= ld_uniform(C.cols.nact, 0)) return;
    const int o = ld_uniform(C.cols.act, col);
    tab = C.tabs[ld_uniform(C.cols.prob, o)];
    if (strip * 16 * CT >= tab.nx) return;
    in = C.column(from, o);
    out = C.column(to, o);
  } else {
    in += (long)col * n;
    out += (long)col * n;
  }
  const int nx = tab.nx, parts = tab.parts, nq = tab.nq, hq = 16 * nq;
  constexpr int CW = 16 * CT;
  T* Q = reinterpret_cast<T*>(smem);  // [parts][hq][CW]
  const Fold F(nx, parts);
  constexpr int SH = sizeof(T) == 4 ? 1 : 0;
  auto place = [&](int p, int j, int c) { return (p * hq + j) * CW + (CT == 2 ? c ^ (((j >> SH) & 1) << 4) : c); };
  const int c = threadIdx.x % CW, l0 = threadIdx.x / CW, lstep = blockDim.x / CW, at = strip * CW + c;
  const int lane = threadIdx.x & 63;
  Products<T, CT, IT> products(parts, nq, INV ? tab.inv : tab.fwd);
  {
    T x[kPassBatch][4];
    const int items = F.items(INV);
    const T* src = in + min(at, nx - 1);  // columns past the end are not stored
#pragma unroll
    for (int u = 0; u < kPassBatch; ++u) {
      const int i = l0 + u * lstep;
      int e[4];
      if (i >= items) continue;
      F.template entries<INV>(i, e);
#pragma unroll
      for (int k = 0; k < 4; ++k) x[u][k] = src[e[k] * nx];
    }
    for (int p = 0; p < parts; ++p)
      for (int j = F.len(p) + l0; j < hq; j += lstep) Q[place(p, j, c)] = T(0);
#pragma unroll
    for (int u = 0; u < kPassBatch; ++u) {
      const int i = l0 + u * lstep;
      if (i >= items) continue;
      F.template fold<INV>(
          i, x[u], [&](int m) { return src[m * nx]; }, [&](int p, int j, T v) { Q[place(p, j, c)] = v; });
    }
  }
  __syncthreads();
  products.run(
      [&](T w, int p, int i, int k, V a) {
        return M::mac(w, Q[place(p, 4 * k + (lane >> 4), 16 * i + (lane & 15))], a);
      },
      [&](int p, int rt, int i, int r, T v) { Q[place(p, 16 * rt + M::row(lane, r), 16 * i + (lane & 15))] = v; });
  const int outs = F.items(!INV);
  if (at < nx)
#pragma unroll
    for (int u = 0; u < kPassBatch; ++u)
      if (l0 + u * lstep < outs)
        F.template unfold<INV>(
            l0 + u * lstep, [&](int p, int k) { return Q[place(p, k, c)]; },
            [&](int e, T v) { out[e * nx + at] = v; });
}

// ---------------------------------------------------------------------------
// Transforms inside a block
// ---------------------------------------------------------------------------

// Where entry q of part p lies in a vector of nx places that is folded in place:
// first + q step.
__device__ __forceinline__ void in_place(const Fold& F, bool inv, int p, int& first, int& step) {
  step = 1;
  if (!F.four) {
    first = p == 0 ? 0 : inv ? F.ho : F.N - 2;
    if (p == 1 && !inv) step = -1;
  } else if (inv) {
    first = p == 0 ? 0 : p == 1 ? F.H - 1 : p == 2 ? F.H : F.H + F.h1;
    if (p == 1) step = -1;
  } else {
    first = p < 2 ? p : p == 2 ? F.N - 2 : F.H;
    step = p < 2 ? 2 : p == 2 ? -1 : 1;
  }
}

constexpr int kFusedSlots = 2;  // pairs of products a wave holds: two products of two tiles or four of one

// Between the lanes of a wave that exchange data through LDS: what they wrote before
// is there for each other after it, and nothing they still read is written before it.
// The hardware takes a wave's LDS accesses in their order, so this costs no instruction;
// it holds the compiler, which sees one lane's places only, to that order.
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// One direction of a transform of the nx x nx array D in LDS, in place: this
// wave's 16 lines (rows along x, ALONG_X; columns along y), which no other wave
// touches meanwhile. at(line, place) is an element of a line; lines past the end
// hold whatever LDS holds and reach no other line.
template <typename T, bool INV, bool ALONG_X, typename At>
__device__ __forceinline__ void line_transform(const Fold& F, int nq, const T* pack, At at) {
  using M = Mac<T>;
  using V = typename M::V;
  // not known to be the same in every call: addresses are computed again instead of being kept
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  const int line = lane & 15, sub = lane >> 4, nx = F.N - 1;
  // slot t takes tile t of the pair (two products) or the tile of pair t
  const int pairs = F.four ? 2 : 1, steps = 4 * nq, part = nq * steps * 64;
  V acc[kFusedSlots][2];
  const T* f[kFusedSlots];
  bool on[kFusedSlots];
#pragma unroll
  for (int t = 0; t < kFusedSlots; ++t) {
    const int pr = F.four ? t : 0, ct = F.four ? 0 : t;
    on[t] = ct < nq;
    f[t] = pack + (2 * pr * nq + ct) * steps * 64;
    acc[t][0] = V{0, 0, 0, 0};
    acc[t][1] = V{0, 0, 0, 0};
  }
  int first[4], step[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) in_place(F, INV, p < 2 * pairs ? p : 0, first[p], step[p]);
  T n0[kFusedSlots], n1[kFusedSlots];
  auto load = [&](int k) {
#pragma unroll
    for (int t = 0; t < kFusedSlots; ++t)
      if (on[t]) {
        n0[t] = f[t][64 * k + lane];
        n1[t] = f[t][part + 64 * k + lane];
      }
  };
  load(0);  // on its way while the lines are folded
  wave_fence();
  // fold
  if (!INV) {
    for (int i = sub; i < F.items(false); i += 4) {
      int e[4];
      F.template entries<false>(i, e);
      T x[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) x[k] = *at(line, e[k]);
      if (F.four) {
        const T v = x[0] - x[1], w = x[2] - x[3];
        const bool mid = e[2] == e[0];
        *at(line, e[0]) = x[0] + x[1];
        *at(line, e[1]) = mid ? v : v + w;
        if (!mid) {
          *at(line, e[2]) = x[2] + x[3];
          *at(line, e[3]) = v - w;
        }
      } else {
        if (e[0] < F.he) {
          *at(line, e[0]) = x[0] + x[1];
          *at(line, e[1]) = x[0] - x[1];
        }
        if (i + (F.ho + 1) / 2 < F.he) {
          *at(line, e[2]) = x[2] + x[3];
          *at(line, e[3]) = x[2] - x[3];
        }
      }
    }
  } else if (F.four) {
    for (int i = sub; i < F.h1; i += 4) {
      const T u = *at(line, i), m = *at(line, F.H - 1 - i);
      *at(line, i) = u + m;
      *at(line, F.H - 1 - i) = u - m;
    }
  }
  wave_fence();
  // products
  for (int k = 0; k < steps; ++k) {
    T w0[kFusedSlots], w1[kFusedSlots], x[4];
#pragma unroll
    for (int t = 0; t < kFusedSlots; ++t) {
      w0[t] = n0[t];
      w1[t] = n1[t];
    }
    if (k + 1 < steps) load(k + 1);
    // entries past a part's length meet zeros of the matrix: any place of the line will do
#pragma unroll
    for (int p = 0; p < 4; ++p)
      if (p < 2 * pairs) x[p] = *at(line, min(max(first[p] + (4 * k + sub) * step[p], 0), nx - 1));
#pragma unroll
    for (int t = 0; t < kFusedSlots; ++t)
      if (on[t]) {
        const T x0 = t == 1 && F.four ? x[2] : x[0], x1 = t == 1 && F.four ? x[3] : x[1];
        acc[t][0] = ALONG_X ? M::mac(x0, w0[t], acc[t][0]) : M::mac(w0[t], x0, acc[t][0]);
        acc[t][1] = ALONG_X ? M::mac(x1, w1[t], acc[t][1]) : M::mac(w1[t], x1, acc[t][1]);
      }
  }
  wave_fence();
  // unfold: the products of a pair meet in a lane
#pragma unroll
  for (int t = 0; t < kFusedSlots; ++t) {
    if (!on[t]) continue;
    const int pr = F.four ? t : 0, ct = F.four ? 0 : t;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int ln = ALONG_X ? M::row(lane, r) : line;
      const int k = 16 * ct + (ALONG_X ? line : M::row(lane, r));
      const T u = acc[t][0][r], v = acc[t][1][r];
      auto put = [&](int e, T y) { *at(ln, e) = y; };
      if (!F.four) {
        if (k < F.ho) put(k, u);
        if (k < F.he) put(INV ? F.N - 2 - k : F.ho + k, v);
      } else if (!INV && pr == 0) {
        if (k < F.h1) {
          put(k, u + v);
          put(F.H - 1 - k, u - v);
        } else if (k < F.H - F.h1) {
          put(k, u);
        }
      } else if (!INV) {
        if (k < F.h1) put(F.H + k, u);
        if (k < F.H - F.h1 - 1) put(F.H + F.h1 + k, v);
      } else if (pr == 0) {
        if (k < F.H - F.h1) put(2 * k, u);
        if (k < F.h1) put(2 * k + 1, v);
      } else if (k < F.H - F.h1 - 1) {
        put(F.N - 2 - k, u + v);
        put(F.H + k, u - v);
      } else if (k < F.h1) {
        put(F.N - 2 - k, u);
      }
    }
  }
  if (INV) {
    wave_fence();
    for (int i = sub; i < F.he; i += 4) {
      const T u = *at(line, i), v = *at(line, F.N - 2 - i);
      *at(line, i) = u + v;
      *at(line, F.N - 2 - i) = u - v;
    }
  }
}

// Both directions on one column of at most 64 rows, src to dst through LDS. A wave
// takes 16 rows, then 16 columns, so the block meets only in between.
template <typename T, bool INV>
__device__ __forceinline__ void column_transform(int nx, int parts, int nq, const T* pack, const T* src, T* dst,
                                                 T* D) {
  nx = __builtin_amdgcn_readfirstlane(nx);
  asm volatile("" : "+s"(nx));
  const Fold F(nx, parts);
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nr = (nx + 15) / 16, ld = 16 * nr + 16 / (int)sizeof(T);
  if (wave < nr) {
    const int r1 = min(16, nx - 16 * wave);
    T* d = D + 16 * wave * ld;
    const T* s = src + 16 * wave * nx;
    for (int c = lane; c < nx; c += 64)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (r < r1) d[r * ld + c] = s[r * nx + c];
    line_transform<T, INV, true>(F, nq, pack, [&](int r, int c) { return d + r * ld + c; });
  }
  __syncthreads();
  if (wave < nr) {
    T* d = D + 16 * wave;
    line_transform<T, INV, false>(F, nq, pack, [&](int c, int r) { return d + r * ld + c; });
  }
  __syncthreads();
  for (int r = wave; r < nx; r += blockDim.x >> 6)
    for (int c = lane; c < nx; c += 64) dst[r * nx + c] = D[r * ld + c];
  __syncthreads();
}

// ---------------------------------------------------------------------------
// Iteration
// ---------------------------------------------------------------------------

// Half sums of two values at once: lanes 0..31 get a of lanes l and l + 32, lanes
// 32..63 the same of b (fold32); or rows 0 and 2 of a, rows 1 and 3 of b (fold16).
// Seven adds sum four values over a wave, against 24 for one after the other.
__device__ __forceinline__ double fold32(double a, double b) {
  const uint2 ua = __builtin_bit_cast(uint2, a), ub = __builtin_bit_cast(uint2, b);
  const auto lo = __builtin_amdgcn_permlane32_swap(ua.x, ub.x, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(ua.y, ub.y, false, false);
  return __builtin_bit_cast(double, make_uint2(lo[0], hi[0])) + __builtin_bit_cast(double, make_uint2(lo[1], hi[1]));
}
__device__ __forceinline__ double fold16(double a, double b) {
  const uint2 ua = __builtin_bit_cast(uint2, a), ub = __builtin_bit_cast(uint2, b);
  const auto lo = __builtin_amdgcn_permlane16_swap(ua.x, ub.x, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(ua.y, ub.y, false, false);
  return __builtin_bit_cast(double, make_uint2(lo[0], hi[0])) + __builtin_bit_cast(double, make_uint2(lo[1], hi[1]));
}

// Sums over a column: the block's threads, then the blocks of its group (in
// a fixed order), the same bits in every thread of the group. A group
// of one block needs its own barrier only. Otherwise the blocks exchange their
// sums through places that are empty until a value is there. Three exchange
// buffers take turns. Passing the wait of one exchange means that every block has read
// the one before it, so a block clears its places of that one, waits until the
// stores are done and only then publishes again: nobody finds an old value.
// The wait is bounded and ends the launch with an error status.
struct ColumnSums {
  double (*red)[kSineThreads / 64][kSumWidth];  // two buffers, used in turn
  double (*all)[kSumWidth];                     // group sums, two buffers
  unsigned long long* ex;                       // the group's exchange [3][groups][kSumWidth]
  int* status;
  int* sflag;
  int groups, g;
  unsigned epoch;
  bool dead;

  __device__ unsigned long long* slot(unsigned e, int k) const { return ex + ((long)(e % 3) * groups + k) * kSumWidth; }

  __device__ __forceinline__ void sum(double (&v)[kSumWidth]) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, row = lane >> 4;
    double (*buf)[kSumWidth] = red[epoch & 1];
    // row i of the lanes ends up with sum i of the wave
    double t = fold16(fold32(v[0], v[2]), fold32(v[1], v[3]));
    t += dpp_f64<0x128>(t);  // row_ror:8
    t += dpp_f64<0x124>(t);  // row_ror:4
    t += dpp_f64<0x122>(t);  // row_ror:2
    t += dpp_f64<0x121>(t);  // row_ror:1
    // before the branch (sunk past it, the adds would keep every slot's terms alive)
    asm volatile("" ::"v"(t));
    if ((lane & 15) == 0) buf[wv][row] = t;
    __syncthreads();
    // lane w (and w + 8) of row i holds sum i of wave w
    t = buf[lane & 7][row];
    t += dpp_f64<0x124>(t);
    t += dpp_f64<0x122>(t);
    t += dpp_f64<0x121>(t);
    if (groups == 1) {
#pragma unroll
      for (int i = 0; i < kSumWidth; ++i) v[i] = lane_f64(t, 16 * i);
      ++epoch;
      return;
    }
    double (*out)[kSumWidth] = all + (epoch & 1);
    if (wv == 0) {
      // row i publishes sum i; then its lanes read the places of 16 blocks at a time
      if ((lane & 15) == 0) {
        __builtin_amdgcn_s_waitcnt(0);  // this lane's clearing store of the last exchange is done
        agent_store(slot(epoch, g) + row, publishable(t));
      }
      double s = 0.0;
      int ok = dead ? 0 : 1;
      for (int k0 = 0; k0 < groups; k0 += 16) {
        const int k = k0 + (lane & 15);
        unsigned long long bits = 0;
        if (k < groups) {
          const unsigned long long* src = slot(epoch, k) + row;
          long spins = 0;
          while ((bits = agent_load(src)) == kEmpty && ok) {
            __builtin_amdgcn_s_sleep(1);
            if (++spins > kSpinLimit) ok = 0;
          }
        }
        double val = __longlong_as_double((long long)bits);
        val += dpp_f64<0x128>(val);
        val += dpp_f64<0x124>(val);
        val += dpp_f64<0x122>(val);
        val += dpp_f64<0x121>(val);
        s += val;
      }
      ok = __all(ok);
      if (!ok && lane == 0) __hip_atomic_store(status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      if ((lane & 15) == 0) {
        (*out)[row] = s;
        if (epoch > 0) agent_store(slot(epoch + 2, g) + row, kEmpty);  // the place of exchange epoch - 1
      }
      if (lane == 0) *sflag = ok;
    }
    __syncthreads();
    if (*sflag == 0) dead = true;
#pragma unroll
    for (int i = 0; i < kSumWidth; ++i) v[i] = lane_f64((*out)[i], 0);
    ++epoch;
  }
};

// One column at a time per group of blocks. Every slot keeps, for its pair of
// modes, rho = the residual polynomial and phi = the direction polynomial at
// the pair's eigenvalue (r = rho r_0, p = pi phi r_0 with pi the factor of the
// preconditioner). With the weight w = the sum of the pair's r_0^2
//   r.z = sum v rho^2,  r.r = sum v rho^2 / pi,  p.q = sum v t phi^2,
// v = pi w and t the eigenvalue of M K_0: one multiple of r_0 per pair stands
// for all vectors of the iteration. p.q of the next direction p' = z + beta p is
// z.K z + 2 beta z.K p + beta^2 p.q, so a single pass over the slots makes an
// iteration (its rounding error is that of the three terms, at most cond(M K_0)
// times p'.q'). All of a block's slots stay in registers (1 / pi and, beyond 11
// slots a thread, what of t fits in LDS; of 27 slots 5 or 6 registers spill). Slots
// without a mode have v = 0 and t = 0.
// Bound by the chain of an iteration: the arithmetic (about 0.8 us on 23 slots a
// thread), the sums over the block (0.3 us) and across the group (1.2 us), so a
// launch of many columns is faster the fewer blocks a column takes: as many slots
// as the registers hold, without a solution vector (x follows from rho). 255^2,
// three blocks of 23 slots a thread: 2.4 us an iteration; the 220 columns of a large
// launch go through 85 groups in three turns, 7.2 us per iteration of all (10.4 us
// with xi = sum alpha phi in registers too, 18 slots and four blocks a column; 23.4
// us with one block a column that streams v, t and 1 / pi). 511^2, 120 columns:
// 13.7 us, ten blocks of 27 slots (22.9 us, fifteen of 18).
// FUSED: columns of at most kSineFusedNx rows, transformed here too.
// RAGGED: the listed columns of several problems; those whose tables have other
// slot and block counts than this launch are left to the launches for theirs.
constexpr int sine_t_regs(int nr) {
  constexpr int arrays = 39;  // of a value per thread, 156 KB
  return nr <= 11 ? nr : 2 * nr > arrays ? 2 * nr - arrays : 0;
}
template <typename T, int NR, bool RAGGED, bool FUSED>
__global__ __launch_bounds__(kSineThreads, FUSED ? 4 : 1) void sine_pcg_kernel(SineArgs<T> A, SineRagged<T> C, int ngroups) {
  constexpr int TR = sine_t_regs(NR);  // slots whose t is in registers
  extern __shared__ unsigned char smem[];
  __shared__ double red[2][kSineThreads / 64][kSumWidth], all[2][kSumWidth];
  __shared__ int sflag;
  const int tid = threadIdx.x;
  const int G = FUSED ? 1 : A.tab.groups;
  // The blocks of a group wait for each other, so groups form in the order in
  // which blocks start: whatever else holds compute units, at most one group of
  // a launch is incomplete, and the complete ones run to their end.
  int place_ = blockIdx.x;
  if (G > 1) {
    if (tid == 0) sflag = (int)atomicAdd(A.sc.arrivals, 1u);
    __syncthreads();
    place_ = __builtin_amdgcn_readfirstlane(sflag);
    __syncthreads();
  }
  const int group = place_ / G, g = place_ - group * G;
  const int sbase = g * NR * kSineThreads;  // this block's first slot
  const int lane_ = tid & 63, w0 = __builtin_amdgcn_readfirstlane(tid >> 6) * NR;
  int nx = A.tab.nx;
  const int4* tiles;
  const double *tt, *ip;
  double* lds = reinterpret_cast<double*>(smem) + tid;
  ColumnSums cs{red, all, reinterpret_cast<unsigned long long*>(A.sc.part) + (long)group * G * 3 * kSumWidth,
                A.sc.status, &sflag, G, g, 0u, false};
  const int ncols = RAGGED ? ld_uniform(C.cols.nact, 0) : A.ncols;
  if (FUSED && blockIdx.x == 0 && tid == 0) *A.sc.status = 0;
  for (int c = group; c < ncols; c += ngroups) {
    T* s = A.s + (long)c * A.n;
    const T* s0 = A.s0 + (long)c * A.n;
    int lane = lane_;
    asm volatile("" : "+v"(lane));  // no address below is kept from one column to the next
    tiles = A.tab.tiles + sbase / 256;
    tt = A.tab.t + sbase + w0 * 64 + lane;  // element e at 64 e
    ip = A.tab.ipi + sbase + w0 * 64 + lane;
    if constexpr (RAGGED) {
      const int o = ld_uniform(C.cols.act, c);
      const SineTables<T>& tab = C.tabs[ld_uniform(C.cols.prob, o)];
      if (tab.ept != NR || tab.groups != G) continue;
      nx = tab.nx;
      tiles = tab.tiles + sbase / 256;
      tt = tab.t + sbase + w0 * 64 + lane;
      ip = tab.ipi + sbase + w0 * 64 + lane;
      s = C.column(COL_S, o);
      s0 = C.column(COL_S0, o);
    }
    if constexpr (FUSED) {
      T* D = reinterpret_cast<T*>(smem);
      column_transform<T, false>(nx, A.tab.parts, A.tab.nq, A.tab.fwd, A.b + (long)c * A.n, s, D);
      if (A.warm)
        column_transform<T, false>(nx, A.tab.parts, A.tab.nq, A.tab.fwd, A.x + (long)c * A.n, const_cast<T*>(s0), D);
    }
    // row and column of element e (its 64 slots are a quarter of a tile)
    auto place = [&](int e, int& a, int& b) {
      return slot_place(tiles[(w0 + e) >> 2], ((w0 + e) & 3) * 64 + lane, a, b);
    };
    // ---- start: weights, b.b, r.r, r.z, z.K z (warm: r = b - K_0 x in place)
    double sums[kSumWidth] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
    for (int e = 0; e < NR; ++e) {
      int a, b;
      const double iv = ip[64 * e];
      double v = 0.0;
      if (place(e, a, b)) {
        const long i1 = (long)a * nx + b, i2 = (long)b * nx + a;
        double b1 = s[i1], b2 = a == b ? 0.0 : (double)s[i2];
        sums[0] += b1 * b1 + b2 * b2;
        const double tv = tt[64 * e];
        if (A.warm) {
          const double kap = tv * iv;
          b1 -= kap * s0[i1];
          s[i1] = (T)b1;
          if (a != b) {
            b2 -= kap * s0[i2];
            s[i2] = (T)b2;
          }
        }
        const double w = b1 * b1 + b2 * b2;
        v = w / iv;
        sums[1] += w;
        sums[2] += v;
        sums[3] = fma(v, tv, sums[3]);
      }
      lds[e * kSineThreads] = v;
    }
    double rho[NR], phi[NR], rv[NR], rt[TR > 0 ? TR : 1];
#pragma unroll
    for (int e = 0; e < NR; ++e) {
      if (e % 4 == 0) __builtin_amdgcn_sched_barrier(0);
      rv[e] = lds[e * kSineThreads];
      rho[e] = 1.0;  // v = t = 0 where there is no mode
      phi[e] = 0.0;
      lds[e * kSineThreads] = ip[64 * e];
      if (e < TR) rt[e < TR ? e : 0] = tt[64 * e];
      else lds[(NR - TR + e) * kSineThreads] = tt[64 * e];
    }
    cs.sum(sums);
    const double bb = sums[0];
    double rr = sums[1], rz = sums[2], pq = sums[3], beta = 0.0;
    int it = 0;
    for (;; ++it) {
      if (cs.dead || it == A.maxit || bb == 0.0 || sqrt(rr) <= A.rtol * sqrt(bb)) break;
      if (!(pq > 0.0) || !isfinite(pq)) break;  // breakdown: the iterate so far
      const double alpha = rz / pq;
      // p = z + beta p, r -= alpha q, and the sums r.r, r.z, z.K z, z.K p of the new residual
      double q[kSumWidth] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int e = 0; e < NR; ++e) {
        if (e % 2 == 0) __builtin_amdgcn_sched_barrier(0);  // the LDS reads of two slots at a time
        const double iv = lds[e * kSineThreads], tv = e < TR ? rt[e < TR ? e : 0] : lds[(NR - TR + e) * kSineThreads];
        phi[e] = fma(beta, phi[e], rho[e]);
        rho[e] = fma(-alpha * phi[e], tv, rho[e]);
        const double vr = rv[e] * rho[e], z = vr * rho[e];
        q[1] += z;
        q[0] = fma(z, iv, q[0]);
        q[2] = fma(z, tv, q[2]);
        q[3] = fma(vr * tv, phi[e], q[3]);
      }
      cs.sum(q);
      beta = q[1] / rz;
      pq = fma(beta, fma(beta, pq, 2.0 * q[3]), q[2]);
      rr = q[0];
      rz = q[1];
    }
    if (tid == 0 && g == 0) A.sc.iters[c] = it;
    // ---- solution: x = x_0 + K_0^-1 (r_0 - r) = x_0 + (1 - rho) / (t / pi) r_0, to the rounding
    // of x's exact value (a zero right-hand side gives 0 also from a warm start)
    const bool guess = A.warm && bb != 0.0;
#pragma unroll
    for (int e = 0; e < NR; ++e) lds[e * kSineThreads] = 1.0 - rho[e];
#pragma unroll 2
    for (int e = 0; e < NR; ++e) {
      int a, b;
      if (!place(e, a, b)) continue;
      const double m = lds[e * kSineThreads] / (tt[64 * e] * ip[64 * e]);
      const long i1 = (long)a * nx + b, i2 = (long)b * nx + a;
      double x1 = guess ? (double)s0[i1] : 0.0, x2 = guess ? (double)s0[i2] : 0.0;
      if (it > 0) {
        x1 = fma(m, (double)s[i1], x1);
        x2 = fma(m, (double)s[i2], x2);
      }
      s[i1] = (T)x1;
      if (a != b) s[i2] = (T)x2;
    }
    if constexpr (FUSED) {
      __syncthreads();
      column_transform<T, true>(nx, A.tab.parts, A.tab.nq, A.tab.inv, s, A.x + (long)c * A.n,
                                reinterpret_cast<T*>(smem));
    }
  }
}

template <typename K>
hipError_t allow_lds(K kfn, size_t bytes) {
  if (bytes <= 64 * 1024) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kfn), hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)bytes);
}

template <typename T>
const T* column_base(const SineArgs<T>& A, int which) {
  return which == COL_B ? A.b : which == COL_X ? A.x : which == COL_S ? A.s : which == COL_S0 ? A.s0 : A.w;
}

// The variant for strips of 32 or 16 lines and one or two product items a wave; refuses
// a shape that the kernels do not provide for.
template <typename T, typename F1, typename F2, typename F3>
hipError_t pass_variant(const SinePass& sh, int nx, int parts, long all, int num_cu, F1 wide, F2 narrow, F3 longest) {
  const int lines = sh.lines(all, num_cu);
  if (!sh.served(nx, parts, lines, sizeof(T))) return hipErrorInvalidValue;
  return sh.per_wave() == 2 ? longest(lines) : lines == 32 ? wide(lines) : narrow(lines);
}

// One pass over every column: `nx` the longest transform, C the columns of a ragged launch.
template <typename T, bool INV, bool RAGGED>
hipError_t x_pass(const SineArgs<T>& A, const SineRagged<T>& C, int nx, int from, int to, const SineReset& reset,
                  int num_cu, hipStream_t s) {
  const SinePass sh(nx, RAGGED);
  const long rows = (long)A.ncols * nx;
  const T* in = RAGGED ? nullptr : column_base(A, from);
  T* out = RAGGED ? nullptr : const_cast<T*>(column_base(A, to));
  auto launch = [&](auto kfn, int R) {
    const size_t sm = sh.lds(sizeof(T), R);
    const hipError_t e = allow_lds(kfn, sm);
    if (e != hipSuccess) return e;
    const int strips = (nx + R - 1) / R;
    const unsigned blocks = RAGGED ? (unsigned)A.ncols * strips : (unsigned)((rows + R - 1) / R);
    hipLaunchKernelGGL(kfn, dim3(blocks), dim3(sh.threads()), sm, s, A.tab, in, out, rows, reset, C, from,
                       to, strips);
    return hipGetLastError();
  };
  return pass_variant<T>(
      sh, nx, sine_sizes(nx).parts, rows, num_cu, [&](int R) { return launch(sine_x_kernel<T, INV, 2, 1, RAGGED>, R); },
      [&](int R) { return launch(sine_x_kernel<T, INV, 1, 1, RAGGED>, R); },
      [&](int R) { return launch(sine_x_kernel<T, INV, 1, 2, RAGGED>, R); });
}

template <typename T, bool INV, bool RAGGED>
hipError_t y_pass(const SineArgs<T>& A, const SineRagged<T>& C, int nx, int from, int to, int num_cu, hipStream_t s) {
  const SinePass sh(nx, RAGGED);
  const T* in = RAGGED ? nullptr : column_base(A, from);
  T* out = RAGGED ? nullptr : const_cast<T*>(column_base(A, to));
  auto launch = [&](auto kfn, int W) {
    const size_t sm = sh.lds(sizeof(T), W);
    const hipError_t e = allow_lds(kfn, sm);
    if (e != hipSuccess) return e;
    const int strips = (nx + W - 1) / W;
    hipLaunchKernelGGL(kfn, dim3((unsigned)strips * A.ncols), dim3(sh.threads()), sm, s, A.tab, in, out, A.n, C, from,
                       to, strips);
    return hipGetLastError();
  };
  return pass_variant<T>(
      sh, nx, sine_sizes(nx).parts, (long)A.ncols * nx, num_cu,
      [&](int W) { return launch(sine_y_kernel<T, INV, 2, 1, RAGGED>, W); },
      [&](int W) { return launch(sine_y_kernel<T, INV, 1, 1, RAGGED>, W); },
      [&](int W) { return launch(sine_y_kernel<T, INV, 1, 2, RAGGED>, W); });
}

template <typename T, bool RAGGED, bool FUSED>
hipError_t pcg(const SineArgs<T>& A, const SineRagged<T>& C, int ngroups, hipStream_t s) {
  auto launch = [&](auto kfn, int nr) {
    size_t sm = sizeof(double) * kSineThreads * (2 * nr - sine_t_regs(nr));
    if (FUSED) {  // the longest column of that many slots, in tiles
      const int rows = nr == 2 ? 32 : 64;
      sm = std::max(sm, sizeof(T) * rows * (rows + 16 / sizeof(T)));
    }
    const hipError_t e = allow_lds(kfn, sm);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kfn, dim3((unsigned)(ngroups * A.tab.groups)), dim3(kSineThreads), sm, s, A, C, ngroups);
    return hipGetLastError();
  };
  switch (A.tab.ept) {
    case 2: return launch(sine_pcg_kernel<T, 2, RAGGED, FUSED>, 2);
    case 5: return launch(sine_pcg_kernel<T, 5, RAGGED, FUSED>, 5);
  }
  if constexpr (!FUSED) switch (A.tab.ept) {
      case 8: return launch(sine_pcg_kernel<T, 8, RAGGED, false>, 8);
      case 11: return launch(sine_pcg_kernel<T, 11, RAGGED, false>, 11);
      case 14: return launch(sine_pcg_kernel<T, 14, RAGGED, false>, 14);
      case 18: return launch(sine_pcg_kernel<T, 18, RAGGED, false>, 18);
      case 23: return launch(sine_pcg_kernel<T, 23, RAGGED, false>, 23);
      case 27: return launch(sine_pcg_kernel<T, 27, RAGGED, false>, 27);
    }
  return hipErrorInvalidValue;
}

// Groups of a launch: one block per compute unit; a group takes its columns in
// turn. A column of one block is a group of its own.
int group_count(int ncols, int groups, int num_cu) {
  return groups == 1 ? ncols : std::min(ncols, num_cu / groups);
}

template <typename T, bool RAGGED>
hipError_t transform_in(const SineArgs<T>& A, const SineRagged<T>& C, int nx, const SineReset& reset, int num_cu,
                        hipStream_t s) {
  hipError_t e = hipSuccess;
  if (A.warm) {
    e = x_pass<T, false, RAGGED>(A, C, nx, COL_X, COL_W, SineReset{}, num_cu, s);
    if (e == hipSuccess) e = y_pass<T, false, RAGGED>(A, C, nx, COL_W, COL_S0, num_cu, s);
  }
  if (e == hipSuccess) e = x_pass<T, false, RAGGED>(A, C, nx, COL_B, COL_W, reset, num_cu, s);
  if (e == hipSuccess) e = y_pass<T, false, RAGGED>(A, C, nx, COL_W, COL_S, num_cu, s);
  return e;
}

template <typename T, bool RAGGED>
hipError_t transform_out(const SineArgs<T>& A, const SineRagged<T>& C, int nx, int num_cu, hipStream_t s) {
  hipError_t e = y_pass<T, true, RAGGED>(A, C, nx, COL_S, COL_W, num_cu, s);
  if (e == hipSuccess) e = x_pass<T, true, RAGGED>(A, C, nx, COL_W, COL_X, SineReset{}, num_cu, s);
  return e;
}

}  // namespace

template <typename T>
void launch_sine_tables(const SineSizes& z, const SineConsts& k, T* pack, int4* tiles, double* t, double* ipi,
                        bool packs, hipStream_t s) {
  auto grid = [](long n) { return dim3((unsigned)std::min<long>((n + 255) / 256, 4096)); };
  if (packs) {
    hipLaunchKernelGGL(sine_pack_kernel<T>, grid(2 * z.parts * z.pack), dim3(256), 0, s, z, k.n_e, pack);
    hipLaunchKernelGGL(sine_tile_kernel, grid(z.ntiles), dim3(256), 0, s, z, tiles);
  }
  hipLaunchKernelGGL(sine_slot_kernel, grid(z.slots), dim3(256), 0, s, z, k, tiles, t, ipi);
}

template <typename T>
hipError_t launch_sine(const SineArgs<T>& A, int num_cu, hipStream_t s) {
  if (A.ncols <= 0) return hipSuccess;
  const SineTables<T>& t = A.tab;
  const SineSizes z = sine_sizes(t.nx);
  const int ngroups = group_count(A.ncols, t.groups, num_cu);
  if (t.nx < 1 || t.nx > kSineMaxNx || A.n != (long)t.nx * t.nx || t.ept != z.ept || t.groups != z.groups ||
      t.parts != z.parts || t.nq != z.nq || ngroups < 1)
    return hipErrorInvalidValue;
  const SineReset reset{reinterpret_cast<unsigned long long*>(A.sc.part),
                        t.groups == 1 ? 0 : ngroups * t.groups * 3 * kSumWidth, A.sc.arrivals, t.groups == 1 ? 0 : 1,
                        A.sc.status};
  const SineRagged<T> none{};
  if (t.nx <= kSineFusedNx) return pcg<T, false, true>(A, none, ngroups, s);
  hipError_t e = transform_in<T, false>(A, none, t.nx, reset, num_cu, s);
  if (e == hipSuccess) e = pcg<T, false, false>(A, none, ngroups, s);
  if (e == hipSuccess) e = transform_out<T, false>(A, none, t.nx, num_cu, s);
  return e;
}

// A class of a ragged launch takes a share of the exchange and a ticket of its own.
size_t sine_exchange_bytes(int nclasses) { return sizeof(double) * (size_t)nclasses * kSineMaxBlocks * 3 * kSumWidth; }

template <typename T>
hipError_t launch_sine_ragged(const SineArgs<T>& args, const PcgCols<T>& cols, const SineTables<T>* tabs, int max_nx,
                              const SineClass* classes, int nclasses, int num_cu, hipStream_t s) {
  if (args.ncols <= 0) return hipSuccess;
  if (!cols.act || max_nx < 1 || max_nx > kSineMaxNx || num_cu > kSineMaxBlocks) return hipErrorInvalidValue;
  const SineRagged<T> C{cols, tabs};
  constexpr int share = kSineMaxBlocks * 3 * kSumWidth;
  const SineReset reset{reinterpret_cast<unsigned long long*>(args.sc.part), nclasses * share, args.sc.arrivals,
                        nclasses, args.sc.status};
  hipError_t e = transform_in<T, true>(args, C, max_nx, reset, num_cu, s);
  for (int k = 0; k < nclasses && e == hipSuccess; ++k) {
    SineArgs<T> a = args;
    a.tab.ept = classes[k].ept;
    a.tab.groups = classes[k].groups;
    a.sc.part = args.sc.part + (long)k * share;
    a.sc.arrivals = args.sc.arrivals + k;
    const int ngroups = group_count(args.ncols, classes[k].groups, num_cu);
    if (ngroups < 1) return hipErrorInvalidValue;
    e = pcg<T, true, false>(a, C, ngroups, s);
  }
  if (e == hipSuccess) e = transform_out<T, true>(args, C, max_nx, num_cu, s);
  return e;
}

template hipError_t launch_sine_ragged<double>(const SineArgs<double>&, const PcgCols<double>&,
                                               const SineTables<double>*, int, const SineClass*, int, int, hipStream_t);
template hipError_t launch_sine_ragged<float>(const SineArgs<float>&, const PcgCols<float>&, const SineTables<float>*,
                                              int, const SineClass*, int, int, hipStream_t);
template void launch_sine_tables<double>(const SineSizes&, const SineConsts&, double*, int4*, double*, double*, bool,
                                         hipStream_t);
template void launch_sine_tables<float>(const SineSizes&, const SineConsts&, float*, int4*, double*, double*, bool,
                                        hipStream_t);
template hipError_t launch_sine<double>(const SineArgs<double>&, int, hipStream_t);
template hipError_t launch_sine<float>(const SineArgs<float>&, int, hipStream_t);

}  // namespace sgk
