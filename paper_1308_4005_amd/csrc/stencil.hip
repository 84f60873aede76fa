// Evaluation on the grids (eq:evaluation, k = 1..l):
//   levels k < l:  e^k[mu] = 2^(-6(k-1)) sum_{delta: |delta o h_1| < 2a} g_1(|delta o h_1|) q^k[(mu - delta) mod n_k]
//                  (the cutoff 2^k a and spacing 2^(k-1) h_1 give the same offsets on every level and
//                  g_k(2^(k-1) s) = 2^(-6(k-1)) g_1(s), Sec. II.A.4)
//   level l:       e^l[mu] = sum_nu K_l[(mu - nu) mod n_l] q^l[nu]   with the pre-summed periodic kernel of
//                  eq:last-grid-periodic-transformed (all-to-all, FP64).
//
// Level stencil kernels: a block owns an 8 x 8 x ZC box of output points and
// reads the box plus an R-wide periodic halo from LDS, whole (k_stencil_tile)
// or in slabs of z planes (k_stencil_slab).  For every tap column (|dx|,|dy|)
// the up to four mirror images q[x+-dx, y+-dy] of a plane are summed once and
// applied to the outputs within hz planes, held in registers.
#include <algorithm>

#include "device_math.h"
#include "mls_internal.h"

namespace mls {

int stencil_window(const mls_plan_s* P);

namespace {

// The stencils' rows and weights, host-written tables read at uniform indexes,
// through the constant address space: scalar loads whatever else the kernel
// stores (the coarsest level's blocks made the compiler read them per lane).
template <class T>
using const_table = const __attribute__((address_space(4))) T*;
template <class T>
__device__ __forceinline__ const_table<T> table(const void* p) {
  return (const_table<T>)p;
}

// What a launch of the level stencils covers: levels 1..kmax, the coarsest
// level too, and (mixed precision, sum_rows > 0) the sum of the charges.
struct StencilOpts {
  int kmax = 0;
  bool coarsest = false;
  int sum_rows = 0;
};


constexpr int kBlock = 256;

// Reference-structured stencil: one thread per output point, taps from the
// level-1 table (used for halos wider than the instantiated window).
__global__ void __launch_bounds__(kBlock) k_stencil_taps_f64(const double* __restrict__ q, GridDims g,
                                                             const Tap* __restrict__ taps, int ntaps, double scale,
                                                             double* __restrict__ e) {
  const int mu = blockIdx.x * blockDim.x + threadIdx.x;
  if (mu >= g.size) return;
  const int x = mu % g.n[0], y = (mu / g.n[0]) % g.n[1], z = mu / (g.n[0] * g.n[1]);
  double acc = 0.0;
  for (int t = 0; t < ntaps; ++t) {
    const Tap tp = taps[t];
    const int sx = wrapi(x - tp.dx, g.n[0]);
    const int sy = wrapi(y - tp.dy, g.n[1]);
    const int sz = wrapi(z - tp.dz, g.n[2]);
    acc += tp.w * q[((size_t)sz * g.n[1] + sy) * g.n[0] + sx];
  }
  e[mu] = scale * acc;
}

// ---------------------------------------------------------------------------
// Tiled level stencil.  A block owns an 8 x 8 x ZC box of output points of
// one level (all levels share one launch through a tile table).  It loads the
// box plus an R-wide periodic halo into LDS once.  Its W waves split the tap
// columns (|dx|,|dy|); for each column the wave reads the column's weights
// once and runs a fully unrolled loop over the ZC + 2 hz input planes: the
// four mirror images q[x+-dx, y+-dy] are summed (on the axes the duplicate
// images are compensated by weights pre-divided on the host) and added with
// weight w[|dz|] into all ZC outputs held in registers.  The W partial sums
// are added in LDS at the end.
}  // namespace

// z extent of a single plan's stencil tile for halo window R: 16 for FP32
// tiles up to R = 6, else 8 (an FP64 tile of depth 16 takes (8 + 2R)^2 (16 +
// 2R) doubles, 90 KB at R = 6: one block per CU; at depth 8, 64 KB: two)
constexpr int tile_zc(int R, bool f64) { return R <= 6 && !f64 ? 16 : 8; }

// tiles16: the plan's tiles at depth 16.  FP64 slab tiles of depth 16 read
// fewer planes per output, and pay once they fill the chip (R = 8 / R = 12,
// depth 8 against 16: 585 tiles of depth 8 50 / 54 us, 3159 tiles 235 / 209;
// 4000 atoms 53 / 73, 585 tiles 146 / 133, 3159 tiles 630 / 467; at R = 10
// depth 16 was never faster, 159 / 176 us at 1975 tiles).
int stencil_tile_zc(int R, bool f64, int64_t tiles16) {
  if (f64 && ((R > 6 && R <= 8 && tiles16 >= 1024) || (R > 10 && R <= 12 && tiles16 >= 256))) return 16;
  return tile_zc(R, f64);
}

namespace {

// Coarsest level: all-to-all over the level (a periodic convolution of the
// charges with the pre-summed kernel K), with K and the charges staged in LDS
// when they fit (kCoarseLds points each).
//
// Rows path (batched launches), for a level whose x extent N is at most 8
// and whose staging fits: a lane owns one output row (y, z) and keeps its N sums in
// registers; the eight waves of the block split the source rows (y', z').
// Per source row a lane reads the N values of the kernel row
// ((y - y') mod n_y, (z - z') mod n_z) and the wave reads the N charges of
// the row (the same address in every lane), then the x-direction convolution
// of the two rows, N^2 FMAs with the (x - x') mod N offsets fixed at compile
// time, runs in registers.  Each K value read from LDS serves N FMAs.  The
// waves' partial rows are added in LDS in wave order (fixed order).  K rows
// sit at an odd stride in LDS so that the 8-byte reads of one wave spread
// over the banks.
//
// General path, for single plans and the levels the rows path does not
// take: a wave per output point (a.outs
// points per wave, one after another): the lanes split the source rows, each
// lane takes its (y - y', z - z') offset once per row and walks x' with
// (x - x') mod n_x, then the lanes add their partial sums across the wave
// (fixed order).
constexpr int kCoarseLds = 2048;
constexpr int kCoarseRowsMaxX = 8;

// Either path works in one LDS buffer of 2 kCoarseLds doubles, `lds`.

// x extent of a level the rows path takes, else 0
__host__ __device__ inline int coarse_rows_n(const GridDims& g) {
  const int N = g.n[0], nrow = g.n[1] * g.n[2];
  if (N < 1 || N > kCoarseRowsMaxX) return 0;
  return (int64_t)nrow * (N | 1) <= kCoarseLds && (int64_t)nrow * N <= kCoarseLds ? N : 0;
}

template <int N>
__device__ __forceinline__ void coarsest_rows(const CoarsestArgs& a, int blk, double* lds) {
  constexpr int S = N | 1;   // LDS stride of a K row, in doubles
  constexpr int kPer = kCoarseLds / kCoarsestThreads;
  double* const sk = lds;
  double* const sq = lds + kCoarseLds;
  const int n1 = a.g.n[1], n2 = a.g.n[2], nrow = n1 * n2, npt = nrow * N;
  {
    // every load of the staging in flight before the first store
    double vq[kPer], vk[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int i = min((int)threadIdx.x + u * kCoarsestThreads, npt - 1);
      vq[u] = a.q[i];
      vk[u] = a.K[i];
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int i = threadIdx.x + u * kCoarsestThreads;
      if (i < npt) {
        const int r = i / N;
        sk[r * S + (i - r * N)] = vk[u];
        sq[i] = vq[u];
      }
    }
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int row = blk * 64 + lane;
  const int y = row < nrow ? row % n1 : 0, z = row < nrow ? row / n1 : 0;
  const int r0 = (nrow * wv) / kCoarsestWaves, r1 = (nrow * (wv + 1)) / kCoarsestWaves;
  double acc[N];
#pragma unroll
  for (int x = 0; x < N; ++x) acc[x] = 0.0;
  int ys = r0 % n1, zs = r0 / n1;
  for (int r = r0; r < r1; ++r) {
    const int ky = y - ys + (y < ys ? n1 : 0), kz = z - zs + (z < zs ? n2 : 0);
    const int kb = (kz * n1 + ky) * S;
    double k[N], q[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      k[j] = sk[kb + j];
      q[j] = sq[r * N + j];
    }
#pragma unroll
    for (int xs = 0; xs < N; ++xs)
#pragma unroll
      for (int x = 0; x < N; ++x) acc[x] = fma(k[(x - xs + N) % N], q[xs], acc[x]);
    if (++ys == n1) {
      ys = 0;
      ++zs;
    }
  }
  __syncthreads();   // staging no longer read: the buffer takes the partial rows
  double* const red = lds;
#pragma unroll
  for (int x = 0; x < N; ++x) red[(wv * N + x) * 64 + lane] = acc[x];
  __syncthreads();
  if (threadIdx.x < 64 * N) {
    const int x = threadIdx.x >> 6;
    double v = 0.0;
#pragma unroll
    for (int w = 0; w < kCoarsestWaves; ++w) v += red[(w * N + x) * 64 + lane];
    if (row < nrow) a.e[row * N + x] = v;
  }
}

// have_q: the charges are already at the end of lds (coarsest_restrict)
template <bool STAGED>
__device__ __forceinline__ void coarsest_sums(const CoarsestArgs& a, int blk, double* lds, bool have_q = false) {
  const GridDims& g = a.g;
  double* const sk = lds;
  double* const sq = lds + (have_q ? 2 * kCoarseLds - g.size : kCoarseLds);
  if (STAGED && have_q) {
    for (int i = threadIdx.x; i < g.size; i += kCoarsestThreads) sk[i] = a.K[i];
    __syncthreads();
  } else if constexpr (STAGED) {
    constexpr int kPer = kCoarseLds / kCoarsestThreads;
    double vq[kPer], vk[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int i = min((int)threadIdx.x + u * kCoarsestThreads, g.size - 1);
      vq[u] = a.q[i];
      vk[u] = a.K[i];
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int i = threadIdx.x + u * kCoarsestThreads;
      if (i < g.size) {
        sq[i] = vq[u];
        sk[i] = vk[u];
      }
    }
    __syncthreads();
  }
  const double* __restrict__ gK = a.K;
  const double* __restrict__ gq = a.q;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int n0 = g.n[0], n1 = g.n[1], n2 = g.n[2], n01 = n0 * n1, nrow = n1 * n2;
  const int b1 = 64 % n1, b2 = 64 / n1, ys0 = lane % n1, zs0 = lane / n1;
  for (int m = 0; m < a.outs; ++m) {
    const int mu = (blk * a.outs + m) * kCoarsestWaves + wv;
    if (mu >= g.size) break;
    const int x = mu % n0, y = (mu / n0) % n1, z = mu / n01;
    double acc = 0.0;
    // (ys, zs) of row r = lane + 64 t, advanced with a carry (no division
    // per row)
    int ys = ys0, zs = zs0;
    for (int r = lane; r < nrow; r += 64) {
      const int ky = y - ys + (y < ys ? n1 : 0), kz = z - zs + (z < zs ? n2 : 0);
      const int kr = kz * n01 + ky * n0, qr = r * n0;
#pragma unroll 4
      for (int xs = 0; xs < n0; ++xs) {
        const int kx = x - xs + (x < xs ? n0 : 0);
        if constexpr (STAGED) acc = fma(sk[kr + kx], sq[qr + xs], acc);
        else acc = fma(gK[kr + kx], gq[qr + xs], acc);
      }
      ys += b1;
      const int cy = ys >= n1;
      ys -= cy ? n1 : 0;
      zs += b2 + cy;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if (lane == 0) a.e[mu] = acc;
  }
}

struct Coarsest {
  using Args = CoarsestArgs;
  static constexpr int kThreads = kCoarsestThreads;
  static __device__ void run(const Args& a, int blk) {
    __shared__ double lds[2 * kCoarseLds];
    switch (a.rows) {
      case 1: coarsest_rows<1>(a, blk, lds); break;
      case 2: coarsest_rows<2>(a, blk, lds); break;
      case 3: coarsest_rows<3>(a, blk, lds); break;
      case 4: coarsest_rows<4>(a, blk, lds); break;
      case 5: coarsest_rows<5>(a, blk, lds); break;
      case 6: coarsest_rows<6>(a, blk, lds); break;
      case 7: coarsest_rows<7>(a, blk, lds); break;
      case 8: coarsest_rows<8>(a, blk, lds); break;
      default:
        if (a.g.size <= kCoarseLds) coarsest_sums<true>(a, blk, lds);
        else coarsest_sums<false>(a, blk, lds);
    }
  }
};
// The level stencils of one grid chain, or of the seven of a Lorentz-Berthelot
// plan: the chains share the levels' geometry and tables, and block b takes
// tile b mod ntiles of chain b / ntiles.  The blocks past the nchain * ntiles
// tiles, if any, do the coarsest level (ncoarse each): it needs only the last
// restriction, as the stencils do, and as a launch of its own it cost 4 us of an
// evaluation's 79 (1000 atoms, FP64), 5 us of a mixed time step's 152 (32000).
struct StencilLaunch {
  StencilLevel lv[16];   // q, e and sum_xi per chain:
  gptr<const double> q[kLbVectors][16];
  gptr<double> e[kLbVectors][16];
  // mixed precision: the sum of the charges, or (sum_rows > 0) its partial sums
  // over 256 rows each, which every block adds up itself
  gptr<const double> sum[kLbVectors];
  int sum_rows;
  int nchain;
  int ntiles;
  int ncoarse;
  gptr<const double> K;  // coarsest level
  GridDims gc;
  gptr<double> qc[kLbVectors];
  gptr<double> ec[kLbVectors];
  // the last restriction, done by the coarsest level's blocks too (qf null: not)
  GridDims gf;
  int taps;              // odd offsets per side
  double w[3];           // their weights
  gptr<const double> qf[kLbVectors];
};

// The coarsest level's charges from the next finer level's, to the end of lds
// (and, by the chain's first block, to memory): the restriction dimension by
// dimension, in the order of sums of RestrictTile (grid.hip).  Every block of the
// level does it for itself, up to kJointCoarse points: a third of the work of
// the points' (p + 1)^3 taps, while the level stencils run, against a launch
// of 4 us on the chain (p = 6: 8 us).
constexpr int kJointCoarse = 2 * kCoarseLds / 7;   // x and y passes (4 + 2 values per point) and the points
__device__ __forceinline__ double restrict_line(const StencilLaunch& L, const double* line, int stride, int n, int X) {
  double s = line[(size_t)wrapi(2 * X, n) * stride];
  for (int k = 0; k < L.taps; ++k) {
    const int o = 2 * k + 1;
    s += L.w[k] * line[(size_t)wrapi(2 * X - o, n) * stride];
    s += L.w[k] * line[(size_t)wrapi(2 * X + o, n) * stride];
  }
  return s;
}

__device__ __forceinline__ void coarsest_restrict(const StencilLaunch& L, int c, int blk, double* lds) {
  const GridDims &f = L.gf, &g = L.gc;
  const int nx = g.n[0], ny = g.n[1], fx = f.n[0], fy = f.n[1], fz = f.n[2];
  double* const tx = lds;                      // (nx, fy, fz)
  double* const ty = lds + nx * fy * fz;       // (nx, ny, fz)
  double* const sq = lds + 2 * kCoarseLds - g.size;
  const double* const q = L.qf[c];
  for (int i = threadIdx.x; i < nx * fy * fz; i += kCoarsestThreads) {
    const int r = i / nx;
    tx[i] = restrict_line(L, q + (size_t)r * fx, 1, fx, i - r * nx);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < nx * ny * fz; i += kCoarsestThreads) {
    const int r = i / nx, z = r / ny;
    ty[i] = restrict_line(L, tx + z * fy * nx + (i - r * nx), nx, fy, r - z * ny);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < g.size; i += kCoarsestThreads) {
    const int z = i / (nx * ny);
    const double v = restrict_line(L, ty + (i - z * nx * ny), nx * ny, fz, z);
    sq[i] = v;
    if (blk == 0) L.qc[c][i] = v;
  }
  __syncthreads();   // tx and ty are free
}

// A block of the coarsest level: done here (true).
__device__ __forceinline__ bool coarsest_block(const StencilLaunch& L, int b, double* lds) {
  const int nt = L.nchain * L.ntiles;
  if (b < nt) return false;
  const int c = (b - nt) / L.ncoarse, blk = (b - nt) - c * L.ncoarse;
  const CoarsestArgs a{(double*)L.qc[c], L.gc, L.K, L.ec[c], 1, 0};
  const bool joint = L.qf[c] != nullptr;
  if (joint) coarsest_restrict(L, c, blk, lds);
  if (L.gc.size <= kCoarseLds) coarsest_sums<true>(a, blk, lds, joint);
  else coarsest_sums<false>(a, blk, lds);
  return true;
}

__device__ __forceinline__ StencilLevel stencil_level(const StencilLaunch& L, int b, const int4* __restrict__ tiles,
                                                      int4& tinfo) {
  const int c = b / L.ntiles;
  tinfo = tiles[b - c * L.ntiles];
  StencilLevel V = L.lv[tinfo.x];
  V.q = L.q[c][tinfo.x];
  V.e = L.e[c][tinfo.x];
  V.sum_xi = L.sum[c];
  return V;
}

// The sum of the charges behind V.sum_xi: read, or added up from its partial
// sums in the order of SumXiFinal (the same bits); lds is free afterwards.
__device__ __forceinline__ double charge_sum(const StencilLevel& V, int rows, double* lds) {
  if (rows <= 0) return *V.sum_xi;
  constexpr int kRows = 256;
  const int nb = (rows + kRows - 1) / kRows, t = threadIdx.x;
  if (t < kRows) {
    double v = 0.0;
    for (int i = t; i < nb; i += kRows) v += V.sum_xi[i];
    lds[t] = v;
  }
  __syncthreads();
  for (int off = kRows / 2; off > 0; off >>= 1) {
    if (t < off) lds[t] += lds[t + off];
    __syncthreads();
  }
  const double sum = lds[0];
  __syncthreads();
  return sum;
}

template <class T, int HZ, int ZC>
__device__ __forceinline__ void tile_column(T (&acc)[ZC], const T* __restrict__ c, int o0, int o1, int o2, int o3,
                                            int pstride, const_table<T> w) {
  T wr[HZ + 1];
#pragma unroll
  for (int d = 0; d <= HZ; ++d) wr[d] = w[d];
#pragma unroll
  for (int zi = -HZ; zi < ZC + HZ; ++zi) {
    const T* p = c + zi * pstride;
    const T s = (p[o0] + p[o1]) + (p[o2] + p[o3]);
#pragma unroll
    for (int dz = -HZ; dz <= HZ; ++dz) {
      const int zo = zi + dz;
      if (zo >= 0 && zo < ZC) acc[zo] += wr[dz < 0 ? -dz : dz] * s;
    }
  }
}

template <class T, int R, int ZC, int H = 0>
__device__ __forceinline__ void tile_switch(int hz, T (&acc)[ZC], const T* c, int o0, int o1, int o2, int o3,
                                            int pstride, const_table<T> w) {
  if constexpr (H <= R) {
    if (hz == H) {
      tile_column<T, H, ZC>(acc, c, o0, o1, o2, o3, pstride, w);
      return;
    }
    tile_switch<T, R, ZC, H + 1>(hz, acc, c, o0, o1, o2, o3, pstride, w);
  }
}

// FP32 tiles hold q - mean (mean = sum_i xi / points, the exact mean by the
// partition of unity); the constant part adds back as mean * sum of weights,
// since a periodic convolution maps a constant c to c times the weight sum.
// lds: the tile, then the reduction buffer of the W partial sums (TileShape).
template <class T, int R, int ZC, int W>
struct TileShape {
  static constexpr int SX = 8 + 2 * R, NP = SX * SX * (ZC + 2 * R), NR = W * ZC * 64;
  static constexpr int NL = NP > NR ? NP : NR;
  static constexpr int kDoubles = (int)((NL * sizeof(T) + 7) / 8);
};

template <class T, int R, int ZC, int W>
__device__ __forceinline__ void stencil_tile(const StencilLevel& V, const int4 tinfo, double sum_xi, double* lds) {
  constexpr int SX = 8 + 2 * R, SY = 8 + 2 * R, SZ = ZC + 2 * R;
  constexpr int PS = SX * SY, NP = PS * SZ, NT = 64 * W;
  T* const tile = reinterpret_cast<T*>(lds);
  __shared__ int wrapx[SX], wrapy[SY], wrapz[SZ];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int x0 = tinfo.y * 8, y0 = tinfo.z * 8, z0 = tinfo.w * ZC;
  if (tid < SX) wrapx[tid] = wrapi(x0 - R + tid, V.n[0]);
  if (tid < SY) wrapy[tid] = wrapi(y0 - R + tid, V.n[1]);
  if (tid < SZ) wrapz[tid] = wrapi(z0 - R + tid, V.n[2]);
  __syncthreads();
  const size_t gps = (size_t)V.n[0] * V.n[1];
  const double* __restrict__ q = V.q;
  const double mean = sizeof(T) < sizeof(double) ? sum_xi * V.inv_size : 0.0;
  // the fill issues kFill global loads per thread before it waits for them
  // (one load per wait leaves the block waiting on memory latency NP / NT
  // times); indexes past the box are clamped, so every load is in range
  constexpr int kIters = (NP + NT - 1) / NT, kFill = 8;
  for (int b0 = 0; b0 < kIters; b0 += kFill) {
    double v[kFill];
#pragma unroll
    for (int u = 0; u < kFill; ++u) {
      const int i = min(tid + (b0 + u) * NT, NP - 1);
      const int lx = i % SX, ly = (i / SX) % SY, lz = i / PS;
      v[u] = q[(size_t)wrapz[lz] * gps + (size_t)wrapy[ly] * V.n[0] + wrapx[lx]];
    }
#pragma unroll
    for (int u = 0; u < kFill; ++u) {
      const int i = tid + (b0 + u) * NT;
      if (i < NP) tile[i] = (T)(v[u] - mean);
    }
  }
  __syncthreads();
  // lanes 0-31 take the even rows, 32-63 the odd ones: with a row pitch of
  // 20 words (R = 6) each half-wave's four rows then cover disjoint banks
  const int tx = lane & 7, ty = ((lane >> 3) & 3) * 2 + (lane >> 5);
  const T* c = tile + R * PS + (ty + R) * SX + (tx + R);
  T acc[ZC];
#pragma unroll
  for (int k = 0; k < ZC; ++k) acc[k] = T(0);
  // the column index is wave-uniform, so the rows and weights are scalar
  // loads (staging them in LDS measured slower)
  const const_table<StencilRow> rows = table<StencilRow>(V.rows);
  const const_table<T> wts = table<T>(V.wts);
  const const_table<int> wave_rows = table<int>(V.wave_rows);
  const int r0 = wave_rows[wv], r1 = wave_rows[wv + 1];
  for (int r = r0; r < r1; ++r) {
    const StencilRow row{rows[r].dx, rows[r].dy, rows[r].hz, rows[r].woff};
    const int o0 = -row.dy * SX - row.dx, o1 = -row.dy * SX + row.dx;
    const int o2 = row.dy * SX - row.dx, o3 = row.dy * SX + row.dx;
    tile_switch<T, R, ZC>(row.hz, acc, c, o0, o1, o2, o3, PS, wts + row.woff);
  }
  // add the W partial sums (the tile is reused as the reduction buffer)
  __syncthreads();
#pragma unroll
  for (int k = 0; k < ZC; ++k) tile[(wv * ZC + k) * 64 + lane] = acc[k];
  __syncthreads();
  const int x = x0 + tx, y = y0 + ty;
  if (x < V.n[0] && y < V.n[1]) {
    for (int k = wv; k < ZC; k += W) {
      const int z = z0 + k;
      if (z >= V.n[2]) break;
      T sum = tile[k * 64 + lane];
#pragma unroll
      for (int w2 = 1; w2 < W; ++w2) sum += tile[(w2 * ZC + k) * 64 + lane];
      V.e[(size_t)z * gps + (size_t)y * V.n[0] + x] = V.scale * ((double)sum + mean * V.wsum);
    }
  }
}

// One plan: all levels of the plan in one launch, level descriptors by value.
template <class T, int R, int ZC, int W>
__global__ void __launch_bounds__(64 * W) k_stencil_tile(StencilLaunch L, const int4* __restrict__ tiles) {
  constexpr int kLds = TileShape<T, R, ZC, W>::kDoubles;
  static_assert(kLds >= 2 * kCoarseLds, "the coarsest level works in the tile's LDS");
  __shared__ double lds[kLds];
  const int b = xcd_block(blockIdx.x, gridDim.x);
  if (coarsest_block(L, b, lds)) return;
  int4 tinfo;
  const StencilLevel V = stencil_level(L, b, tiles, tinfo);
  stencil_tile<T, R, ZC, W>(V, tinfo, sizeof(T) < sizeof(double) ? charge_sum(V, L.sum_rows, lds) : 0.0, lds);
}

// FP64 tile read in NCH slabs of z planes: the same columns, weights and
// register outputs, but only a slab of the ZC + 2 R input planes is in LDS at a
// time: an FP64 tile of R = 10 would take 176 KB.  LDS reads bound it (four
// 8-byte reads per plane and column against 2 hz + 1 FMAs per output), so the
// slabs are as large as two blocks per CU allow.  Level stencils of 60,013 atoms
// at a = 4, h = 0.8 (56^3 and two coarser levels, R = 10): 950 us with a kernel
// that streamed single planes through LDS, 46 us here; R = 12 at 300,000 atoms
// 467 us; R = 8 at 10^6 atoms 266 us with whole tiles (110 KB, one block per
// CU), 209 us here.  Up to R = 6 the whole tile (64 KB) is faster: 71 against
// 82 us at 10^6 atoms in two slabs.
template <int R, int ZC, int P0, int P1, int HZ>
__device__ __forceinline__ void slab_column(double (&acc)[ZC], const double* __restrict__ c, int o0, int o1, int o2,
                                            int o3, const_table<double> w) {
  constexpr int PS = (8 + 2 * R) * (8 + 2 * R);
  double wr[HZ + 1];
#pragma unroll
  for (int d = 0; d <= HZ; ++d) wr[d] = w[d];
#pragma unroll
  for (int p = P0; p < P1; ++p) {
    const int zi = p - R;   // relative to the first output plane
    if (zi < -HZ || zi >= ZC + HZ) continue;
    const double* q = c + (p - P0) * PS;
    const double s = (q[o0] + q[o1]) + (q[o2] + q[o3]);
#pragma unroll
    for (int dz = -HZ; dz <= HZ; ++dz) {
      const int zo = zi + dz;
      if (zo >= 0 && zo < ZC) acc[zo] += wr[dz < 0 ? -dz : dz] * s;
    }
  }
}

template <int R, int ZC, int P0, int P1, int H = 0>
__device__ __forceinline__ void slab_switch(int hz, double (&acc)[ZC], const double* c, int o0, int o1, int o2, int o3,
                                            const_table<double> w) {
  if constexpr (H <= R) {
    if (hz == H) {
      slab_column<R, ZC, P0, P1, H>(acc, c, o0, o1, o2, o3, w);
      return;
    }
    slab_switch<R, ZC, P0, P1, H + 1>(hz, acc, c, o0, o1, o2, o3, w);
  }
}

template <int R, int ZC, int NCH, int W>
struct SlabShape {
  static constexpr int SX = 8 + 2 * R, PS = SX * SX, NZ = ZC + 2 * R, SP = (NZ + NCH - 1) / NCH, NT = 64 * W;
  static constexpr int RZ = 8;   // output planes added up at a time
  static constexpr int NL = PS * SP > W * RZ * 64 ? PS * SP : W * RZ * 64;
  static_assert(NL >= 2 * kCoarseLds, "the coarsest level works in the slab's LDS");
};

// Slab CH and the ones after it: fill, then every column of the wave.
template <int R, int ZC, int NCH, int W, int CH>
__device__ __forceinline__ void slab_pass(const StencilLevel& V, double* slab, const int* wrapx, const int* wrapy,
                                          const int* wrapz, int tid, int wv, int c0, double (&acc)[ZC]) {
  if constexpr (CH < NCH) {
    using S = SlabShape<R, ZC, NCH, W>;
    constexpr int P0 = CH * S::SP, P1 = P0 + S::SP < S::NZ ? P0 + S::SP : S::NZ;
    constexpr int NP = S::PS * (P1 - P0), kIters = (NP + S::NT - 1) / S::NT, kFill = 8;
    const size_t gps = (size_t)V.n[0] * V.n[1];
    const double* __restrict__ q = V.q;
    if constexpr (CH > 0) __syncthreads();   // the slab before it has been read
    // kFill loads in flight per thread; indexes past the slab are clamped
    for (int b0 = 0; b0 < kIters; b0 += kFill) {
      double v[kFill];
#pragma unroll
      for (int u = 0; u < kFill; ++u) {
        const int i = min(tid + (b0 + u) * S::NT, NP - 1);
        const int lx = i % S::SX, ly = (i / S::SX) % S::SX, lz = i / S::PS;
        v[u] = q[(size_t)wrapz[P0 + lz] * gps + (size_t)wrapy[ly] * V.n[0] + wrapx[lx]];
      }
#pragma unroll
      for (int u = 0; u < kFill; ++u) {
        const int i = tid + (b0 + u) * S::NT;
        if (i < NP) slab[i] = v[u];
      }
    }
    __syncthreads();
    const const_table<StencilRow> rows = table<StencilRow>(V.rows);
    const const_table<double> wts = table<double>(V.wts);
    const const_table<int> wave_rows = table<int>(V.wave_rows);
    const int r0 = wave_rows[wv], r1 = wave_rows[wv + 1];
    for (int r = r0; r < r1; ++r) {
      const StencilRow row{rows[r].dx, rows[r].dy, rows[r].hz, rows[r].woff};
      const int o0 = -row.dy * S::SX - row.dx, o1 = -row.dy * S::SX + row.dx;
      const int o2 = row.dy * S::SX - row.dx, o3 = row.dy * S::SX + row.dx;
      slab_switch<R, ZC, P0, P1>(row.hz, acc, slab + c0, o0, o1, o2, o3, wts + row.woff);
    }
    slab_pass<R, ZC, NCH, W, CH + 1>(V, slab, wrapx, wrapy, wrapz, tid, wv, c0, acc);
  }
}

// slab: the slab, then the reduction buffer of the W partial sums.
template <int R, int ZC, int NCH, int W>
__device__ __forceinline__ void stencil_slab(const StencilLevel& V, const int4 tinfo, double* slab) {
  using S = SlabShape<R, ZC, NCH, W>;
  __shared__ int wrapx[S::SX], wrapy[S::SX], wrapz[S::NZ];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int x0 = tinfo.y * 8, y0 = tinfo.z * 8, z0 = tinfo.w * ZC;
  if (tid < S::SX) {
    wrapx[tid] = wrapi(x0 - R + tid, V.n[0]);
    wrapy[tid] = wrapi(y0 - R + tid, V.n[1]);
  }
  if (tid < S::NZ) wrapz[tid] = wrapi(z0 - R + tid, V.n[2]);
  __syncthreads();
  const int tx = lane & 7, ty = ((lane >> 3) & 3) * 2 + (lane >> 5);   // as stencil_tile
  double acc[ZC];
#pragma unroll
  for (int k = 0; k < ZC; ++k) acc[k] = 0.0;
  slab_pass<R, ZC, NCH, W, 0>(V, slab, wrapx, wrapy, wrapz, tid, wv, (ty + R) * S::SX + (tx + R), acc);
  const int x = x0 + tx, y = y0 + ty;
  const size_t gps = (size_t)V.n[0] * V.n[1];
#pragma unroll
  for (int k0 = 0; k0 < ZC; k0 += S::RZ) {
    __syncthreads();
#pragma unroll
    for (int k = 0; k < S::RZ; ++k) slab[(wv * S::RZ + k) * 64 + lane] = acc[k0 + k];
    __syncthreads();
    for (int k = wv; k < S::RZ; k += W) {
      const int z = z0 + k0 + k;
      if (x < V.n[0] && y < V.n[1] && z < V.n[2]) {
        double sum = slab[k * 64 + lane];
#pragma unroll
        for (int w = 1; w < W; ++w) sum += slab[(w * S::RZ + k) * 64 + lane];
        V.e[(size_t)z * gps + (size_t)y * V.n[0] + x] = V.scale * sum;
      }
    }
  }
}

// Batched, one block per item.  Without the loop over items the compiler keeps
// 78 instead of 127 VGPRs (FP32, R = 6), so that LDS alone limits the blocks
// per CU to three instead of the registers to two.
template <class T, int R, int ZC, int W>
__global__ void __launch_bounds__(64 * W) k_stencil_tile_each(const StencilLevel* __restrict__ lv,
                                                              const int4* __restrict__ tiles) {
  const int4 tinfo = tiles[xcd_block(blockIdx.x, gridDim.x)];
  const StencilLevel V = lv[tinfo.x];
  __shared__ double lds[TileShape<T, R, ZC, W>::kDoubles];
  stencil_tile<T, R, ZC, W>(V, tinfo, sizeof(T) < sizeof(double) ? (double)*V.sum_xi : 0.0, lds);
}

template <int R, int ZC, int NCH, int W>
__global__ void __launch_bounds__(64 * W) k_stencil_slab(StencilLaunch L, const int4* __restrict__ tiles) {
  __shared__ double slab[SlabShape<R, ZC, NCH, W>::NL];
  const int b = xcd_block(blockIdx.x, gridDim.x);
  if (coarsest_block(L, b, slab)) return;
  int4 tinfo;
  const StencilLevel V = stencil_level(L, b, tiles, tinfo);
  stencil_slab<R, ZC, NCH, W>(V, tinfo, slab);
}

template <int R, int ZC, int NCH, int W>
__global__ void __launch_bounds__(64 * W) k_stencil_slab_batched(const StencilLevel* __restrict__ lv,
                                                                 const int4* __restrict__ tiles, int ntiles) {
  __shared__ double slab[SlabShape<R, ZC, NCH, W>::NL];
  for (int t = xcd_block(blockIdx.x, gridDim.x); t < ntiles; t += gridDim.x) {
    const int4 tinfo = tiles[t];
    const StencilLevel V = lv[tinfo.x];
    stencil_slab<R, ZC, NCH, W>(V, tinfo, slab);
    __syncthreads();
  }
}

// MFMA recast of the FP32 tile (window R <= 6, 8 x 8 x 16 outputs per block).
// For one tap column (dx, dy) the z sum is a banded Toeplitz product:
// e[z][xy] += sum_t A[z][t] B[t][xy] with A[z][t] = w(|t - hz - z|) (input
// plane t counted from hz below the tile) and B[t][xy] the four mirror
// images q[x -+ dx, y -+ dy] of plane t summed, as in the VALU tile.  Each
// v_mfma_f32_16x16x4_f32 takes 16 output planes (M), 16 xy points (N) and
// four input planes (K): a column needs S = ceil((16 + 2 hz) / 4) chunks for
// each of the tile's four 16-point xy blocks.  The A operands come from a
// host table (one coalesced load per chunk, shared by the four blocks); B is
// folded from LDS.  The W waves split the columns and add their partial
// tiles in LDS, as the VALU tile does.  Operand layouts (lane = row + 16 *
// column of A, column + 16 * row of B; D[i][j] in lane j + 16 (i / 4),
// register i % 4) were checked on the device.
typedef float mfma_f4 __attribute__((ext_vector_type(4)));

template <int R, int HZ>
__device__ __forceinline__ void mfma_column(mfma_f4 (&acc)[4], const float* __restrict__ tile, const int (&base)[4],
                                            int o0, int o1, int o2, int o3, const float* __restrict__ at) {
  constexpr int SX = 8 + 2 * R, PS = SX * SX;
  constexpr int S = (16 + 2 * HZ + 3) / 4;
#pragma unroll
  for (int sc = 0; sc < S; ++sc) {
    const float a = at[64 * sc];
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
      const float* p = tile + base[nb] + 4 * sc * PS;
      const float b = (p[o0] + p[o1]) + (p[o2] + p[o3]);
      acc[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc[nb], 0, 0, 0);
    }
  }
}

template <int R, int H = 0>
__device__ __forceinline__ void mfma_switch(int hz, mfma_f4 (&acc)[4], const float* tile, int (&base)[4], int o0,
                                            int o1, int o2, int o3, const float* at) {
  if constexpr (H <= R) {
    if (hz == H) {
      constexpr int SX = 8 + 2 * R, PS = SX * SX;
      // chunk 0 starts hz planes below the tile's first output plane
      int b[4];
#pragma unroll
      for (int nb = 0; nb < 4; ++nb) b[nb] = base[nb] + (R - H) * PS;
      mfma_column<R, H>(acc, tile, b, o0, o1, o2, o3, at);
      return;
    }
    mfma_switch<R, H + 1>(hz, acc, tile, base, o0, o1, o2, o3, at);
  }
}

template <int R, int W>
__global__ void __launch_bounds__(64 * W) k_stencil_mfma(StencilLaunch L, const int4* __restrict__ tiles) {
  constexpr int ZC = 16;
  // four zero planes above the halo: the last K chunk of a column may reach
  // up to three planes past its band
  constexpr int SX = 8 + 2 * R, SY = 8 + 2 * R, SZH = ZC + 2 * R, SZ = SZH + 4;
  constexpr int PS = SX * SY, NP = PS * SZ, NT = 64 * W;
  constexpr int NL = NP > W * ZC * 64 ? NP : W * ZC * 64;
  __shared__ float tile[NL];
  __shared__ int wrapx[SX], wrapy[SY], wrapz[SZH];
  int4 tinfo;
  const StencilLevel V = stencil_level(L, xcd_block(blockIdx.x, gridDim.x), tiles, tinfo);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int x0 = tinfo.y * 8, y0 = tinfo.z * 8, z0 = tinfo.w * ZC;
  if (tid < SX) wrapx[tid] = wrapi(x0 - R + tid, V.n[0]);
  if (tid < SY) wrapy[tid] = wrapi(y0 - R + tid, V.n[1]);
  if (tid < SZH) wrapz[tid] = wrapi(z0 - R + tid, V.n[2]);
  __syncthreads();
  const size_t gps = (size_t)V.n[0] * V.n[1];
  const double* __restrict__ q = V.q;
  const double mean = *V.sum_xi * V.inv_size;
  constexpr int kIters = (NP + NT - 1) / NT, kFill = 8;
  for (int b0 = 0; b0 < kIters; b0 += kFill) {
    double v[kFill];
#pragma unroll
    for (int u = 0; u < kFill; ++u) {
      const int i = min(tid + (b0 + u) * NT, NP - 1);
      const int lx = i % SX, ly = (i / SX) % SY, lz = min(i / PS, SZH - 1);
      v[u] = q[(size_t)wrapz[lz] * gps + (size_t)wrapy[ly] * V.n[0] + wrapx[lx]];
    }
#pragma unroll
    for (int u = 0; u < kFill; ++u) {
      const int i = tid + (b0 + u) * NT;
      if (i < NP) tile[i] = i < PS * SZH ? (float)(v[u] - mean) : 0.0f;
    }
  }
  __syncthreads();
  // B operand of lane (k = lane / 16, j = lane % 16): plane k of the chunk,
  // xy point j of block nb (x = j % 8, y = 2 nb + j / 8)
  const int kk = lane >> 4, j = lane & 15;
  int base[4];
#pragma unroll
  for (int nb = 0; nb < 4; ++nb) base[nb] = kk * PS + (2 * nb + (j >> 3) + R) * SX + ((j & 7) + R);
  mfma_f4 acc[4];
#pragma unroll
  for (int nb = 0; nb < 4; ++nb) acc[nb] = mfma_f4{0.0f, 0.0f, 0.0f, 0.0f};
  const StencilRow* __restrict__ rows = V.rows;
  const float* __restrict__ atab = (const float*)(const void*)V.wts;
  const int r0 = V.wave_rows[wv], r1 = V.wave_rows[wv + 1];
  for (int r = r0; r < r1; ++r) {
    const StencilRow row = rows[r];
    const int o0 = -row.dy * SX - row.dx, o1 = -row.dy * SX + row.dx;
    const int o2 = row.dy * SX - row.dx, o3 = row.dy * SX + row.dx;
    mfma_switch<R>(row.hz, acc, tile, base, o0, o1, o2, o3, atab + row.woff + lane);
  }
  // add the W partial tiles (the tile is reused): D[i][j] of block nb is
  // output plane i = 4 (lane / 16) + register, xy point 16 nb + j
  __syncthreads();
#pragma unroll
  for (int nb = 0; nb < 4; ++nb)
#pragma unroll
    for (int rg = 0; rg < 4; ++rg) tile[(wv * ZC + 4 * kk + rg) * 64 + 16 * nb + j] = acc[nb][rg];
  __syncthreads();
  for (int o = tid; o < ZC * 64; o += NT) {
    const int z = o >> 6, xy = o & 63;
    const int x = x0 + (xy & 7), y = y0 + (xy >> 3), zz = z0 + z;
    if (x >= V.n[0] || y >= V.n[1] || zz >= V.n[2]) continue;
    float sum = 0.0f;
#pragma unroll
    for (int w2 = 0; w2 < W; ++w2) sum += tile[(w2 * ZC + z) * 64 + xy];
    V.e[(size_t)zz * gps + (size_t)y * V.n[0] + x] = V.scale * ((double)sum + mean * V.wsum);
  }
}

// Batched: tiles of many plans' levels; tinfo.x indexes the descriptor array.
template <class T, int R, int ZC, int W>
__global__ void __launch_bounds__(64 * W) k_stencil_tile_batched(const StencilLevel* __restrict__ lv,
                                                                 const int4* __restrict__ tiles, int ntiles) {
  __shared__ double lds[TileShape<T, R, ZC, W>::kDoubles];
  for (int t = xcd_block(blockIdx.x, gridDim.x); t < ntiles; t += gridDim.x) {
    const int4 tinfo = tiles[t];
    const StencilLevel V = lv[tinfo.x];
    stencil_tile<T, R, ZC, W>(V, tinfo, sizeof(T) < sizeof(double) ? (double)*V.sum_xi : 0.0, lds);
    __syncthreads();
  }
}

inline int nblocks(int64_t n, int b) { return (int)((n + b - 1) / b); }

}  // namespace

// Blocks of the coarsest-level kernel for grid g with `outs` output points
// per wave.
int coarsest_rows_form(const GridDims& g) { return coarse_rows_n(g); }

int coarsest_blocks(const GridDims& g, int outs, int rows) {
  if (rows) return (g.n[1] * g.n[2] + 63) / 64;
  return (int)(((int64_t)g.size + (int64_t)kCoarsestWaves * outs - 1) / ((int64_t)kCoarsestWaves * outs));
}

int stencil_window(const mls_plan_s* P) {
  return std::max(P->stencil_R[0], std::max(P->stencil_R[1], P->stencil_R[2]));
}

// Descriptors of levels 1..kmax of a plan's chains (kmax = l - 1: all; the tile
// table lists the levels in order, so levels 1..kmax are its head), with the
// coarsest level where asked for; returns the blocks of a launch over them.
int stencil_levels(const mls_plan_s* P, const StencilRow* rows, const void* wts, const StencilOpts& o,
                   StencilLaunch& L) {
  static_assert(sizeof(StencilLaunch) <= 3840, "kernel arguments");
  const int zc = P->stencil_zc;
  const ChainSet cs = chains(P);
  int t = 0;
  for (int k = 1; k <= o.kmax; ++k) {
    const Level& Lv = P->lv[k - 1];
    StencilLevel& V = L.lv[k - 1];
    for (int d = 0; d < 3; ++d) V.n[d] = Lv.g.n[d];
    V.tiles_z = nblocks(Lv.g.n[2], zc);
    V.tile0 = t;
    V.scale = std::ldexp(1.0, -6 * (k - 1));
    V.inv_size = 1.0 / (double)Lv.g.size;
    V.rows = rows;
    V.wave_rows = P->d_wave_rows;
    V.wts = wts;
    V.wsum = P->taps_wsum;
    t += nblocks(Lv.g.n[0], 8) * nblocks(Lv.g.n[1], 8) * V.tiles_z;
    for (int v = 0; v < cs.n; ++v) {
      L.q[v][k - 1] = (*cs.lv[v])[k - 1].q;
      L.e[v][k - 1] = (*cs.lv[v])[k - 1].e;
    }
  }
  const Level& C = P->lv[P->levels - 1];
  L.nchain = cs.n;
  L.ntiles = t;
  L.ncoarse = o.coarsest ? coarsest_blocks(C.g, 1, 0) : 0;
  L.K = P->d_Kl;
  L.gc = C.g;
  L.sum_rows = o.sum_rows;
  const bool joint = o.coarsest && coarsest_restricts(P);
  L.gf = P->lv[P->levels - 2].g;
  const double w4[3] = {9.0 / 16.0, -1.0 / 16.0, 0.0}, w6[3] = {75.0 / 128.0, -25.0 / 256.0, 3.0 / 256.0};
  L.taps = P->order / 2;
  for (int k = 0; k < 3; ++k) L.w[k] = P->order == 4 ? w4[k] : w6[k];
  for (int v = 0; v < cs.n; ++v) {
    L.qc[v] = (*cs.lv[v])[P->levels - 1].q;
    L.ec[v] = (*cs.lv[v])[P->levels - 1].e;
    L.qf[v] = joint ? (*cs.lv[v])[P->levels - 2].q : nullptr;
    L.sum[v] = o.sum_rows > 0 ? (cs.n == 1 ? P->d_xi_partial : lb_partial_buf(P, v)) : cs.sum[v];
  }
  return (t + L.ncoarse) * cs.n;
}

template <class T, int R, int ZC = tile_zc(R, sizeof(T) == 8)>
hipError_t launch_tile(mls_plan_s* P, const T* wts, hipStream_t s, const StencilOpts& o) {
  if (P->stencil_zc != ZC) return hipErrorInvalidValue;   // the tile table is laid out for another depth
  StencilLaunch L;
  const int t = stencil_levels(P, P->d_rows, wts, o, L);
  k_stencil_tile<T, R, ZC, kStencilWaves><<<t, 64 * kStencilWaves, 0, s>>>(L, P->d_tiles);
  return hipGetLastError();
}

template <int R, int ZC, int NCH>
hipError_t launch_slab(mls_plan_s* P, hipStream_t s, const StencilOpts& o) {
  if (P->stencil_zc != ZC) return hipErrorInvalidValue;   // as launch_tile
  StencilLaunch L;
  const int t = stencil_levels(P, P->d_rows, P->d_row_w_tile, o, L);
  k_stencil_slab<R, ZC, NCH, kStencilWaves><<<t, 64 * kStencilWaves, 0, s>>>(L, P->d_tiles);
  return hipGetLastError();
}

hipError_t launch_slab_f64(mls_plan_s* P, int R, hipStream_t s, const StencilOpts& o) {
  const bool deep = P->stencil_zc == 16;
  if (R <= 4) return launch_slab<4, 8, 1>(P, s, o);
  if (R <= 6) return launch_slab<6, 8, 1>(P, s, o);
  if (R <= 8) return deep ? launch_slab<8, 16, 2>(P, s, o) : launch_slab<8, 8, 2>(P, s, o);
  if (R <= 10) return launch_slab<10, 8, 3>(P, s, o);
  if (R <= 12) return deep ? launch_slab<12, 16, 5>(P, s, o) : launch_slab<12, 8, 4>(P, s, o);
  return hipErrorInvalidValue;
}

hipError_t launch_tile_f64(mls_plan_s* P, int R, hipStream_t s, const StencilOpts& o) {
  const double* w = P->d_row_w_tile;
  switch (R) {
    case 1: case 2: case 3: case 4: return launch_tile<double, 4>(P, w, s, o);
    case 5: case 6: return launch_tile<double, 6>(P, w, s, o);
    case 7: case 8: return launch_slab_f64(P, R, s, o);
    default: return hipErrorInvalidValue;
  }
}

// FP32 tiles reach R = 12: (8 + 2R)^2 (8 + 2R) floats, 88 KB at R = 10 and
// 128 KB at R = 12 (one block per CU; an FP64 tile of that size does not fit)
hipError_t launch_tile_f32(mls_plan_s* P, int R, hipStream_t s, const StencilOpts& o) {
  const float* w = P->d_row_wf_tile;
  switch (R) {
    case 1: case 2: case 3: case 4: return launch_tile<float, 4>(P, w, s, o);
    case 5: case 6: return launch_tile<float, 6>(P, w, s, o);
    case 7: case 8: return launch_tile<float, 8>(P, w, s, o);
    case 9: case 10: return launch_tile<float, 10>(P, w, s, o);
    case 11: case 12: return launch_tile<float, 12>(P, w, s, o);
    default: return hipErrorInvalidValue;
  }
}

template <int R>
hipError_t launch_mfma(mls_plan_s* P, hipStream_t s, const StencilOpts& o) {
  if (P->stencil_zc != 16) return hipErrorInvalidValue;   // as launch_tile
  StencilLaunch L;
  const int t = stencil_levels(P, P->d_rows_mfma, P->d_mfma_a, o, L);
  k_stencil_mfma<R, kStencilWaves><<<t, 64 * kStencilWaves, 0, s>>>(L, P->d_tiles);
  return hipGetLastError();
}

hipError_t launch_tile_mfma(mls_plan_s* P, int R, hipStream_t s, const StencilOpts& o) {
  switch (R) {
    case 1: case 2: case 3: case 4: return launch_mfma<4>(P, s, o);
    case 5: case 6: return launch_mfma<6>(P, s, o);
    default: return hipErrorInvalidValue;
  }
}

int stencil_path(const mls_plan_s* P) {
  if (P->levels < 2) return MLS_STENCIL_NONE;
  const int R = stencil_window(P);
  if (P->stencil_mfma) return MLS_STENCIL_TILE_MFMA_F32;
  if (P->stencil_kernel == 1 && P->precision == MLS_MIXED && R >= 1 && R <= 12) return MLS_STENCIL_TILE_F32;
  if (P->stencil_kernel == 1 && R >= 1 && R <= 8) return MLS_STENCIL_TILE_F64;
  if (R >= 1 && R <= 12) return MLS_STENCIL_STREAM_F64;
  return MLS_STENCIL_TAPS_F64;
}

// Atoms up to which the FP32 tiles add up the partial sums of the charges
// themselves: one read per thread, against a launch of 4 us on the chain.  Beyond,
// several reads per thread of every tile.
constexpr int64_t kSumRows = 65536;

bool stencil_adds_sum(const mls_plan_s* P, int64_t n) {
  return n > 0 && n + kSortedPad <= kSumRows && stencil_path(P) == MLS_STENCIL_TILE_F32;
}

bool coarsest_restricts(const mls_plan_s* P) {
  const int path = stencil_path(P);
  return P->levels >= 2 && P->lv[P->levels - 1].g.size <= kJointCoarse &&
         (path == MLS_STENCIL_TILE_F32 || path == MLS_STENCIL_TILE_F64 || path == MLS_STENCIL_STREAM_F64);
}

hipError_t launch_stencils(mls_plan_s* P, int n, hipStream_t s, int kmax, bool coarsest) {
  if (P->levels < 2) return coarsest ? launch_coarsest(P, s) : hipSuccess;
  const int R = stencil_window(P);
  const int path = stencil_path(P);
  StencilOpts o;
  o.kmax = kmax <= 0 || kmax > P->levels - 1 ? P->levels - 1 : kmax;
  if (stencil_adds_sum(P, n)) o.sum_rows = n + (P->mixing == MLS_LORENTZ_BERTHELOT ? kSortedPad : 0);
  o.coarsest = coarsest;
  if (path == MLS_STENCIL_TILE_F32) return launch_tile_f32(P, R, s, o);
  if (path == MLS_STENCIL_STREAM_F64) return launch_slab_f64(P, R, s, o);
  if (path == MLS_STENCIL_TILE_F64) return launch_tile_f64(P, R, s, o);
  if (path == MLS_STENCIL_TILE_MFMA_F32) {
    o.coarsest = false;
    const hipError_t e = launch_tile_mfma(P, R, s, o);
    return e != hipSuccess || !coarsest ? e : launch_coarsest(P, s);
  }
  const int ntaps = (int)P->taps.size();
  const ChainSet cs = chains(P);
  for (int v = 0; v < cs.n; ++v)
    for (int k = 1; k <= o.kmax; ++k) {
      const Level& L = (*cs.lv[v])[k - 1];
      const double scale = std::ldexp(1.0, -6 * (k - 1));
      k_stencil_taps_f64<<<nblocks(L.g.size, kBlock), kBlock, 0, s>>>(L.q, L.g, P->d_taps, ntaps, scale, L.e);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
  return coarsest ? launch_coarsest(P, s) : hipSuccess;
}

hipError_t launch_coarsest(mls_plan_s* P, hipStream_t s) {
  const ChainSet cs = chains(P);
  ChainArgs<Coarsest> c;
  for (int v = 0; v < cs.n; ++v) {
    const Level& L = (*cs.lv[v])[P->levels - 1];
    c.add(CoarsestArgs{L.q, L.g, P->d_Kl, L.e, 1, 0});
  }
  return launch_chains(c, coarsest_blocks(P->lv[P->levels - 1].g, 1, 0), s);
}

bool stencil_tile_ok(int R, int zc, bool f64) {
  if (R < 1 || R > 8) return false;
  if (zc == 8) return true;
  return zc == 16 && R <= 6 && !f64;
}

template <class T, int R, int ZC>
hipError_t launch_tiles_batched(const BatchPhase& ph, hipStream_t s) {
  const StencilLevel* lv = (const StencilLevel*)ph.args;
  const int4* work = (const int4*)ph.work;
  if (ph.grid > 0 && ph.grid < ph.nwork)
    k_stencil_tile_batched<T, R, ZC, kStencilWaves><<<ph.grid, 64 * kStencilWaves, 0, s>>>(lv, work, ph.nwork);
  else
    k_stencil_tile_each<T, R, ZC, kStencilWaves><<<ph.nwork, 64 * kStencilWaves, 0, s>>>(lv, work);
  return hipGetLastError();
}

hipError_t launch_slabs_batched(const BatchPhase& ph, hipStream_t s) {
  const int grid = ph.grid > 0 ? std::min(ph.grid, ph.nwork) : ph.nwork;
  k_stencil_slab_batched<8, 8, 2, kStencilWaves><<<grid, 64 * kStencilWaves, 0, s>>>((const StencilLevel*)ph.args,
                                                                                    (const int4*)ph.work, ph.nwork);
  return hipGetLastError();
}

// Batched phases of this file.  Stencil variant = window template (4, 6, 8)
// | z extent << 8 | 0x10000 for FP32 tiles.
hipError_t launch_batched_stencil(const BatchPhase& ph, hipStream_t s) {
  if (ph.nwork == 0) return hipSuccess;
  if (ph.kernel == BK_COARSEST) return launch_batched_phase<Coarsest>(ph, s);
  if (ph.kernel != BK_STENCIL) return hipErrorInvalidValue;
  const int R = ph.variant & 0xff, zc = (ph.variant >> 8) & 0xff;
  const bool f32 = (ph.variant & 0x10000) != 0;
  if (f32) {
    if (R == 4 && zc == 16) return launch_tiles_batched<float, 4, 16>(ph, s);
    if (R == 4 && zc == 8) return launch_tiles_batched<float, 4, 8>(ph, s);
    if (R == 6 && zc == 16) return launch_tiles_batched<float, 6, 16>(ph, s);
    if (R == 6 && zc == 8) return launch_tiles_batched<float, 6, 8>(ph, s);
    if (R == 8 && zc == 8) return launch_tiles_batched<float, 8, 8>(ph, s);
  } else {
    if (R == 4 && zc == 8) return launch_tiles_batched<double, 4, 8>(ph, s);
    if (R == 6 && zc == 8) return launch_tiles_batched<double, 6, 8>(ph, s);
    if (R == 8 && zc == 8) return launch_slabs_batched(ph, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace mls
