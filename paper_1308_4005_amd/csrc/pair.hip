// Local part of the evaluation step (eq:evaluation with k = 0): for every
// atom i, over all atoms j and periodic images n with (j,n) != (i,0) and
// r = |x_i - x_j - n o L| < a,
//     e0_i   = sum xi_j g_0(r),        g_0 = r^-6 - a^-6 gamma(r/a)   (eq:g_0)
//     F_i   += xi_i sum xi_j (g_0'(r)/r) d,   d = x_i - x_j - n o L
// with g_0'(r)/r = -6 r^-8 + a^-8 (15 rho^10 - 9 rho^22), rho = r/a, from
// eq:gamma.  Pairs are found through the linked cells of the binning step;
// the neighbour-cell offsets carry their image shift, which covers boxes
// narrower than three cells.
#include <type_traits>

#include "device_math.h"
#include "mls_internal.h"

namespace mls {
namespace {

constexpr int kBlock = 128;

// 1/s for g_0(r) and g_0'(r)/r from s = r^2 (caller guarantees 0 < s < a^2).
// FP64: the hardware reciprocal refined by two Newton steps (cheaper than
// the correctly rounded division sequence, accurate to the last bit or so).
// FP32: the hardware reciprocal alone (within about one ulp; the mixed path's
// force error stays two orders below its 1e-5 bound).
__device__ __forceinline__ double recip(double s) {
  double r = __builtin_amdgcn_rcp(s);
  r = fma(fma(-s, r, 1.0), r, r);
  return fma(fma(-s, r, 1.0), r, r);
}
__device__ __forceinline__ float recip(float s) { return __builtin_amdgcn_rcpf(s); }

// g_0(r) and g_0'(r)/r from s = r^2 (caller guarantees 0 < s < a^2), with
// rho = r/a and v = rho^12:
//   g_0     = r^-6 - a^-6 gamma_k(rho),            gamma_k = sum_j gc[j] v^j
//   g_0'/r  = -6 r^-8 - a^-8 rho^10 sum_j gq[j] v^j
// K = 2 is eq:gamma with its constants folded in; K = 0 takes any member of
// the family (k <= 4) from the plan's coefficients, zero-padded to degree 4.
template <class T, int K, class C>
__device__ __forceinline__ void g0_pair(T s, const C& pc, T& g, T& fr) {
  T ir2 = recip(s);
  T ir6 = ir2 * ir2 * ir2;
  T u = s * pc.inv_a2;         // rho^2
  T u2 = u * u;
  if constexpr (K == 2) {
    // eq:gamma: gamma = 15/8 - 5/4 v + 3/8 v^2 with v = rho^12 = u3^2, and
    // gamma'(rho)/rho = -15 rho^10 + 9 rho^22 = rho^10 (9 v - 15)
    const T u3 = u2 * u;
    const T v = u3 * u3;
    // FP64 takes the constants from the arguments (scalar registers: computed
    // here they held ten vector registers, two more than five waves per SIMD
    // leave); FP32 has room for them
    T c[5];
    if constexpr (sizeof(T) == 8) {
      for (int k = 0; k < 5; ++k) c[k] = pc.k2[k];
    } else {
      c[0] = T(-15.0 / 8.0) * pc.inv_a6;
      c[1] = T(5.0 / 4.0) * pc.inv_a6;
      c[2] = T(-3.0 / 8.0) * pc.inv_a6;
      c[3] = T(-9) * pc.inv_a8;
      c[4] = T(15) * pc.inv_a8;
    }
    g = ir6 + fma(v, fma(v, c[2], c[1]), c[0]);
    const T t = fma(v, c[3], c[4]);
    fr = fma(T(-6) * ir6, ir2, (u3 * u2) * t);
  } else {
    T u4 = u2 * u2;
    T u5 = u4 * u;
    T u6 = u4 * u2;
    T P = pc.gc[4];
    P = fma(P, u6, pc.gc[3]);
    P = fma(P, u6, pc.gc[2]);
    P = fma(P, u6, pc.gc[1]);
    P = fma(P, u6, pc.gc[0]);
    T Q = pc.gq[3];
    Q = fma(Q, u6, pc.gq[2]);
    Q = fma(Q, u6, pc.gq[1]);
    Q = fma(Q, u6, pc.gq[0]);
    g = ir6 - pc.inv_a6 * P;
    fr = T(-6) * ir6 * ir2 - pc.inv_a8 * u5 * Q;
  }
}

// Source weight of a pair: xi_j (geometric mixing), or under Lorentz-Berthelot
// e_j ((sigma_i + sigma_j) / 2)^6 with e_j = sqrt(2 eps_j) = xs.w, so that the
// target's factor e_i times it is C_ij of eq:xi-lj.
template <bool LB>
__device__ __forceinline__ double src_weight(double wj, const double* __restrict__ sig, double sig_i, int j) {
  if constexpr (LB) {
    const double m = 0.5 * (sig_i + sig[j]);
    const double m3 = m * m * m;
    return wj * (m3 * m3);
  } else {
    return wj;
  }
}

// FP64: one thread per cell-sorted target atom.
template <int K, bool LB = false>
struct PairGeneric {
  using Args = PairArgs;
  static constexpr int kThreads = kBlock;
  static __device__ void run(const Args& a, int blk) {
    const int s = blk * kBlock + threadIdx.x;
    if (s >= a.n) return;
    const CellGeom& g = a.g;
    const PairConst& pc = a.pc;
    const double4* __restrict__ xs = a.xs;
    const double4 xi = xs[s];
    const double sig_i = LB ? a.sig[s] : 0.0;
    const int c = a.cell_s[s];
    const int cx = c % g.nc[0], cy = (c / g.nc[0]) % g.nc[1], cz = c / (g.nc[0] * g.nc[1]);
    double e = 0.0, fx = 0.0, fy = 0.0, fz = 0.0;
    for (int oz = -g.noff[2]; oz <= g.noff[2]; ++oz) {
      int tz = cz + oz;
      const int iz = floordiv(tz, g.nc[2]);
      tz -= iz * g.nc[2];
      const double sz = iz * g.L[2];
      for (int oy = -g.noff[1]; oy <= g.noff[1]; ++oy) {
        int ty = cy + oy;
        const int iy = floordiv(ty, g.nc[1]);
        ty -= iy * g.nc[1];
        const double sy = iy * g.L[1];
        for (int ox = -g.noff[0]; ox <= g.noff[0]; ++ox) {
          int tx = cx + ox;
          const int ix = floordiv(tx, g.nc[0]);
          tx -= ix * g.nc[0];
          const double sx = ix * g.L[0];
          const bool home = (ix | iy | iz) == 0;
          const int t = (tz * g.nc[1] + ty) * g.nc[0] + tx;
          const int j0 = a.cstart[t], j1 = a.cstart[t + 1];
          for (int j = j0; j < j1; ++j) {
            const double4 xj = xs[j];
            const double dx = xi.x - (xj.x + sx);
            const double dy = xi.y - (xj.y + sy);
            const double dz = xi.z - (xj.z + sz);
            const double r2 = dx * dx + dy * dy + dz * dz;
            if (r2 < pc.a2 && !(home && j == s)) {
              double gg, fr;
              g0_pair<double, K>(r2, pc, gg, fr);
              const double wj = src_weight<LB>(xj.w, a.sig, sig_i, j);
              e += wj * gg;
              const double f = wj * fr;
              fx += f * dx;
              fy += f * dy;
              fz += f * dz;
            }
          }
        }
      }
    }
    a.e0[s] = e;
    a.floc[3 * (size_t)s + 0] = xi.w * fx;
    a.floc[3 * (size_t)s + 1] = xi.w * fy;
    a.floc[3 * (size_t)s + 2] = xi.w * fz;
  }
};

// FP64, one wave per target, for boxes too narrow for half-cutoff cells
// (few, crowded cells, often several images of one atom inside the cutoff).
// The wave walks the target's neighbour cells as contiguous runs of sorted
// atoms (a run ends where the periodic image changes) and its 64 lanes split
// each run; the lane sums are added in LDS.  Same cells, images and pairs as
// PairGeneric.
template <int K, bool LB = false>
struct PairWave {
  using Args = PairArgs;
  static constexpr int kThreads = 64;
  static __device__ void run(const Args& a, int s) {
    __shared__ double red[4][64];
    const int lane = threadIdx.x;
    const CellGeom& g = a.g;
    const PairConst& pc = a.pc;
    const double4* __restrict__ xs = a.xs;
    const double4 xi = xs[s];
    const double sig_i = LB ? a.sig[s] : 0.0;
    const int c = a.cell_s[s];
    const int cx = c % g.nc[0], cy = (c / g.nc[0]) % g.nc[1], cz = c / (g.nc[0] * g.nc[1]);
    double e = 0.0, fx = 0.0, fy = 0.0, fz = 0.0;
    for (int oz = -g.noff[2]; oz <= g.noff[2]; ++oz) {
      int tz = cz + oz;
      const int iz = floordiv(tz, g.nc[2]);
      tz -= iz * g.nc[2];
      const double sz = iz * g.L[2];
      for (int oy = -g.noff[1]; oy <= g.noff[1]; ++oy) {
        int ty = cy + oy;
        const int iy = floordiv(ty, g.nc[1]);
        ty -= iy * g.nc[1];
        const double sy = iy * g.L[1];
        const int row = (tz * g.nc[1] + ty) * g.nc[0];
        int u = cx - g.noff[0];
        const int uend = cx + g.noff[0];
        while (u <= uend) {
          const int ix = floordiv(u, g.nc[0]);
          const int tx = u - ix * g.nc[0];
          const int run = min(uend - u + 1, g.nc[0] - tx);
          const int j1 = a.cstart[row + tx + run];
          const double sx = ix * g.L[0];
          const bool home = (ix | iy | iz) == 0;
          for (int j = a.cstart[row + tx] + lane; j < j1; j += 64) {
            const double4 xj = xs[j];
            const double dx = xi.x - (xj.x + sx);
            const double dy = xi.y - (xj.y + sy);
            const double dz = xi.z - (xj.z + sz);
            const double r2 = dx * dx + dy * dy + dz * dz;
            if (r2 < pc.a2 && !(home && j == s)) {
              double gg, fr;
              g0_pair<double, K>(r2, pc, gg, fr);
              const double wj = src_weight<LB>(xj.w, a.sig, sig_i, j);
              e += wj * gg;
              const double f = wj * fr;
              fx += f * dx;
              fy += f * dy;
              fz += f * dz;
            }
          }
          u += run;
        }
      }
    }
    red[0][lane] = e;
    red[1][lane] = fx;
    red[2][lane] = fy;
    red[3][lane] = fz;
    __syncthreads();
    for (int off = 32; off > 0; off >>= 1) {
      if (lane < off)
        for (int k = 0; k < 4; ++k) red[k][lane] += red[k][lane + off];
      __syncthreads();
    }
    if (lane == 0) {
      a.e0[s] = red[0][0];
      a.floc[3 * (size_t)s + 0] = xi.w * red[1][0];
      a.floc[3 * (size_t)s + 1] = xi.w * red[2][0];
      a.floc[3 * (size_t)s + 2] = xi.w * red[3][0];
    }
  }
};

// FP64, filter-and-drain over half-cutoff cells: one wave of 64 lanes takes
// 64 consecutive cell-sorted targets.  Each lane visits the 5 x 5 rows
// of cells around its target's cell, skips rows whose y/z gap to the target
// is at least a, and trims every other row to the cells the cutoff sphere
// can reach along x (at most two runs of cells: one per periodic image).  A
// cheap FP32 distance test (both precisions; see pair_scan_f32) appends
// sources inside the cutoff to the lane's LDS queue, four candidates per step;
// whenever a queue may overflow all lanes drain up to kDrain of their entries
// through the full g_0 evaluation (FP64: the newest, so the slot of the next
// entry is its count alone; FP32: the oldest, the rest moves up), and at the
// end everything left, so the expensive arithmetic runs on nearly full waves
// instead of being masked per candidate.  An FP64 entry packs the source
// index (< 2^25) with two bits per dimension for its image.
//
// At 10^6 atoms the vector ALU issues 80 (FP64) to 97 % (FP32) of the time and
// the L1 serves a line in three of four cycles, so what counts is the number
// of instructions: of a filter step (48 to 50 vector ones for four candidates), of a
// drained entry (FP64 52, FP32 42) and of a row's set-up (about 75); idle lanes
// load nothing.  With 57, 67, 57 and 130 the kernel took 516 us in FP64
// instead of 454 (10^6 atoms at density 0.8, a = 3), in FP32 392 instead of 376.
constexpr int kWaveQ = 64;    // lanes per block (one wave)
// Entries per lane: with the sums' 2 KB, 8 KB of LDS per wave, and held to 96
// VGPRs (kWavesPerSimd), 20 waves share a CU.  32 entries and 16 waves: fewer
// and fuller drains, but an evaluation of 10^6 atoms 777 us instead of 745.
constexpr int kQueue = 24;
// The FP32 kernel's queue and its table of shifts: 5.2 KB of LDS, 28 waves per
// CU (its VGPRs allow as many).
constexpr int kQueueF = 16;   // entries per lane of the FP32 kernel
constexpr int kBatchF = 4;    // candidates per filter step

// 16-byte load from a 4-byte aligned address (four consecutive floats)
// element j of a uniform array through a 32-bit byte offset (the caller
// guarantees j * sizeof(T) < 2^32), so the load takes its base from scalar
// registers instead of a 64-bit per-lane address
template <class T>
__device__ __forceinline__ const T& at32(const T* base, int j) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + (unsigned)j * (unsigned)sizeof(T));
}

// the same for the element that the low 24 bits of ent name
template <class T>
__device__ __forceinline__ const T& at24(const T* base, int ent) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + __umul24((unsigned)ent, (unsigned)sizeof(T)));
}

template <class T>
__device__ __forceinline__ const T& at24(const gptr<const T>& base, int ent) {
  return at24((const T*)base, ent);
}

__device__ __forceinline__ float4 load4f(const float* p) {
  float4 v;
  __builtin_memcpy(&v, p, sizeof(v));   // 4-byte aligned 16-byte load
  return v;
}

// image indices -1, 0, 1 as two's-complement fields
__device__ __forceinline__ int image_bits(int ix, int iy, int iz) { return (ix & 3) | ((iy & 3) << 2) | ((iz & 3) << 4); }

// Four FP64 sums of one lane (energy, force x, y, z) of the FP64 kernel, kept in
// LDS at stride kWaveQ while the lane's rows are scanned: only the drains read and write
// them, so the filter loop carries none of them (their eight registers would
// cost the fifth wave per SIMD).
// Each drain starts with a compiler memory barrier (sums_fence): without it
// the sums were hoisted out of the loop into registers again (the queue and
// the sums are distinct LDS arrays), and volatile accesses instead made every
// update wait for its own load.
struct LaneSums {
  double* s;   // slot 0 of this lane
  __device__ __forceinline__ double& operator[](int k) const { return s[k * kWaveQ]; }
};

__device__ __forceinline__ void sums_fence() { asm volatile("" ::: "memory"); }

// Per-lane sums of a pair kernel: e_0 and the force in LDS, queue state in
// registers
struct PairAcc {
  LaneSums a;
  int cnt;   // entries in the lane's queue
};

// Per-lane sums of the repulsive term (MD entry points): sum_j sqrt(C12_j)
// r^-12 and sum_j 12 sqrt(C12_j) r^-14 d over the pairs with r < rc.  Kept in
// registers: 2 KB more LDS per wave would cost the kernels occupancy.
struct RepAcc {
  double v[4];
  __device__ __forceinline__ double& operator[](int k) { return v[k]; }
  __device__ __forceinline__ double operator[](int k) const { return v[k]; }
};

// The kernels' LDS for the sums: four slots per lane.
constexpr int kSumSlots = 4 * kWaveQ;

// A drain during the scan consumes at most this many entries per lane: the
// lane that forced it is then well below the limit, and lanes with few
// entries idle for fewer steps than in a drain to empty.
constexpr int kDrain = 8;

// Full g_0 evaluation of the newest queued sources of each lane, up to `limit`.
// The loop body has no branches: slots past a lane's count (and the target
// itself) evaluate a harmless pair with zero weight, adding exactly 0.
template <int K, bool LB, bool R>
__device__ __forceinline__ void pair_drain_f64(const int* queue, int limit, int lane, int self_ent,
                                               int safe_ent, const double4& xi, const double4* __restrict__ xs,
                                               const CellGeom& g, const PairConst& pc, const double* __restrict__ sig,
                                               double sig_i, PairAcc& A, const PairRep& rp, RepAcc& B) {
  sums_fence();
  const double r2_idle = 0.25 * pc.a2;
  const int done = min(A.cnt, limit);
  const int* q0 = queue + (A.cnt - done) * kWaveQ + lane;
  // the lane's running sums, added to pair by pair as if held throughout
  double ae = A.a[0], afx = A.a[1], afy = A.a[2], afz = A.a[3];
  double be = 0.0, bfx = 0.0, bfy = 0.0, bfz = 0.0;
  if constexpr (R) {
    be = B[0];
    bfx = B[1];
    bfy = B[2];
    bfz = B[3];
  }
  // loop-carried: an idle lane keeps what it read last (at first its own row)
  double4 xj = xi;
  for (int t = 0; t < limit && __any(t < done); ++t, q0 += kWaveQ) {
    const int q = *q0;
    const bool ok = (t < done) & (q != self_ent);
    const int ent = ok ? q : safe_ent;
    const int j = (int)((unsigned)ent >> 6);
    if (ok) xj = at32(xs, j);
    const double dx = fma((double)((ent << 30) >> 30), -g.L[0], xi.x) - xj.x;
    const double dy = fma((double)((ent << 28) >> 30), -g.L[1], xi.y) - xj.y;
    const double dz = fma((double)((ent << 26) >> 30), -g.L[2], xi.z) - xj.z;
    const double d2 = dx * dx + dy * dy + dz * dz;
    // the FP32 filter passes a superset: the pair set is decided here, in
    // FP64, by r^2 < a^2 (rejected entries add exactly 0)
    const bool in = ok & (d2 < pc.a2);
    const double r2 = in ? d2 : r2_idle;
    double gg, fr;
    g0_pair<double, K>(r2, pc, gg, fr);
    const double wj = in ? src_weight<LB>(xj.w, sig, sig_i, j) : 0.0;
    ae += wj * gg;
    const double f = wj * fr;
    afx += f * dx;
    afy += f * dy;
    afz += f * dz;
    if constexpr (R) {
      const double ir2 = recip(r2);
      const double ir6 = ir2 * ir2 * ir2;
      const double v = (in && r2 < rp.rc2 ? rp.x12[j] : 0.0) * ir6 * ir6;
      const double fv = 12.0 * v * ir2;
      be += v;
      bfx += fv * dx;
      bfy += fv * dy;
      bfz += fv * dz;
    }
  }
  A.a[0] = ae;
  A.a[1] = afx;
  A.a[2] = afy;
  A.a[3] = afz;
  if constexpr (R) {
    B[0] = be;
    B[1] = bfx;
    B[2] = bfy;
    B[3] = bfz;
  }
  A.cnt -= done;
}

// Four registers whatever they hold: what lanes without a load of their own
// pass on, where a mask then discards it.  (Kept live instead, the last
// candidates took twelve registers through every drain.)
__device__ __forceinline__ float4 any4() {
  float4 v;
  asm volatile("" : "=v"(v.x), "=v"(v.y), "=v"(v.z), "=v"(v.w));
  return v;
}

// The filter's three coordinate arrays (absolute x, cell-relative y and z).
struct FilterRows {
  const float *x, *y, *z;
  __device__ __forceinline__ FilterRows(const float* xf, int stride) : x(xf), y(xf + stride), z(xf + 2 * (size_t)stride) {}
};

// One filter step: the four candidates at byte offset `off` of the arrays
// against the target's ax, ay, az, those past `off1` left out.  Every
// candidate writes its entry to the lane's next free queue slot, which the
// count passes only on a hit.  Few and cheap instructions are the point: the
// byte offset serves the loads, the entries and the tests of the run's end
// (against limits set once per run), and the slot follows from the count by
// one shift and add.  IB: bits below the source index in an entry (0: the
// run's bits lie above it).
template <int IB>
struct FilterRun {
  int off, lim[4];
  float ax, ay, az;
  int bits;
  __device__ __forceinline__ FilterRun(int j0, int j1, float ax_, float ay_, float az_, int bits_)
      : off(4 * j0), ax(ax_), ay(ay_), az(az_), bits(bits_) {
    // candidate b of a step counts while off < 4 (j1 - b); an empty run: never
#pragma unroll
    for (int b = 0; b < 4; ++b) lim[b] = 4 * j1 - 4 * b;
  }
  __device__ __forceinline__ bool more() const { return off < lim[0]; }
  __device__ __forceinline__ void load(const FilterRows& f, float4& X, float4& Y, float4& Z) const {
    X = load4f(reinterpret_cast<const float*>(reinterpret_cast<const char*>(f.x) + (unsigned)off));
    Y = load4f(reinterpret_cast<const float*>(reinterpret_cast<const char*>(f.y) + (unsigned)off));
    Z = load4f(reinterpret_cast<const float*>(reinterpret_cast<const char*>(f.z) + (unsigned)off));
  }
  __device__ __forceinline__ int test(const float4& X, const float4& Y, const float4& Z, float a2f, int* qlane, int cnt) {
    const float xb[4] = {X.x, X.y, X.z, X.w}, yb[4] = {Y.x, Y.y, Y.z, Y.w}, zb[4] = {Z.x, Z.y, Z.z, Z.w};
    const int ent0 = (IB ? off << (IB - 2) : off >> 2) | bits;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const float dx = ax - xb[b], dy = ay - yb[b], dz = az - zb[b];
      const float r2 = fmaf(dz, dz, fmaf(dx, dx, dy * dy));
      const bool hit = (off < lim[b]) & (r2 < a2f);
      qlane[kWaveQ * cnt] = ent0 + (b << IB);
      cnt += hit ? 1 : 0;
    }
    off += 16;
    return cnt;
  }
};

// Scan sources [j, j1) seen through image bits `img` (convergent: every lane
// calls it; lanes with an empty range just take part in the votes).
// Candidates are tested by the FP32 filter of the mixed kernel (threshold a2f
// widened for FP32 rounding): it passes a superset of the pairs inside the
// cutoff, and the drain decides each pair in FP64.  Reads may run up to three
// rows past j1 (padded array); lanes past their range load nothing, and the end
// test masks what they hold.  One loop level, the drain inside it: the
// accumulators change only on the drain path.
template <int K, bool LB, bool R>
__device__ __forceinline__ void pair_scan_f64(FilterRun<6> r, int* __restrict__ queue, int lane, int self_ent,
                                              int safe_ent, const double4& xi, const double4* __restrict__ xs,
                                              const FilterRows& f, const CellGeom& g, const PairConst& pc,
                                              const double* __restrict__ sig, double sig_i, PairAcc& A,
                                              const PairRep& rp, RepAcc& B) {
  int* const qlane = queue + lane;
  int cnt = A.cnt;
  while (__any(r.more())) {
    float4 X = any4(), Y = any4(), Z = any4();
    if (r.more()) r.load(f, X, Y, Z);
    cnt = r.test(X, Y, Z, pc.a2f, qlane, cnt);
    if (__builtin_expect(__any(cnt > kQueue - 4), 0)) {
      A.cnt = cnt;
      pair_drain_f64<K, LB, R>(queue, kDrain, lane, self_ent, safe_ent, xi, xs, g, pc, sig, sig_i, A, rp, B);
      cnt = A.cnt;
    }
  }
  A.cnt = cnt;
}

// The two runs [j0, j1), [k0, k1) of one row of cells (x images ix1, ix2) that
// a target's cutoff sphere can reach; empty for an idle lane.
struct RowRuns {
  int j0, j1, ix1, k0, k1, ix2;
};

// Rows are chosen and trimmed in the target's cell-relative FP32 coordinates.
// The gaps are shrunk and the reach grown by margins (1e-5 of a cell, 2e-5 of
// the cutoff) far above their FP32 rounding (~1e-7), so no cell that holds a
// source inside the cutoff is ever skipped; mg, the skin margin of neighbour
// reuse (atoms may sit that far outside their cells), does the same.
struct RowTrim {
  const int* cstart;
  float w[3], inv_wx, a2m, mg;
  int nc[3];
  __device__ __forceinline__ RowTrim(const int* start, const CellGeom& g, const float* wf, float a2)
      : cstart(start), w{wf[0], wf[1], wf[2]}, inv_wx(1.0f / wf[0]), a2m(a2 * (1.0f + 2e-5f)), mg((float)g.margin),
        nc{g.nc[0], g.nc[1], g.nc[2]} {}
  // distance of a target at cell-relative coordinate x to the cells d away
  __device__ __forceinline__ float gap(int k, int d, float x) const {
    return d == 0 ? 0.0f
                  : fmaxf(0.0f, (d > 0 ? fmaf((float)d, w[k], -x) : fmaf((float)(-d - 1), w[k], x)) - 1e-5f * w[k] - mg);
  }
  // Runs of the row whose first cell is `row`, rem = a^2 minus the squared
  // gaps in y and z, of a target at cell-relative x in cell cx.  Most waves
  // have no lane whose run crosses the periodic edge.
  __device__ __forceinline__ RowRuns runs(int cx, float x, bool active, float rem, int row) const {
    const float reach = 1.0f + 2e-5f;
    const int nc0 = nc[0];
    int clo = 0, chi = -1;
    if (active && rem > 0.0f) {
      // hardware square root (about 1 ulp): far inside the margin
      const float rx = fmaf(__builtin_amdgcn_sqrtf(rem), reach, 1e-5f * w[0] + mg);
      clo = cx + max(-2, (int)floorf((x - rx) * inv_wx));
      chi = cx + min(2, (int)floorf((x + rx) * inv_wx));
    }
    RowRuns r{0, 0, 0, 0, 0, 0};
    int lo1 = clo, hi1 = chi;
    if (__any((clo < 0) | (chi >= nc0))) {
      int lo2 = 0, hi2 = -1;
      if (clo < 0) {
        lo1 = clo + nc0; hi1 = nc0 - 1; r.ix1 = -1;
        lo2 = 0; hi2 = chi; r.ix2 = 0;
      } else if (chi >= nc0) {
        lo1 = clo; hi1 = nc0 - 1; r.ix1 = 0;
        lo2 = 0; hi2 = chi - nc0; r.ix2 = 1;
      }
      if (lo2 <= hi2) {
        r.k0 = at32(cstart, row + lo2);
        r.k1 = at32(cstart, row + hi2 + 1);
      }
    }
    if (lo1 <= hi1) {
      r.j0 = at32(cstart, row + lo1);
      r.j1 = at32(cstart, row + hi1 + 1);
    }
    return r;
  }
};

// A wave's walk over its targets' rows (dz, dy): scan(runs, dz, dy, iz, iy) for
// each, with the row's periodic images.  The wrapped row's first cell is kept
// by additions.  Span: the loops' bounds (RowSpan).
template <class Span, class Scan>
__device__ __forceinline__ void walk_rows(const RowTrim& w, const Span& span, int cx, int cy, int cz, float x, float y,
                                          float z, bool active, Scan&& scan) {
  const int slab = w.nc[1] * w.nc[0];
  for (int dz = span.z0(); dz <= span.z1(); ++dz) {
    const int uz = cz + dz;
    const int iz = uz < 0 ? -1 : (uz >= w.nc[2] ? 1 : 0);
    const int rowz = (uz - iz * w.nc[2]) * slab;
    const float gz = w.gap(2, dz, z);
    const float rem_z = w.a2m - gz * gz;
    const int y0 = span.y0(dz), y1 = span.y1(dz);
    int uy = cy + y0;
    int iy = uy < 0 ? -1 : (uy >= w.nc[1] ? 1 : 0);
    int rowy = (uy - iy * w.nc[1]) * w.nc[0];
    for (int dy = y0; dy <= y1; ++dy) {
      const float gy = w.gap(1, dy, y);
      scan(w.runs(cx, x, active, rem_z - gy * gy, rowz + rowy), dz, dy, iz, iy);
      rowy += w.nc[0];
      if (rowy == slab) {
        rowy = 0;
        ++iy;
      }
    }
  }
}

// Per-wave sum of one value (lanes of a 64-wide block).
__device__ __forceinline__ double wave_sum(double v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// Repulsive outputs of target sc: its sorted forces and, per block (one
// wave), the sum of sqrt(C12_i) times the lanes' energy sums.
__device__ __forceinline__ void store_rep(const PairRep& rp, bool active, int sc, int lane, int blk,
                                          const RepAcc& B) {
  double e = 0.0;
  if (active) {
    const double ci = rp.x12[sc];
    e = ci * B[0];
    rp.frep[3 * (size_t)sc + 0] = ci * B[1];
    rp.frep[3 * (size_t)sc + 1] = ci * B[2];
    rp.frep[3 * (size_t)sc + 2] = ci * B[3];
  }
  e = wave_sum(e);
  if (lane == 0) rp.partial[blk] = e;
}

// NS waves share a block's 64 targets (pair_split): each scans a contiguous
// share of the 25 rows (a simulation gives 3.7 to 5.6 filter steps per row: it
// takes as many as its slowest lane), and the waves' sums are added in wave
// order at the end.
template <int NS>
struct RowSpan {
  int wv = 0, r0 = 0, r1 = 25;
  __device__ __forceinline__ RowSpan() {
    if constexpr (NS > 1) {
      wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveQ);
      r0 = 25 * wv / NS;
      r1 = 25 * (wv + 1) / NS;
    }
  }
  // the rows as (dz, dy) loops over [-2, 2]^2
  __device__ __forceinline__ int z0() const { return NS > 1 ? r0 / 5 - 2 : -2; }
  __device__ __forceinline__ int z1() const { return NS > 1 ? (r1 - 1) / 5 - 2 : 2; }
  __device__ __forceinline__ int y0(int dz) const { return NS > 1 ? max(r0 - 5 * (dz + 2), 0) - 2 : -2; }
  __device__ __forceinline__ int y1(int dz) const { return NS > 1 ? min(r1 - 5 * (dz + 2), 5) - 3 : 2; }
};

// Outputs of a block of NS waves from their sums: e_0 and the force in
// `sums` (kSumSlots per wave), the repulsive ones (R) put into the waves' own
// parts of the drained queues (qw ints each) first.  Component c of every
// target is added up by wave c mod NS, over the waves in order.
template <int NS, bool R>
__device__ __forceinline__ void store_split(const double* sums, int* queues, int qw, const RepAcc& B, int wv, int lane,
                                            bool active, int sc, int blk, double wi, double* __restrict__ e0,
                                            double* __restrict__ floc, const PairRep& rp) {
  if constexpr (R) {
    double* const mine = reinterpret_cast<double*>(queues + wv * qw);
    sums_fence();
#pragma unroll
    for (int c = 0; c < 4; ++c) mine[c * kWaveQ + lane] = B[c];
  }
  __syncthreads();
  for (int c = wv; c < 4; c += NS) {
    double v = 0.0;
#pragma unroll
    for (int w = 0; w < NS; ++w) v += sums[w * kSumSlots + c * kWaveQ + lane];
    if (active) {
      if (c == 0) e0[sc] = v;
      else floc[3 * (size_t)sc + c - 1] = wi * v;
    }
    if constexpr (R) {
      v = 0.0;
#pragma unroll
      for (int w = 0; w < NS; ++w) v += reinterpret_cast<const double*>(queues + w * qw)[c * kWaveQ + lane];
      const double ci = active ? rp.x12[sc] : 0.0;
      if (c == 0) {
        const double e = wave_sum(active ? ci * v : 0.0);
        if (lane == 0) rp.partial[blk] = e;
      } else if (active) {
        rp.frep[3 * (size_t)sc + c - 1] = ci * v;
      }
    }
  }
}

template <int K, bool LB = false, bool R = false, int NS = 1>
struct PairTrimF64 {
  using Args = PairArgs;
  static constexpr int kThreads = kWaveQ * NS;
  static constexpr int kWavesPerSimd = NS == 1 && !R ? 5 : 1;   // with R's sums it would spill
  static __device__ void run(const Args& ar, int blk) {
  const double4* __restrict__ xs = ar.xs;
  const int* __restrict__ cstart = ar.cstart;
  const CellGeom& g = ar.g;
  const PairConst& pc = ar.pc;
  const int n = ar.n;
  __shared__ __attribute__((aligned(16))) int queues[NS * kQueue * kWaveQ];
  const int lane = threadIdx.x & (kWaveQ - 1);
  const RowSpan<NS> span;
  int* const queue = queues + span.wv * (kQueue * kWaveQ);
  const int k = blk * kWaveQ + lane;
  const bool active = k < n;
  const int sc = active ? k : n - 1;
  const double4 xi = xs[sc];
  const double sig_i = LB ? ar.sig[sc] : 0.0;
  const FilterRows f(ar.xf, ar.xf_stride);
  const float3 xf_i = make_float3(f.x[sc], f.y[sc], f.z[sc]);
  const int c = ar.cell_s[sc];
  const int cx = c % g.nc[0], cy = (c / g.nc[0]) % g.nc[1], cz = c / (g.nc[0] * g.nc[1]);
  // the target itself, seen in the home image, is skipped in the drain
  const int safe_ent = sc << 6;
  const int self_ent = active ? safe_ent | image_bits(0, 0, 0) : -1;
  __shared__ double all_sums[NS * kSumSlots];
  double* const sums = all_sums + span.wv * kSumSlots;
  for (int k = 0; k < kSumSlots / kWaveQ; ++k) sums[k * kWaveQ + lane] = 0.0;
  PairAcc A{LaneSums{sums + lane}, 0};
  RepAcc B{{0.0, 0.0, 0.0, 0.0}};
  const PairRep& rp = ar.rep;
  const RowTrim w(cstart, g, pc.wf, (float)pc.a2);
  walk_rows(w, span, cx, cy, cz, (float)(xi.x - cx * g.w[0]), xf_i.y, xf_i.z, active,
            [&](const RowRuns& r, int dz, int dy, int iz, int iy) {
    auto scan = [&](int j0, int j1, int ix) {
      if (!__any(j0 < j1)) return;
      const FilterRun<6> run(j0, j1, fmaf((float)-ix, pc.Lf[0], xf_i.x), fmaf((float)-dy, pc.wf[1], xf_i.y),
                             fmaf((float)-dz, pc.wf[2], xf_i.z), image_bits(ix, iy, iz));
      pair_scan_f64<K, LB, R>(run, queue, lane, self_ent, safe_ent, xi, xs, f, g, pc, ar.sig, sig_i, A, rp, B);
    };
    scan(r.j0, r.j1, r.ix1);
    scan(r.k0, r.k1, r.ix2);
  });
  pair_drain_f64<K, LB, R>(queue, kQueue, lane, self_ent, safe_ent, xi, xs, g, pc, ar.sig, sig_i, A, rp, B);
  if constexpr (NS > 1) {
    store_split<NS, R>(all_sums, queues, kQueue * kWaveQ, B, span.wv, lane, active, sc, blk, xi.w, ar.e0, ar.floc, rp);
    return;
  }
  if (active) {
    ar.e0[sc] = A.a[0];
    ar.floc[3 * (size_t)sc + 0] = xi.w * A.a[1];
    ar.floc[3 * (size_t)sc + 1] = xi.w * A.a[2];
    ar.floc[3 * (size_t)sc + 2] = xi.w * A.a[3];
  }
  if constexpr (R) store_rep(rp, active, sc, lane, blk, B);
  }
};

// ---------------------------------------------------------------------------
// FP32-mixed variant of the same scheme.  Sources carry cell-relative FP32
// coordinates (x - cx w, y - cy w, z - cz w) and their cell x index (exact in
// FP32) in the fourth component; xi is a separate FP32 array read only in the
// drain.  The displacement is rebuilt as
//   d_x = (cx_i - ix nc - cx_j) w_x + xr_i - xr_j,  d_y = yr_i - dy w_y - yr_j, ...
// with integer cell offsets, so no large coordinates enter FP32 arithmetic.
// Queue entries pack the source index (< 2^24) and, in the top byte, one of the
// 75 row offsets dz, dy and x images, looked up in LDS as shifts: cells along x
// and lengths along y and z.  Pair arithmetic is FP32; each drain sums its terms in
// FP32, and e_0 and the forces accumulate the drains' sums in FP64.
struct PairAccM {
  double a[4];  // e_0 and the force
  int cnt;      // entries in the lane's queue
};

// An FP32 drain consumes at most this many entries per lane: the lane that
// forced it is then below the limit again (at most 16 - 8 = 8 entries, one
// filter step adds at most 4 to the 12 that trigger a drain), and lanes with
// few entries idle for fewer steps than in a drain to empty (at 10^6 atoms the
// kernel took 0.44 ms with 8 and with 4, 0.46 ms with 12).
constexpr int kDrainF = 8;

// Per-lane target data of the FP32 scan.
struct PairLaneF {
  float xx, yy, zz;     // target cell-relative coordinates
  float cxf;            // target cell x index
  int self_ent;         // the target's own home-row entry (-1 for idle lanes)
  int safe_ent;         // the target as an entry: a valid source for idle drain slots
  const float4* shift;  // shifts by the entries' top byte (LDS)
  float sig_i;          // Lorentz-Berthelot: the target's sigma
  float xa;             // target absolute x (filter)
};

// Top byte of a queue entry: x image ix and row offsets dy, dz.
constexpr int kShifts = 75;
__device__ __forceinline__ int entry_bits(int ix, int dy, int dz) { return ((dz + 2) * 15 + (dy + 2) * 3 + ix + 1) << 24; }

// The shifts; dy w and dz w are exact (a power of two times w).  One wave.
__device__ __forceinline__ void fill_shifts(float4* tab, int lane, const CellGeom& g, const PairConstF& pc) {
  for (int c = lane; c < kShifts; c += kWaveQ) {
    const int dz = c / 15 - 2, dy = c / 3 % 5 - 2, ix = c % 3 - 1;
    tab[c] = make_float4((float)(-ix * g.nc[0]), (float)-dy * pc.w[1], (float)-dz * pc.w[2], 0.0f);
  }
}

// The (at most 16) terms of one drain are summed in FP32: e_0, the force and,
// with R, the repulsive energy and force.
template <bool R>
struct DrainF {
  float s[R ? 8 : 4] = {};
};

// One source (queue entry ent, rows xj, wsrc) through the full g_0
// evaluation, added to D; !ok: a harmless pair of weight 0, which adds exactly
// 0 (no branches).
template <int K, bool R, bool LB>
__device__ __forceinline__ void pair_term_f32(bool ok, int ent, const float4& xj, float wsrc, const PairLaneF& L,
                                              const float* __restrict__ sig, const PairConstF& pc, const PairRep& rp,
                                              DrainF<R>& D) {
  const float4 sh = L.shift[(unsigned)ent >> 24];
  const float dxv = fmaf((L.cxf + sh.x) - xj.w, pc.w[0], L.xx) - xj.x;
  const float dyv = (L.yy + sh.y) - xj.y;
  const float dzv = (L.zz + sh.z) - xj.z;
  const float r2 = ok ? fmaf(dzv, dzv, fmaf(dyv, dyv, dxv * dxv)) : 0.25f * pc.a2;
  float gg, fr;
  g0_pair<float, K>(r2, pc, gg, fr);
  float wj = wsrc;
  if constexpr (LB) {
    // source weight e_j ((sigma_i + sigma_j) / 2)^6, as in the FP64 kernels
    const float m = 0.5f * (L.sig_i + at24(sig, ent));
    const float m3 = m * m * m;
    wj *= m3 * m3;
  }
  D.s[0] = fmaf(wj, gg, D.s[0]);
  const float f = wj * fr;
  D.s[1] = fmaf(f, dxv, D.s[1]);
  D.s[2] = fmaf(f, dyv, D.s[2]);
  D.s[3] = fmaf(f, dzv, D.s[3]);
  if constexpr (R) {
    const float ir2 = recip(r2);
    const float ir6 = ir2 * ir2 * ir2;
    const float v = (ok && r2 < (float)rp.rc2 ? at24(rp.x12f, ent) : 0.0f) * ir6 * ir6;
    const float fv = 12.0f * v * ir2;
    D.s[4] += v;
    D.s[5] = fmaf(fv, dxv, D.s[5]);
    D.s[6] = fmaf(fv, dyv, D.s[6]);
    D.s[7] = fmaf(fv, dzv, D.s[7]);
  }
}

// Full g_0 evaluation of up to `limit` queued sources per lane, oldest first;
// what is left moves to the front (at most kQueueF - kDrainF entries).
template <int K, bool R, bool LB>
__device__ __forceinline__ void pair_drain_f32(int* queue, int limit, int lane, const PairLaneF& L,
                                               const float4* __restrict__ xr, const float* __restrict__ xif,
                                               const float* __restrict__ sig, const PairConstF& pc, PairAccM& A,
                                               const PairRep& rp, RepAcc& B) {
  int* const qlane = queue + lane;
  const int cnt = A.cnt;
  DrainF<R> D;
  // loop-carried: an idle lane keeps what it read last (at first its own row)
  float4 xj = make_float4(L.xx, L.yy, L.zz, L.cxf);
  float w = 0.0f;
  const int* q0 = qlane;
  for (int t = 0; t < limit && __any(t < cnt); ++t, q0 += kWaveQ) {
    const int q = *q0;
    // idle slots and the target itself load nothing and weigh 0
    const bool ok = (t < cnt) & (q != L.self_ent);
    const int ent = ok ? q : L.safe_ent;
    if (ok) {
      xj = at24(xr, ent);
      w = at24(xif, ent);
    }
    pair_term_f32<K, R, LB>(ok, ent, xj, ok ? w : 0.0f, L, sig, pc, rp, D);
  }
  for (int c = 0; c < 4; ++c) A.a[c] += (double)D.s[c];
  if constexpr (R)
    for (int c = 0; c < 4; ++c) B[c] += (double)D.s[4 + c];
  if (limit < kQueueF) {
    int rest[kQueueF - kDrainF];
#pragma unroll
    for (int u = 0; u < kQueueF - kDrainF; ++u) rest[u] = qlane[(kDrainF + u) * kWaveQ];
#pragma unroll
    for (int u = 0; u < kQueueF - kDrainF; ++u) qlane[u * kWaveQ] = rest[u];
  }
  A.cnt = cnt - min(cnt, limit);
}

// Scan sources of one row run.  The filter takes x from the absolute FP32
// coordinates (one subtraction per candidate instead of rebuilding the cell
// offset) and y, z cell-relative; its threshold a2f covers the rounding of
// absolute x (a few ulp of L), and the few extra pairs it passes, just outside
// a, add g_0 ~ 0 in the drain, which rebuilds the displacement exactly from
// the cell-relative data.  The coordinates are three arrays, so one 16-byte
// load brings one coordinate of a batch of four candidates; lanes past the end
// of their run load nothing, and the end test masks them.  One loop level, the
// drain inside it: the accumulators change only on the drain path (a loop
// nest made the compiler copy them every filter step).
template <int K, bool R, bool LB>
__device__ __forceinline__ void pair_scan_f32(FilterRun<0> r, int* __restrict__ queue, int lane, const PairLaneF& L,
                                              const float4* __restrict__ xr, const FilterRows& f,
                                              const float* __restrict__ xif, const float* __restrict__ sig,
                                              const PairConstF& pc, PairAccM& A, const PairRep& rp, RepAcc& B) {
  static_assert(kBatchF == 4, "one 16-byte load per coordinate and batch");
  int* const qlane = queue + lane;
  int cnt = A.cnt;
  while (__any(r.more())) {
    float4 X = any4(), Y = any4(), Z = any4();
    if (r.more()) r.load(f, X, Y, Z);
    cnt = r.test(X, Y, Z, pc.a2f, qlane, cnt);
    if (__builtin_expect(__any(cnt > kQueueF - kBatchF), 0)) {
      A.cnt = cnt;
      pair_drain_f32<K, R, LB>(queue, kDrainF, lane, L, xr, xif, sig, pc, A, rp, B);
      cnt = A.cnt;
    }
  }
  A.cnt = cnt;
}

// Set-up of a block's targets: lane's target, its cell and its scan data.
struct TargetF {
  int lane, sc, cx, cy, cz;
  bool active;
  float4 xi;
  PairLaneF L;
};

template <bool LB>
__device__ __forceinline__ TargetF pair_target_f32(const PairArgsF& ar, int blk, const float4* shift) {
  TargetF t;
  const CellGeom& g = ar.g;
  t.lane = threadIdx.x & (kWaveQ - 1);
  const int k = blk * kWaveQ + t.lane;
  t.active = k < ar.n;
  t.sc = t.active ? k : ar.n - 1;
  t.xi = ar.xr[t.sc];
  const int c = ar.cell_s[t.sc];
  t.cx = c % g.nc[0];
  t.cy = (c / g.nc[0]) % g.nc[1];
  t.cz = c / (g.nc[0] * g.nc[1]);
  t.L = PairLaneF{t.xi.x, t.xi.y, t.xi.z, (float)t.cx,
                  t.active ? (t.sc | entry_bits(0, 0, 0)) : -1, t.sc | entry_bits(0, 0, 0), shift,
                  LB ? ar.sig[t.sc] : 0.0f, ar.xf[t.sc]};
  return t;
}

// One wave's scan of all rows of its targets, into A and B.
template <int K, bool R, bool LB>
__device__ __forceinline__ void pair_rows_f32(const PairArgsF& ar, const TargetF& t, int* queue, PairAccM& A, RepAcc& B) {
  const PairConstF& pc = ar.pc;
  const FilterRows f(ar.xf, ar.xf_stride);
  const RowTrim w(ar.cstart, ar.g, pc.w, pc.a2);
  walk_rows(w, RowSpan<1>(), t.cx, t.cy, t.cz, t.xi.x, t.xi.y, t.xi.z, t.active,
            [&](const RowRuns& r, int dz, int dy, int, int) {
    // the second run (across the periodic edge) is empty for most waves: its
    // set-up is skipped unless some lane has one
    auto scan = [&](int j0, int j1, int ix) {
      if (!__any(j0 < j1)) return;
      const FilterRun<0> run(j0, j1, fmaf((float)-ix, pc.L[0], t.L.xa), fmaf((float)-dy, pc.w[1], t.L.yy),
                             fmaf((float)-dz, pc.w[2], t.L.zz), entry_bits(ix, dy, dz));
      pair_scan_f32<K, R, LB>(run, queue, t.lane, t.L, ar.xr, f, ar.xif, ar.sig, pc, A, ar.rep, B);
    };
    scan(r.j0, r.j1, r.ix1);
    scan(r.k0, r.k1, r.ix2);
  });
  pair_drain_f32<K, R, LB>(queue, kQueueF, t.lane, t.L, ar.xr, ar.xif, ar.sig, pc, A, ar.rep, B);
}

template <int K, bool R = false, bool LB = false>
struct PairTrimF32 {
  using Args = PairArgsF;
  static constexpr int kThreads = kWaveQ;
  static __device__ void run(const Args& ar, int blk) {
    __shared__ int queue[kQueueF * kWaveQ];
    __shared__ float4 shift[kShifts];
    const TargetF t = pair_target_f32<LB>(ar, blk, shift);
    fill_shifts(shift, t.lane, ar.g, ar.pc);
    PairAccM A{{0.0, 0.0, 0.0, 0.0}, 0};
    RepAcc B{{0.0, 0.0, 0.0, 0.0}};
    pair_rows_f32<K, R, LB>(ar, t, queue, A, B);
    if (t.active) {
      const double wi = (double)ar.xif[t.sc];
      ar.e0[t.sc] = A.a[0];
      ar.floc[3 * (size_t)t.sc + 0] = wi * A.a[1];
      ar.floc[3 * (size_t)t.sc + 1] = wi * A.a[2];
      ar.floc[3 * (size_t)t.sc + 2] = wi * A.a[3];
    }
    if constexpr (R) store_rep(ar.rep, t.active, t.sc, t.lane, blk, B);
  }
};

// The FP32 scan dealt to the eight waves of a block (pair_split), with the
// sums of PairTrimF32 to the last FP32 bit: there the terms that meet in one
// drain are summed in FP32, and which terms meet depends on all 64 lanes'
// queues.  So the waves first only filter: each scans its share of the rows
// and leaves, per step of four candidates and lane, the mask of its hits and
// the step's place (run, step of the run).  Then each lane's hits are listed in
// order, every wave replays the queue lengths over all steps (counts only)
// and evaluates every eighth drain, and the drains' sums are added in FP64.
// LDS: 80,336 bytes, two blocks per CU.  Rows that leave more steps or hits
// than fit (all 25 of a target with more than about 280 neighbours) are done in
// several passes, half as many rows in each, the queues' last entries carried
// from one to the next.  A pass of one row takes as many of its steps as the
// lists hold whatever hits, the waves sharing them.  Evaluations of 32,000
// atoms at density 0.8 with a = 4 / 5 / 6 in passes 210 / 545 / 732 us, with
// such blocks left to one wave 313 / 627 / 999.
constexpr int kSplitF = 8;           // waves per block
// Filter steps of one wave: as many as the LDS of two blocks leaves.  With 40
// every lattice (near-equal atoms per cell row) had blocks that did not fit: 4000
// atoms on a jittered one 189 us an evaluation, now 124.
constexpr int kSplitSteps = 48;
constexpr int kSplitHits = 288;      // hits of one target
constexpr int kSplitShare = kSplitHits / kBatchF / kSplitF;   // a wave's steps in a pass of one row
constexpr int kSplitRuns = 50;       // 25 rows, two runs each
constexpr int kSplitCarry = kQueueF - kBatchF;   // entries a queue holds between two steps

template <int K, bool R = false, bool LB = false>
struct PairSplitF32 {
  using Args = PairArgsF;
  static constexpr int kThreads = kWaveQ * kSplitF;
  static constexpr int kWavesPerSimd = 4;   // two blocks per CU, as the LDS allows
  static __device__ void run(const Args& ar, int blk) {
    constexpr int NS = kSplitF, W = kWaveQ;
    __shared__ unsigned char mask[NS * kSplitSteps * W];
    __shared__ unsigned short place[NS * kSplitSteps];
    __shared__ int first[kSplitRuns * W];       // queue entry of a run's first source
    // hit lists (step << 2 | candidate); later the waves' sums
    __shared__ __attribute__((aligned(16))) unsigned short list[kSplitHits * W];
    __shared__ int carry[kSplitCarry * W];      // queue entries left by the passes before
    __shared__ unsigned short hits[NS * W];
    __shared__ int steps[NS];                   // filter steps of each wave, -1: too many
    __shared__ float4 shift[kShifts];
    static_assert(sizeof(mask) + sizeof(place) + sizeof(first) + sizeof(list) + sizeof(carry) + sizeof(hits) +
                      sizeof(steps) + sizeof(shift) <= 80 * 1024, "two blocks per CU");
    const TargetF t = pair_target_f32<LB>(ar, blk, shift);
    const int lane = t.lane;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / W);
    if (wv == 0) fill_shifts(shift, lane, ar.g, ar.pc);   // read after the barrier below
    const PairConstF& pc = ar.pc;
    const PairRep& rp = ar.rep;
    const CellGeom& g = ar.g;
    const RowTrim trim(ar.cstart, g, pc.w, pc.a2);
    const FilterRows f(ar.xf, ar.xf_stride);
    double sum[R ? 8 : 4] = {};
    int cnt = 0, drain = 0;   // the lane's queue length, drains so far
    // the pass: from step `seg` of the first of `rows` rows (seg > 0: a part of one)
    int row = 0, rows = 25, seg = 0;
    // One pass; true when all rows are done.  ALL: the first one, of every row,
    // without what only the others need (4000 atoms: 37.3 us; one form for all
    // passes cost 2.6 us).
    auto pass = [&](auto all) -> bool {
      constexpr bool ALL = decltype(all)::value;
      if (ALL) rows = 25;
      else rows = min(rows, 25 - row);
      const bool single = !ALL && rows == 1;
      int row_steps = 0;   // single: steps of the row
      // ---- filter: this wave's share of the pass's rows
      {
        const int r0 = single ? row : row + rows * wv / NS;
        const int r1 = single ? row + 1 : row + rows * (wv + 1) / NS;
        int ns = 0, nh = 0;
        // the cell ranges of all rows first, their loads in flight together
        constexpr int kRows = (25 + NS - 1) / NS;
        RowRuns rr[kRows];
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
          const int r = r0 + u;
          const int dz = r / 5 - 2, dy = r % 5 - 2;
          int tz = t.cz + dz, ty = t.cy + dy;
          tz = tz < 0 ? tz + g.nc[2] : (tz >= g.nc[2] ? tz - g.nc[2] : tz);
          ty = ty < 0 ? ty + g.nc[1] : (ty >= g.nc[1] ? ty - g.nc[1] : ty);
          const float gz = trim.gap(2, dz, t.xi.z), gy = trim.gap(1, dy, t.xi.y);
          const float rem = r < r1 ? (trim.a2m - gz * gz) - gy * gy : 0.0f;
          rr[u] = trim.runs(t.cx, t.xi.x, t.active, rem, (tz * g.nc[1] + ty) * g.nc[0]);
        }
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
          const int r = r0 + u;
          const int dz = r / 5 - 2, dy = r % 5 - 2;
          const float ay = fmaf((float)-dy, pc.w[1], t.L.yy);
          const float az = fmaf((float)-dz, pc.w[2], t.L.zz);
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            int j = h ? rr[u].k0 : rr[u].j0;
            const int j1 = h ? rr[u].k1 : rr[u].j1, ix = h ? rr[u].ix2 : rr[u].ix1;
            if (!__any(j < j1)) continue;
            int k = 0, kend = 1 << 30;   // the wave's steps of the run
            if (single) {
              int len = j1 - j + kBatchF - 1;
#pragma unroll
              for (int off = 32; off > 0; off >>= 1) len = max(len, __shfl_xor(len, off));
              // counted from the pass's first step of the run
              const int from = max(0, seg - row_steps);
              j += from * kBatchF;
              k = max(0, seg + wv * kSplitShare - row_steps - from);
              kend = seg + (wv + 1) * kSplitShare - row_steps - from;
              row_steps += len / kBatchF;
            }
            const float ax = fmaf((float)-ix, pc.L[0], t.L.xa);
            first[(2 * r + h) * W + lane] = j | entry_bits(ix, dy, dz);
            // the next step's candidates are loaded before this step's are used
            float4 X = make_float4(0.0f, 0.0f, 0.0f, 0.0f), Y = X, Z = X, Xn = X, Yn = X, Zn = X;
            auto load = [&](int i) {
              if (i < j1) {
                const unsigned off = (unsigned)i * 4u;
                Xn = load4f(reinterpret_cast<const float*>(reinterpret_cast<const char*>(f.x) + (unsigned)off));
                Yn = load4f(reinterpret_cast<const float*>(reinterpret_cast<const char*>(f.y) + (unsigned)off));
                Zn = load4f(reinterpret_cast<const float*>(reinterpret_cast<const char*>(f.z) + (unsigned)off));
              }
            };
            j += k * kBatchF;
            load(j);
            for (; ns >= 0 && (!single || k < kend) && __any(j < j1); ++k) {
              if (ns == kSplitSteps) {
                ns = -1;
                break;
              }
              const int rem = j1 - j;
              X = Xn;
              Y = Yn;
              Z = Zn;
              load(j + kBatchF);
              const float xb[4] = {X.x, X.y, X.z, X.w}, yb[4] = {Y.x, Y.y, Y.z, Y.w}, zb[4] = {Z.x, Z.y, Z.z, Z.w};
              int m = 0;
#pragma unroll
              for (int b = 0; b < kBatchF; ++b) {
                const float dxv = ax - xb[b], dyv = ay - yb[b], dzv = az - zb[b];
                const float r2 = fmaf(dzv, dzv, fmaf(dxv, dxv, dyv * dyv));
                m |= ((b < rem) & (r2 < pc.a2f)) ? 1 << b : 0;
              }
              mask[(wv * kSplitSteps + ns) * W + lane] = (unsigned char)m;
              if (lane == 0) place[wv * kSplitSteps + ns] = (unsigned short)((2 * r + h) | (k << 6));
              nh += __builtin_popcount(m);
              ++ns;
              j += kBatchF;
            }
          }
        }
        hits[wv * W + lane] = (unsigned short)nh;
        if (lane == 0) steps[wv] = ns;
      }
      __syncthreads();
      int base = 0, total = 0, few = 0;
#pragma unroll
      for (int w = 0; w < NS; ++w) {
        const int h = hits[w * W + lane];
        base += w < wv ? h : 0;
        total += h;
        few = min(few, steps[w]);
      }
      if (few < 0 || __any(total > kSplitHits)) {   // the same in every wave
        rows = (rows + 1) / 2;   // never one row: kSplitShare steps, kSplitHits hits
        __syncthreads();   // hits and steps have been read
        return false;
      }
      // ---- the hits in order
      for (int st = wv * kSplitSteps, n = st + steps[wv]; st < n; ++st) {
        const int m = mask[st * W + lane];
#pragma unroll
        for (int b = 0; b < kBatchF; ++b)
          if (m >> b & 1) list[base++ * W + lane] = (unsigned short)(st << 2 | b);
      }
      __syncthreads();
      // ---- the drains; a lane's entries are its carried ones, then its list
      const int old = cnt;
      int pos = 0;
      auto entry = [&](int i) {
        if (!ALL && i < old) return carry[i * W + lane];
        const int e = list[(i - old) * W + lane];
        const int pl = place[e >> 2];
        return first[(pl & 63) * W + lane] + ((pl >> 6) << 2) + (e & 3);
      };
      auto evaluate = [&](int m) {
        DrainF<R> D;
        // four sources at a time, their look-ups and loads in flight together
        constexpr int kAhead = 4;
        for (int u0 = 0; __any(u0 < m); u0 += kAhead) {
          bool ok[kAhead];
          int ent[kAhead];
          float4 xj[kAhead];
          float wsrc[kAhead];
#pragma unroll
          for (int u = 0; u < kAhead; ++u) {
            const int q = u0 + u < m ? entry(pos + u0 + u) : t.L.self_ent;
            // idle slots (and the target itself): as in pair_drain_f32
            ok[u] = q != t.L.self_ent;
            ent[u] = ok[u] ? q : t.L.safe_ent;
            xj[u] = at24(ar.xr, ent[u]);
            wsrc[u] = at24(ar.xif, ent[u]);
          }
#pragma unroll
          for (int u = 0; u < kAhead; ++u)
            pair_term_f32<K, R, LB>(ok[u], ent[u], xj[u], ok[u] ? wsrc[u] : 0.0f, t.L, ar.sig, pc, rp, D);
        }
#pragma unroll
        for (int c = 0; c < (R ? 8 : 4); ++c) sum[c] += (double)D.s[c];
      };
      for (int w = 0; w < NS; ++w) {
        int st = w * kSplitSteps;
        const int n = st + steps[w];
        int next = mask[st * W + lane];
        for (; st < n; ++st) {
          cnt += __builtin_popcount(next);
          next = mask[min(st + 1, NS * kSplitSteps - 1) * W + lane];
          if (__any(cnt > kQueueF - kBatchF)) {
            const int m = min(cnt, kDrainF);
            if ((drain++ & (NS - 1)) == wv) evaluate(m);
            pos += m;
            cnt -= m;
          }
        }
      }
      if (single && seg + NS * kSplitShare < row_steps) {
        seg += NS * kSplitShare;
      } else {
        row += rows;
        seg = 0;
      }
      if (!ALL && row < 25) {
        // what the queues still hold (at most kSplitCarry entries) for the next pass
        int v[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) v[u] = wv + u * NS < cnt ? entry(pos + wv + u * NS) : 0;
        static_assert(kSplitCarry <= 2 * NS, "two entries per wave");
        __syncthreads();   // carry, and the lists and masks behind it, have been read
#pragma unroll
        for (int u = 0; u < 2; ++u)
          if (wv + u * NS < cnt) carry[(wv + u * NS) * W + lane] = v[u];
        return false;
      }
      if ((drain & (NS - 1)) == wv) evaluate(cnt);
      return true;
    };
    bool done = pass(std::true_type{});
    while (!done) done = pass(std::false_type{});
    __syncthreads();
    // ---- the waves' sums, in wave order
    double* const out = reinterpret_cast<double*>(list);
    static_assert(sizeof(list) >= sizeof(double) * 8 * NS * W, "the sums reuse the hit lists");
#pragma unroll
    for (int c = 0; c < (R ? 8 : 4); ++c) out[(wv * 8 + c) * W + lane] = sum[c];
    __syncthreads();
    if (wv < (R ? 8 : 4)) {
      double v = 0.0;
#pragma unroll
      for (int w = 0; w < NS; ++w) v += out[(w * 8 + wv) * W + lane];
      if (wv >= 4) {
        const double ci = t.active ? rp.x12[t.sc] : 0.0;
        if (wv == 4) {
          const double e = wave_sum(t.active ? ci * v : 0.0);
          if (lane == 0) rp.partial[blk] = e;
        } else if (t.active) {
          rp.frep[3 * (size_t)t.sc + wv - 5] = ci * v;
        }
      } else if (t.active) {
        if (wv == 0) ar.e0[t.sc] = v;
        else ar.floc[3 * (size_t)t.sc + wv - 1] = (double)ar.xif[t.sc] * v;
      }
    }
  }
};

}  // namespace

// Threshold of the FP32 candidate filters: the filter's |dx| is within ex of
// the exact value (absolute coordinates and the image shift rounded to FP32,
// at most a few ulp of L + a; neighbour reuse lets atoms sit skin/2 outside
// the box), so r^2 < a^2 + 2 a ex + ex^2, plus FP32 rounding of the sum,
// keeps every pair inside the cutoff.
float filter_a2(const mls_plan_s* P) {
  const double a = std::sqrt(P->a2);
  const double ex = 4.0 * (P->cg.L[0] + P->cg.margin + a) * std::ldexp(1.0, -24);
  return std::nextafter((float)(P->a2 * (1.0 + 4.0 * std::ldexp(1.0, -23)) + 2.0 * a * ex + ex * ex), INFINITY);
}

PairConst pair_const(const mls_plan_s* P) {
  PairConst pc{P->a2, P->inv_a2, P->inv_a6, P->inv_a8, {}, {}, filter_a2(P), {}, {},
               {-15.0 / 8.0 * P->inv_a6, 5.0 / 4.0 * P->inv_a6, -3.0 / 8.0 * P->inv_a6, -9.0 * P->inv_a8,
                15.0 * P->inv_a8}};
  for (int j = 0; j < 5; ++j) pc.gc[j] = P->gamma_c[j];
  for (int j = 0; j < 4; ++j) pc.gq[j] = 12.0 * (j + 1) * P->gamma_c[j + 1];
  for (int d = 0; d < 3; ++d) {
    pc.wf[d] = (float)P->cg.w[d];
    pc.Lf[d] = (float)P->cg.L[d];
  }
  return pc;
}

PairConstF pair_const_f(const mls_plan_s* P) {
  const PairConst pc = pair_const(P);
  PairConstF pf{(float)pc.a2, (float)pc.inv_a2, (float)pc.inv_a6, (float)pc.inv_a8,
                {(float)P->cg.w[0], (float)P->cg.w[1], (float)P->cg.w[2]}, {}, {}};
  for (int j = 0; j < 5; ++j) pf.gc[j] = (float)pc.gc[j];
  for (int j = 0; j < 4; ++j) pf.gq[j] = (float)pc.gq[j];
  for (int d = 0; d < 3; ++d) pf.L[d] = (float)P->cg.L[d];
  pf.a2f = pc.a2f;
  return pf;
}

int pair_variant(const mls_plan_s* P) { return P->continuity == 2 ? 2 : 0; }

// Waves per 64 targets.  One wave walks its 25 rows in about 95 us whatever
// the number of atoms (dependent cell-range and candidate loads), so a launch
// of fewer waves than the chip holds (20 per CU in FP64, 28 in FP32) is bound
// by that chain; dealing the rows to more waves shortens it.  Pair kernel
// alone with 1 / 2 / 4 / 8 waves (us, FP64; cube at density 0.8, a = 3):
// 1000 atoms 95 / 60 / 36 / 24, 32,000 atoms 99 / 63 / 41 / 31, 10^5 atoms
// 113 / 80 / 82 / 86, 250,000 atoms 161 / 155 / 161 / 176, 10^6 atoms 461 /
// 473 / 538 / 606 (the filter steps of a row are set by its slowest lane
// either way; what grows is the set-up): hence at most kPairSlots waves.
// Beside the grid chain two waves at most: the chain's kernels then find free
// slots (evaluation of 64,000 atoms, FP64: 155 / 128 / 135 / 135 us).
int pair_split(int64_t groups, bool alone) {
  for (int ns = alone ? 8 : 2; ns > 1; ns /= 2)
    if (groups * ns <= kPairSlots) return ns;
  return 1;
}

// Beside the grid chain the FP32 kernel holds only so many waves of a CU and
// walks its groups with them: a grid of all groups takes every slot that falls
// free, and the anterpolation submitted before it, whose blocks want 22 KB of
// LDS each, got through only as the pair kernel ended (59 us alone, 420 us
// beside it), with the rest of the chain after that.  Evaluation, all slots /
// 20 waves (us): 310,000 atoms 289 / 288, 500,000 390 / 363, 800,000 557 / 508,
// 10^6 660 / 619, 2,000,000 1194 / 1199; 16 waves 312 / 369 / 558 / 654 / 1274.
// The seven chains of Lorentz-Berthelot mixing want more room, all / 14 waves:
// 310,000 574 / 545, 500,000 716 / 659, 800,000 1087 / 972, 1,200,000 2039 /
// 1920; 20 waves 579 / 682 / 1046 / 2017.  The FP64 kernel leaves no slots worth
// having at 20 waves, and fewer cost it what they give the chain (10^6 atoms,
// all / 18 / 16: 734 / 734 / 762).  With the repulsion (R) a CU holds 20 anyway.
// In a captured graph, whose replay starts both branches together, the one
// chain's anterpolation comes first and the whole grid is better (10^6 atoms
// mixed, all / 20 waves: 604 / 627 us a replay; 633 / 597 a call); the seven
// chains still want the room (all / 14: 1406 / 1378 us a replay of a jittered
// lattice, 1388 / 1324 on another card).
constexpr int kBesideWaves = 20, kBesideSeven = 14;

bool capturing(hipStream_t s) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &st) == hipSuccess) return st == hipStreamCaptureStatusActive;
  (void)hipGetLastError();   // not an error of the launch that follows
  return false;
}

template <int K, bool R, bool LB>
hipError_t launch_split_f32(const mls_plan_s* P, const PairArgsF& a, int groups, bool alone, hipStream_t s) {
  int blocks = P->pair_blocks;
  if (blocks <= 0) {
    // (so few beside a chain: one with the tap stencil, whose waves the eight
    // would displace: 30,000 atoms at a = 4, h = 0.5 19.1 ms in one, 24.9 in eight)
    if (alone && groups <= kSplitGroupsF) return launch_one<PairSplitF32<K, R, LB>>(a, groups, s);
    if (!alone && !R && (LB || !capturing(s))) blocks = P->cus * (LB ? kBesideSeven : kBesideWaves);
  }
  return launch_persist<PairTrimF32<K, R, LB>>(a, groups, blocks, s);
}

template <int K, bool LB, bool R>
hipError_t launch_split_f64(const mls_plan_s* P, const PairArgs& a, int groups, bool alone, hipStream_t s) {
  switch (P->pair_blocks > 0 ? 1 : pair_split(groups, alone)) {
    case 8: return launch_one<PairTrimF64<K, LB, R, 8>>(a, groups, s);
    case 4: return launch_one<PairTrimF64<K, LB, R, 4>>(a, groups, s);
    case 2: return launch_one<PairTrimF64<K, LB, R, 2>>(a, groups, s);
    default: return launch_persist<PairTrimF64<K, LB, R>>(a, groups, P->pair_blocks, s);
  }
}

template <int K>
hipError_t launch_pair_k(mls_plan_s* P, int n, hipStream_t s, const PairRep* rep, bool* fused, bool alone) {
  const CellGeom& g = P->cg;
  const int waves = (n + kWaveQ - 1) / kWaveQ;
  if (P->precision == MLS_MIXED && P->pair_fast && n < (1 << 24)) {
    PairArgsF a{P->d_xr, P->d_xif, P->d_xs, P->d_cell_s, P->d_cell_start, n, g, pair_const_f(P), P->d_e0,
                P->d_floc};
    a.xf = P->d_xf;
    a.xf_stride = P->xf_stride;
    if (!rep) return launch_split_f32<K, false, false>(P, a, waves, alone, s);
    a.rep = *rep;
    *fused = true;
    P->rep_nb = waves;
    return launch_split_f32<K, true, false>(P, a, waves, alone, s);
  }
  PairArgs a{P->d_xs, P->d_cell_s, P->d_cell_start, n, g, pair_const(P), P->d_e0, P->d_floc, nullptr};
  a.xf = P->d_xf;
  a.xf_stride = P->xf_stride;
  if (P->pair_fast && n < (1 << 25)) {
    if (!rep) return launch_split_f64<K, false, false>(P, a, waves, alone, s);
    a.rep = *rep;
    *fused = true;
    P->rep_nb = waves;
    return launch_split_f64<K, false, true>(P, a, waves, alone, s);
  }
  if (!P->pair_fast) return launch_one<PairWave<K>>(a, n, s);
  return launch_one<PairGeneric<K>>(a, (n + kBlock - 1) / kBlock, s);
}

// Lorentz-Berthelot: the same kernels with the LB source weight.
template <int K>
hipError_t launch_pair_lb_k(mls_plan_s* P, int n, hipStream_t s, bool alone) {
  if (P->precision == MLS_MIXED && P->pair_fast && n < (1 << 24)) {
    PairArgsF a{P->d_xr, P->d_xif, P->d_xs, P->d_cell_s, P->d_cell_start, n, P->cg, pair_const_f(P), P->d_e0,
                P->d_floc};
    a.sig = P->d_sigf;
    a.xf = P->d_xf;
    a.xf_stride = P->xf_stride;
    return launch_split_f32<K, false, true>(P, a, (n + kWaveQ - 1) / kWaveQ, alone, s);
  }
  PairArgs a{P->d_xs, P->d_cell_s, P->d_cell_start, n, P->cg, pair_const(P), P->d_e0, P->d_floc, P->d_sig};
  a.xf = P->d_xf;
  a.xf_stride = P->xf_stride;
  if (P->pair_fast && n < (1 << 25)) return launch_split_f64<K, true, false>(P, a, (n + kWaveQ - 1) / kWaveQ, alone, s);
  if (!P->pair_fast) return launch_one<PairWave<K, true>>(a, n, s);
  return launch_one<PairGeneric<K, true>>(a, (n + kBlock - 1) / kBlock, s);
}

hipError_t launch_pair_lb(mls_plan_s* P, int n, hipStream_t s, bool alone) {
  if (n == 0) return hipSuccess;
  return pair_variant(P) == 2 ? launch_pair_lb_k<2>(P, n, s, alone) : launch_pair_lb_k<0>(P, n, s, alone);
}

hipError_t launch_pair(mls_plan_s* P, int n, hipStream_t s, const PairRep* rep, bool* fused, bool alone) {
  bool f = false;
  if (!fused) fused = &f;
  *fused = false;
  if (n == 0) return hipSuccess;
  return pair_variant(P) == 2 ? launch_pair_k<2>(P, n, s, rep, fused, alone)
                              : launch_pair_k<0>(P, n, s, rep, fused, alone);
}

template <int K, int NS>
hipError_t launch_batched_trim(const BatchPhase& ph, hipStream_t s, bool lb) {
  if (ph.kernel == BK_PAIR_TRIM_F64)
    return lb ? launch_batched_phase<PairTrimF64<K, true, false, NS>>(ph, s)
              : launch_batched_phase<PairTrimF64<K, false, false, NS>>(ph, s);
  if constexpr (NS == kSplitF)
    return lb ? launch_batched_phase<PairSplitF32<K, false, true>>(ph, s)
              : launch_batched_phase<PairSplitF32<K>>(ph, s);
  return lb ? launch_batched_phase<PairTrimF32<K, false, true>>(ph, s) : launch_batched_phase<PairTrimF32<K>>(ph, s);
}

template <int K>
hipError_t launch_batched_pair_k(const BatchPhase& ph, hipStream_t s, bool lb) {
  switch (ph.kernel) {
    case BK_PAIR_GENERIC:
      return lb ? launch_batched_phase<PairGeneric<K, true>>(ph, s) : launch_batched_phase<PairGeneric<K>>(ph, s);
    case BK_PAIR_WAVE:
      return lb ? launch_batched_phase<PairWave<K, true>>(ph, s) : launch_batched_phase<PairWave<K>>(ph, s);
    case BK_PAIR_TRIM_F64:
    case BK_PAIR_TRIM_F32:
      switch (ph.variant >> 8) {
        case 8: return launch_batched_trim<K, 8>(ph, s, lb);
        case 4: return launch_batched_trim<K, 4>(ph, s, lb);
        case 2: return launch_batched_trim<K, 2>(ph, s, lb);
        default: return launch_batched_trim<K, 1>(ph, s, lb);
      }
    default: return hipErrorInvalidValue;
  }
}

// Batched phases of this file; variant = the pair_variant of its boxes, | 0x10
// under Lorentz-Berthelot mixing, | waves per block << 8 of the trimmed kernels.
hipError_t launch_batched_pair(const BatchPhase& ph, hipStream_t s) {
  const bool lb = (ph.variant & 0x10) != 0;
  return (ph.variant & 0xf) == 2 ? launch_batched_pair_k<2>(ph, s, lb) : launch_batched_pair_k<0>(ph, s, lb);
}

}  // namespace mls
