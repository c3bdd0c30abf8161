// Device side of the batched r-cell MD library (gfx950).
//
// Data layout (one batch = all cells of a context, atoms of cell c at [off_c, off_c + n_c)):
//   x, y, z     FP64 SoA master positions        vx, vy, vz  FP64 SoA velocities
//   fx, fy, fz  FP64 total force of the last completed step (read by the first kick of a run)
//   s[2]        double-buffered fixed-point scaled coordinates: S = frac(H^-1 x) * 2^32 (int32,
//               mixed) or * 2^64 (int64, FP64 mode); .w carries F'(rho) for the EAM force pass (scaled by sc_fscale).
//               Differences of two such integers wrap modulo 2^32 (2^64), which is exactly the
//               per-component minimum image in scaled space: the pair separation needs no
//               image shifts (d = H dS, formed in FP64 and rounded once in mixed precision).
//   sb          s at the last neighbour build, quantised to its top 16 bits per component (8 bytes;
//               the displacement check allows for the quantisation, see qeps)
//   nbr         Verlet list within rc + skin, cell-local j, as 16-bit indices when every cell has
//               at most 65536 atoms (mixed precision), else 32-bit; entries of one atom in blocks
//               of B = 8 (Kremer-Grest) or 16 (Sutton-Chen), the blocks of entries [b B, (b+1) B) of
//               all atoms side by side (list_index), so a lane loads its UNR entries of a trip with
//               one vector load
//   pl, pn      pruned list: the entries of nbr within a little more than rc, rewritten every few steps
//               by a force pass and walked by the passes between (PruneWalk)
//   bond        up to four FENE partners per atom (cell-local positions; the atom's own position marks an
//               empty slot), 16-bit slots when the list entries are 16-bit, else 32-bit
//   gid         original cell-local index of the atom stored at each position; pos_of inverts it;
//               bond0 holds the partners by original index.  At every neighbour build a cell's
//               atoms are reordered by (bin, original index), so that neighbours sit close in
//               memory; everything that identifies an atom (noise counter, host API order) uses gid.
// Work is distributed over 64-atom tiles (a tile never straddles two cells); each tile writes
// one partial record and a per-cell kernel reduces them in a fixed order (deterministic).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace rcell {

constexpr int TILE = 64;
constexpr int BIN_BITS = 10;     // bins per dimension < 2^BIN_BITS (bin coordinates are packed)
constexpr int BIN_MASK = (1 << BIN_BITS) - 1;
constexpr int UNR = 4;           // neighbour-loop unroll: gathers in flight per lane
constexpr int NBLK_MAX = 16;     // list blocks: 2^lblk consecutive entries of one atom, 8 or 16 (the
                                 // capacity is a multiple of 16)
constexpr double TWO32 = 4294967296.0;
constexpr double TWOM32 = 1.0 / 4294967296.0;

enum Mode : int { MODE_PRIME = 0, MODE_STEP = 1, MODE_LAST = 2, MODE_STATIC = 4 };
enum RedMode : int { RED_START = 0, RED_PRIME = 1, RED_STEP = 2, RED_LAST = 3, RED_STATIC = 4, RED_MOVE = 5 };
enum Status : int { ST_OK = 0, ST_BOND = -4, ST_CAP = -8, ST_BOX = -3, ST_BAD_F = -2 };

struct alignas(32) S64 { long long x, y, z, w; };

// Element index of list entry k of atom i (batch position) in a list of npad atoms: blocks of
// B = 2^lb consecutive entries of one atom, the blocks of all atoms for entries [b B, (b+1) B) stored
// together in atom order.  The list holds < 2^32 elements, so 32-bit arithmetic is exact.  Short
// Kremer-Grest lists (~20 entries) take B = 8, so that an atom's last block wastes fewer fetched
// bytes; Sutton-Chen lists take B = 16, so that the 16 entries its lane group reads per trip are one
// contiguous piece.
__host__ __device__ inline unsigned list_index(unsigned k, unsigned npad, unsigned i, int lb) {
  return (((k >> lb) * npad + i) << lb) | (k & ((1u << lb) - 1u));
}

struct CellDev {
  double H[9], Hi[9];             // box (upper triangular) and its inverse
  double Rprev[9], Q[9], R[9], F[9];
  double J, V;
  double xi_mean[3];              // per-cell mean of the integer noise for the next time level
  double wsum[6], last[6];        // stress window sum and last sample (Voigt, tension +)
  double pe;
  double Hd[6];                   // H * 2^-64, upper triangle (FP64 mode)
  double Hm[6];                   // H * 2^-32, upper triangle (mixed mode)
  long long wcount, step, nrebuild;
  int off, n, tile_off, ntile;
  int nb[3], bin_off, bin_cap;
  int rebuild, pending, status;
  int span;                       // list build: bins that a wave takes together, at most
  float span_rate;                // and as many of them per tile that is built
  double Hb[6];                   // H at the last neighbour build, upper triangle (0 1 2 4 5 8)
  float hs2;                      // squared (measured) displacement that still keeps the list complete
  float dmax2;                    // largest squared measured displacement since the last build, as last reduced
  float qeps;                     // bound on the error of a measured displacement: the 16-bit build reference
  float list_lo2, list_hi2;       // list build: |d|^2 from FP32 offsets surely below / above (rc + skin)^2
  float pmove;                    // bound on how far any atom has moved since the pruned list was written
  int prune;                      // the next force pass walks the full list and writes the pruned one
  // molecular statics (FIRE): time step, mixing parameter, the velocity update of this iteration
  // (v = fa v + fb f, or zero when frozen), iterations since the power last turned negative,
  // converged flag and iterations used
  double fdt, falpha, fa, fb;
  int fcount, fdone, ffreeze, fiter;
};

struct Tile { int cell, begin, count, pad; };

// Tile-grid kernels: the grid has ntiles blocks rounded up to a multiple of 8; block w works on
// tile w (w < ntiles).  The pair kernels use block_tile_xcd instead: the GPU hands consecutive
// blocks to its 8 XCDs in turn, so XCD x receives blocks x, x + 8, ..., and this mapping gives it
// the contiguous tile range [x per, (x + 1) per) - whole cells whose positions then stay in that
// XCD's own L2 for the neighbour gathers.
__host__ __device__ inline int tile_grid(int ntiles) { return (ntiles + 7) / 8 * 8; }
__device__ __forceinline__ int block_tile(int ntiles, int block) { return block; }
__device__ __forceinline__ int block_tile_xcd(int ntiles, int block) {
  return (block % 8) * ((ntiles + 7) / 8) + block / 8;
}
// The same placement for block-strided loops over n work items (the rebuild phases): with a grid
// that is a multiple of 8, XCD x runs blocks x, x + 8, ..., and they share out the contiguous item
// range [x per, (x + 1) per), per = ceil(n / 8), so the cells that XCD rebuilds stay in its own L2.
// A block may split its share further over sub workers (its waves): worker w of a block takes the
// items k, k + step, ... below end.
struct XcdLoop {
  int k, end, step;
  __device__ XcdLoop(int n, int sub = 1, int w = 0) {
    const int per = (n + 7) / 8, x = (int)(blockIdx.x & 7u);
    k = x * per + (int)(blockIdx.x >> 3) * sub + w;
    end = min(n, (x + 1) * per);
    step = (int)(gridDim.x >> 3) * sub;
  }
};

struct Part {                     // one tile's contribution
  double V[6];                    // MD: pair virial minus the kinetic term; statics: the FIRE sums
  double pe;
  long long xi[3];
  float maxd2;
  float step2;                    // largest squared displacement of this step
  int status, pad;
};

struct Stage {                    // set_deformation staging, one per cell
  double Q[9], R[9], dR[9], Hn[9], F[9];
  double J, wmin;
  int nb[3], nbins, status;
  int hold, go;                    // the host has to look at this cell first; the whole batch was committed
  double density;
};

struct MDArgs {
  double *x, *y, *z, *vx, *vy, *vz;
  void *fx, *fy, *fz;
  void *s_cur, *s_nxt;
  uint2* sb;
  void* bond;                      // 4 partner slots per atom: uint16_t when bond16, else int
  const int4* bond0;
  int bond16;
  int* gid;
  int* pos_of;
  char* pscr;                      // reorder scratch: 6 doubles, one S and two ints per atom (npad rows)
  int* nn;
  void* nbr;                       // LT entries (uint16_t or int), see the kernels' LT parameter
  long long npad;
  int maxnb;
  int lblk;                        // list blocks of 2^lblk entries (list_index)
  // pruned list (PruneWalk): entries and, per lane of every atom, their number; null: not in use
  void* pl;
  unsigned short* pn;
  double prune_rc2;                // entries within this squared distance are kept
  float prune_move;                // and serve while no atom has moved further than this
  int prune_mode;                  // 0: as the cells' flags say, 1: every pass writes it, 2: no pass does
  CellDev* cells;
  const Tile* tiles;
  Part* parts;
  int ntiles, ncells;
  int* abin; int* bcount; int* bstart; int* bnum; int* bfill; int* binned; int* bkey;
  // work list of the rebuild phases: the cells flagged for a rebuild and the exclusive prefix sums of
  // their tiles; *work_pack = cells << 32 | tiles (work_add, k_rebuild_work)
  int *work_cells, *work_tstart;
  unsigned long long* work_pack;
  int bin_factor;                  // bins at least (rc + skin) / bin_factor wide; stencil +- bin_factor
  // integrator constants (computed once on the host, documented expressions)
  double dt, h, drag, c24, mmv, half_skin2, rcs2;
  double fire_ftol2;               // statics: converged when max_i |f_i|^2 <= fire_ftol2
  int fire_max_iter;               // statics: at most this many moves per cell
  uint32_t key0, key1;
  int gamma_on, include_kinetic, pot;
  // pair constants
  double rc2, lj_eps, lj_sig2, lj_shift, fene_K, fene_R02, sc_eps, sc_a, sc_c, sc_phic, sc_rhoc;
  int sc_n, sc_m;
};

// ------------------------------------------------------------------ Philox4x32-10
// Salmon, Moraes, Dror & Shaw (SC'11): 10 rounds of two 32x32->64 multiplies with the published
// multipliers; the key is bumped by the published Weyl increments between rounds.
__device__ __forceinline__ void philox(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                       uint32_t k0, uint32_t k1, uint32_t out[4]) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint32_t lo0 = 0xD2511F53u * c0, hi0 = __umulhi(0xD2511F53u, c0);
    const uint32_t lo1 = 0xCD9E8D57u * c2, hi1 = __umulhi(0xCD9E8D57u, c2);
    const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
    k0 += 0x9E3779B9u; k1 += 0xBB67AE85u;
  }
  out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// integer noise units k = (w >> 8) - 2^23 for the three components of atom gid of cell at level step
__device__ __forceinline__ void noise_units(const MDArgs& a, int gid, int cell, long long step, int k[3]) {
  uint32_t w[4];
  philox((uint32_t)gid, (uint32_t)cell, (uint32_t)(unsigned long long)step,
         (uint32_t)((unsigned long long)step >> 32), a.key0, a.key1, w);
  k[0] = (int)(w[0] >> 8) - (1 << 23);
  k[1] = (int)(w[1] >> 8) - (1 << 23);
  k[2] = (int)(w[2] >> 8) - (1 << 23);
}

// squared displacement of one drift, rounded up (FP32: three squares and two sums, each within 2^-24)
__device__ __forceinline__ float drift2(double dt, double vx, double vy, double vz) {
  const float ux = (float)(dt * vx), uy = (float)(dt * vy), uz = (float)(dt * vz);
  return 1.000001f * (ux * ux + uy * uy + uz * uz);
}

// ------------------------------------------------------------------ precision policies
struct Mixed {
  using S = int4;
  using R = float;
  using Fst = double;   // stored total force: touched once per run, kept in FP64 so runs split bitwise
  __device__ static S load(const void* p, long long i) { return ((const int4*)p)[i]; }
  // element j of a per-cell base pointer, as a 32-bit unsigned byte offset
  __device__ static S load_rel(const S* base, int j) {
    return *(const S*)((const char*)base + ((unsigned)j << 4));
  }
  __device__ static void store_xyz(void* p, long long i, const S& v) { ((int4*)p)[i] = v; }
  __device__ static void store_w(void* p, long long i, R fp) { ((int4*)p)[i].w = __float_as_int(fp); }
  __device__ static R get_w(const S& v) { return __int_as_float(v.w); }
  // scaled fraction f in [0,1) -> 32-bit fixed point (2^32 wraps to 0)
  __device__ static int fix1(double f) {
    return (int)(unsigned int)(unsigned long long)(long long)rint(f * TWO32);
  }
  __device__ static S make(double f0, double f1, double f2) { return make_int4(fix1(f0), fix1(f1), fix1(f2), 0); }
  // the cell's H * 2^-32 (upper triangular: 0 xx, 1 xy, 2 xz, 3 yy, 4 yz, 5 zz), held in
  // registers across a neighbour loop.  The separation H dS is formed in FP64 (full rate on this
  // GPU, like FP32 without packing) and rounded once to FP32, so no rounding of H acts as a
  // strain of the whole cell.
  struct Geo { double h[6]; };
  __device__ static Geo geo(const CellDev& C) {
    Geo g;
#pragma unroll
    for (int q = 0; q < 6; ++q) g.h[q] = C.Hm[q];
    return g;
  }
  __device__ static void sep(const S& sj, const S& si, const Geo& g, R d[3]) {
    const double a = (double)(int)((unsigned)sj.x - (unsigned)si.x);
    const double b = (double)(int)((unsigned)sj.y - (unsigned)si.y);
    const double c = (double)(int)((unsigned)sj.z - (unsigned)si.z);
    d[0] = (float)fma(g.h[0], a, fma(g.h[1], b, g.h[2] * c));
    d[1] = (float)fma(g.h[3], b, g.h[4] * c);
    d[2] = (float)(g.h[5] * c);
  }
  __device__ static void sep(const S& sj, const S& si, const CellDev& C, R d[3]) { sep(sj, si, geo(C), d); }
  // the same separation, also kept in FP64 before the rounding: the pair virial is accumulated
  // from it in FP64, so neither the rounding of d nor FP32 sums enter the stress
  __device__ static void sep2(const S& sj, const S& si, const Geo& g, R d[3], double dd[3]) {
    const double a = (double)(int)((unsigned)sj.x - (unsigned)si.x);
    const double b = (double)(int)((unsigned)sj.y - (unsigned)si.y);
    const double c = (double)(int)((unsigned)sj.z - (unsigned)si.z);
    dd[0] = fma(g.h[0], a, fma(g.h[1], b, g.h[2] * c));
    dd[1] = fma(g.h[3], b, g.h[4] * c);
    dd[2] = g.h[5] * c;
    d[0] = (float)dd[0]; d[1] = (float)dd[1]; d[2] = (float)dd[2];
  }
  // single hardware instructions (about 1 ulp): ample for FP32 pair forces
  __device__ static R rsq(R x) { return __builtin_amdgcn_rsqf(x); }
  __device__ static R rcp(R x) { return __builtin_amdgcn_rcpf(x); }
  // the build reference: each fixed-point component rounded to its top 16 bits (x | y << 16, z)
  __device__ static uint2 quant(const S& s) {
    const unsigned qx = ((unsigned)s.x + 0x8000u) >> 16, qy = ((unsigned)s.y + 0x8000u) >> 16;
    const unsigned qz = ((unsigned)s.z + 0x8000u) >> 16;
    return make_uint2(qx | (qy << 16), qz);
  }
  // displacement of sn from a quantised reference (minimum image, like sep)
  __device__ static void disp(const S& sn, uint2 q, const Geo& g, R d[3]) {
    const double a = (double)(int)((unsigned)sn.x - ((q.x & 0xffffu) << 16));
    const double b = (double)(int)((unsigned)sn.y - (q.x & 0xffff0000u));
    const double c = (double)(int)((unsigned)sn.z - ((q.y & 0xffffu) << 16));
    d[0] = (float)fma(g.h[0], a, fma(g.h[1], b, g.h[2] * c));
    d[1] = (float)fma(g.h[3], b, g.h[4] * c);
    d[2] = (float)(g.h[5] * c);
  }
};

struct FP64 {
  using S = S64;
  using R = double;
  using Fst = double;
  __device__ static S load(const void* p, long long i) { return ((const S64*)p)[i]; }
  __device__ static S load_rel(const S* base, int j) {
    return *(const S*)((const char*)base + ((unsigned)j << 5));
  }
  __device__ static void store_xyz(void* p, long long i, const S& v) { ((S64*)p)[i] = v; }
  __device__ static void store_w(void* p, long long i, R fp) { ((S64*)p)[i].w = __double_as_longlong(fp); }
  __device__ static R get_w(const S& v) { return __longlong_as_double(v.w); }
  // scaled fraction f in [0,1) -> 64-bit fixed point, rounded to nearest, 2^64 wraps to 0
  __device__ static long long fix1(double f) {
    const double t = f * TWO32;
    const double hi = floor(t);
    const double lo = rint((t - hi) * TWO32);
    const unsigned long long u = ((unsigned long long)(unsigned int)(long long)hi << 32) + (unsigned long long)(long long)lo;
    return (long long)u;
  }
  __device__ static S make(double f0, double f1, double f2) { S s; s.x = fix1(f0); s.y = fix1(f1); s.z = fix1(f2); s.w = 0; return s; }
  __device__ static double cvt(long long v) {       // signed 64-bit integer to double, rounded
    return (double)v;
  }
  struct Geo { double h[6]; };                     // H * 2^-64, upper triangle
  __device__ static Geo geo(const CellDev& C) {
    Geo g;
#pragma unroll
    for (int q = 0; q < 6; ++q) g.h[q] = C.Hd[q];
    return g;
  }
  __device__ static void sep(const S& sj, const S& si, const Geo& g, R d[3]) {
    const double a = cvt((long long)((unsigned long long)sj.x - (unsigned long long)si.x));
    const double b = cvt((long long)((unsigned long long)sj.y - (unsigned long long)si.y));
    const double c = cvt((long long)((unsigned long long)sj.z - (unsigned long long)si.z));
    d[0] = g.h[0] * a + g.h[1] * b + g.h[2] * c;
    d[1] = g.h[3] * b + g.h[4] * c;
    d[2] = g.h[5] * c;
  }
  __device__ static void sep(const S& sj, const S& si, const CellDev& C, R d[3]) { sep(sj, si, geo(C), d); }
  __device__ static void sep2(const S& sj, const S& si, const Geo& g, R d[3], double dd[3]) {
    sep(sj, si, g, d);
    dd[0] = d[0]; dd[1] = d[1]; dd[2] = d[2];
  }
  __device__ static R rsq(R x) { return 1.0 / sqrt(x); }
  __device__ static R rcp(R x) { return 1.0 / x; }
  __device__ static uint2 quant(const S& s) {
    const unsigned long long h = 1ull << 47;
    const unsigned qx = (unsigned)(((unsigned long long)s.x + h) >> 48);
    const unsigned qy = (unsigned)(((unsigned long long)s.y + h) >> 48);
    const unsigned qz = (unsigned)(((unsigned long long)s.z + h) >> 48);
    return make_uint2(qx | (qy << 16), qz);
  }
  __device__ static void disp(const S& sn, uint2 q, const Geo& g, R d[3]) {
    const double a = cvt((long long)((unsigned long long)sn.x - ((unsigned long long)(q.x & 0xffffu) << 48)));
    const double b = cvt((long long)((unsigned long long)sn.y - ((unsigned long long)(q.x >> 16) << 48)));
    const double c = cvt((long long)((unsigned long long)sn.z - ((unsigned long long)(q.y & 0xffffu) << 48)));
    d[0] = g.h[0] * a + g.h[1] * b + g.h[2] * c;
    d[1] = g.h[3] * b + g.h[4] * c;
    d[2] = g.h[5] * c;
  }
};

// S = H^-1 x for upper-triangular H^-1, reduced to its fractional part
// (explicit fused multiply-adds: every caller rounds identically, so the fixed-point coordinates
// that the Kremer-Grest force pass recomputes from x equal the stored ones bit for bit)
template <class Box>
__device__ __forceinline__ void scaled_frac(const Box& C, double x, double y, double z, double f[3]) {
  const double s0 = fma(C.Hi[0], x, fma(C.Hi[1], y, C.Hi[2] * z));
  const double s1 = fma(C.Hi[4], y, C.Hi[5] * z);
  const double s2 = C.Hi[8] * z;
  f[0] = s0 - floor(s0);
  f[1] = s1 - floor(s1);
  f[2] = s2 - floor(s2);
}

template <class P, class Box>
__device__ __forceinline__ typename P::S fixed_pos(const Box& C, double x, double y, double z) {
  double f[3];
  scaled_frac(C, x, y, z, f);
  return P::make(f[0], f[1], f[2]);
}

// t^N for a compile-time exponent (binary powering)
template <int N, class T>
__device__ __forceinline__ T powc(T t) {
  if constexpr (N == 0) return (T)1;
  else if constexpr (N == 1) return t;
  else if constexpr (N % 2 == 0) { const T h = powc<N / 2>(t); return h * h; }
  else return powc<N - 1>(t) * t;
}

// t^n for a run-time exponent 0 <= n < 32, branch free (the exponent is uniform over the grid)
template <class T>
__device__ __forceinline__ T powr(T t, int n) {
  T r = (T)1;
#pragma unroll
  for (int b = 0; b < 5; ++b) {
    r = ((n >> b) & 1) ? r * t : r;
    t *= t;
  }
  return r;
}

// Sutton-Chen powers tn = t^n and tm = t^m; SN = SM = 0 takes the exponents at run time
template <int SN, int SM, class T>
__device__ __forceinline__ void sc_powers(T t, int n, int m, T& tn, T& tm) {
  if constexpr (SN == 9 && SM == 6) {
    const T t3 = t * t * t;
    tm = t3 * t3;
    tn = tm * t3;
  } else if constexpr (SN > 0) {
    tn = powc<SN>(t);
    tm = powc<SM>(t);
  } else {
    tn = powr(t, n);
    tm = powr(t, m);
  }
}

// ------------------------------------------------------------------ block reductions
template <int NT>
__device__ __forceinline__ double block_sum(double v, double* sh) {
  // fixed-shape tree: deterministic for a given block size
  const int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
#pragma unroll
  for (int s = NT / 2; s > 0; s >>= 1) {
    if (t < s) sh[t] += sh[t + s];
    __syncthreads();
  }
  const double r = sh[0];
  __syncthreads();
  return r;
}

// reduce a value across the TPA consecutive lanes that share one atom (result in every lane)
template <int TPA, class T>
__device__ __forceinline__ T lane_sum(T v) {
#pragma unroll
  for (int o = TPA / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, TPA);
  return v;
}

// ------------------------------------------------------------------ per-atom integration tail
// The fields of a cell that a force pass needs, read before its first store: the compiler then loads
// them once through the scalar cache, where loads behind stores went through the vector memory path
// one round trip after another at the end of every wave.
template <class P>
struct CellK {
  double Hi[9], xm[3];
  typename P::Geo g;
  long long step;
  __device__ explicit CellK(const CellDev& C) : g(P::geo(C)), step(C.step) {
#pragma unroll
    for (int q = 0; q < 9; ++q) Hi[q] = C.Hi[q];
#pragma unroll
    for (int q = 0; q < 3; ++q) xm[q] = C.xi_mean[q];
  }
};

// Completes the time level of atom i after its conservative force fc is known:
//   Langevin (drag + noise with the per-cell mean removed), second half kick (v_full), the
//   kinetic stress term, and in MODE_STEP the next first half kick and drift with the new
//   fixed-point position, displacement check and the next level's noise sums.
struct TailIn {                   // the atom's own data, requested ahead of the last gathers of its forces
  double x[3], v[3];
  int gid;
  uint2 sb;
  __device__ void load(const MDArgs& a, long long i, bool step) {
    v[0] = a.vx[i]; v[1] = a.vy[i]; v[2] = a.vz[i];
    gid = a.gid[i];
    if (step) sb = a.sb[i];
  }
};

struct TailOut {
  double K[6];
  float maxd2, step2;
  int xi[3];
};

template <class P>
__device__ __forceinline__ void atom_tail(const MDArgs& a, const CellK<P>& C, int cell, long long i,
                                          double fcx, double fcy, double fcz, int mode, TailOut& o, const TailIn& in) {
  double vx = in.v[0], vy = in.v[1], vz = in.v[2];
  const int gid = in.gid;
  double f0 = fcx, f1 = fcy, f2 = fcz;
  o.step2 = 0.f;
  if (mode == MODE_STATIC) {
    // statics: keep the conservative force and report f.v, |f|^2, |v|^2 and max |f|^2 (FIRE)
    ((typename P::Fst*)a.fx)[i] = (typename P::Fst)f0;
    ((typename P::Fst*)a.fy)[i] = (typename P::Fst)f1;
    ((typename P::Fst*)a.fz)[i] = (typename P::Fst)f2;
    const double ff = f0 * f0 + f1 * f1 + f2 * f2;
    o.K[0] = f0 * vx + f1 * vy + f2 * vz; o.K[1] = ff; o.K[2] = vx * vx + vy * vy + vz * vz;
    o.K[3] = o.K[4] = o.K[5] = 0.0;
    o.maxd2 = (float)ff;
    o.xi[0] = o.xi[1] = o.xi[2] = 0;
    return;
  }
  if (mode == MODE_PRIME) {
    // forces after create / deformation / restore: conservative part only; v is a full-step velocity
    ((typename P::Fst*)a.fx)[i] = (typename P::Fst)f0;
    ((typename P::Fst*)a.fy)[i] = (typename P::Fst)f1;
    ((typename P::Fst*)a.fz)[i] = (typename P::Fst)f2;
  } else {
    if (a.gamma_on) {
      int k[3];
      noise_units(a, gid, cell, C.step + 1, k);
      f0 = (f0 + a.drag * vx) + a.c24 * ((double)k[0] - C.xm[0]);
      f1 = (f1 + a.drag * vy) + a.c24 * ((double)k[1] - C.xm[1]);
      f2 = (f2 + a.drag * vz) + a.c24 * ((double)k[2] - C.xm[2]);
    }
    vx += a.h * f0;  // v(t + dt) from the half-step velocity
    vy += a.h * f1;
    vz += a.h * f2;
  }
  o.K[0] = a.mmv * vx * vx; o.K[1] = a.mmv * vy * vy; o.K[2] = a.mmv * vz * vz;
  o.K[3] = a.mmv * vx * vy; o.K[4] = a.mmv * vx * vz; o.K[5] = a.mmv * vy * vz;
  o.maxd2 = 0.f;
  o.xi[0] = o.xi[1] = o.xi[2] = 0;
  if (mode == MODE_LAST) {
    a.vx[i] = vx; a.vy[i] = vy; a.vz[i] = vz;
    ((typename P::Fst*)a.fx)[i] = (typename P::Fst)f0;
    ((typename P::Fst*)a.fy)[i] = (typename P::Fst)f1;
    ((typename P::Fst*)a.fz)[i] = (typename P::Fst)f2;
  } else if (mode == MODE_STEP) {
    vx += a.h * f0;  // first half kick of the next step
    vy += a.h * f1;
    vz += a.h * f2;
    const double x = in.x[0] + a.dt * vx, y = in.x[1] + a.dt * vy, z = in.x[2] + a.dt * vz;
    a.vx[i] = vx; a.vy[i] = vy; a.vz[i] = vz;
    a.x[i] = x; a.y[i] = y; a.z[i] = z;
    o.step2 = drift2(a.dt, vx, vy, vz);
    const typename P::S sn = fixed_pos<P>(C, x, y, z);
    P::store_xyz(a.s_nxt, i, sn);
    typename P::R d[3];
    P::disp(sn, in.sb, C.g, d);
    o.maxd2 = (float)(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
    if (a.gamma_on) noise_units(a, gid, cell, C.step + 2, o.xi);
  }
}

// sum over the 64 lanes of a wave by xor shuffles (fixed pattern: deterministic)
template <class T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  return v;
}
__device__ __forceinline__ int wave_min(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o));
  return v;
}

// Inclusive prefix sum over the 64 lanes of a wave: row shifts by 1, 2, 4, 8 inside the 16-lane rows, then
// the row totals broadcast onwards (lanes without a source add 0).  Six register-to-register adds,
// where shuffles took six round trips through the LDS crossbar.
__device__ __forceinline__ int wave_inclusive_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1, 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2, 3
  return v;
}

// Sums over a wave by halving: at the first two levels two values share the work, one half of the lanes
// taking over each (a register swap between lane halves, then one addition), the last four levels run
// inside the 16-lane rows (DPP).  Six doubles take 39 register operations, where a tree of shuffles per
// value took 108 and as many trips through the LDS crossbar.  Fixed pattern: deterministic.
// sums2x / sums4x: values a, b (, c, d) of every lane; afterwards the rows of 16 lanes hold, in every
// lane, the sums of a, c, b, d (row 0, 1, 2, 3).
__device__ __forceinline__ void half_swap(int& a, int& b) {
  const auto r = __builtin_amdgcn_permlane32_swap((unsigned)a, (unsigned)b, false, false);
  a = (int)r[0]; b = (int)r[1];
}
__device__ __forceinline__ void row_swap(int& a, int& b) {
  const auto r = __builtin_amdgcn_permlane16_swap((unsigned)a, (unsigned)b, false, false);
  a = (int)r[0]; b = (int)r[1];
}
__device__ __forceinline__ void half_swap(double& a, double& b) {
  int al = __double2loint(a), ah = __double2hiint(a), bl = __double2loint(b), bh = __double2hiint(b);
  half_swap(al, bl); half_swap(ah, bh);
  a = __hiloint2double(ah, al); b = __hiloint2double(bh, bl);
}
__device__ __forceinline__ void row_swap(double& a, double& b) {
  int al = __double2loint(a), ah = __double2hiint(a), bl = __double2loint(b), bh = __double2hiint(b);
  row_swap(al, bl); row_swap(ah, bh);
  a = __hiloint2double(ah, al); b = __hiloint2double(bh, bl);
}
__device__ __forceinline__ void half_swap(float& a, float& b) {
  int x = __float_as_int(a), y = __float_as_int(b);
  half_swap(x, y);
  a = __int_as_float(x); b = __int_as_float(y);
}
__device__ __forceinline__ void row_swap(float& a, float& b) {
  int x = __float_as_int(a), y = __float_as_int(b);
  row_swap(x, y);
  a = __int_as_float(x); b = __int_as_float(y);
}
// rotation of a 16-lane row by N lanes
template <int N>
__device__ __forceinline__ int row_ror(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x120 + N, 0xf, 0xf, false); }
template <int N>
__device__ __forceinline__ double row_ror(double v) {
  return __hiloint2double(row_ror<N>(__double2hiint(v)), row_ror<N>(__double2loint(v)));
}
template <int N>
__device__ __forceinline__ float row_ror(float v) { return __int_as_float(row_ror<N>(__float_as_int(v))); }
template <class T>
__device__ __forceinline__ T row_sum(T v) {
  v += row_ror<8>(v); v += row_ror<4>(v); v += row_ror<2>(v); v += row_ror<1>(v);
  return v;
}
template <class T>
__device__ __forceinline__ T sums4x(T a, T b, T c, T d) {
  half_swap(a, b); half_swap(c, d);
  T u = a + b, w = c + d;          // lower half of the lanes: sums of a and c, upper half: of b and d
  row_swap(u, w);                  // rows 0, 2: u; rows 1, 3: w
  return row_sum(u + w);
}
template <class T>
__device__ __forceinline__ T sums2x(T a, T b) { return sums4x(a, b, (T)0, (T)0); }
// the larger value over the wave of a in the lower half of the lanes, of b in the upper half
__device__ __forceinline__ float maxs2x(float a, float b) {
  half_swap(a, b);
  float u = fmaxf(a, b), w = u;
  row_swap(u, w);
  u = fmaxf(u, w);
  u = fmaxf(u, row_ror<8>(u)); u = fmaxf(u, row_ror<4>(u)); u = fmaxf(u, row_ror<2>(u));
  return fmaxf(u, row_ror<1>(u));
}

template <int NW>
struct PartShared { Part w[NW]; };

// Reduce one tile's contributions (every thread of the block calls this) and write its Part: each wave
// its sums, then, in a block of several waves, the wave results in order.  A wave's noise sum (at most
// 64 integers below 2^23 in magnitude) fits 32 bits.  The energy is reduced only where it is reported
// (with_pe, uniform over the block).
template <int NT>
__device__ __forceinline__ void write_part(Part* parts, int part, const double V[6], double pe, bool with_pe,
                                           const int xi[3], float maxd2, float step2, int status,
                                           PartShared<NT / 64>& sh) {
  constexpr int NW = NT / 64;
  const int wv = threadIdx.x >> 6, ln = threadIdx.x & 63, row = ln >> 4;
  const double v0 = sums4x(V[0], V[1], V[2], V[3]), v1 = sums2x(V[4], V[5]);
  const double e = with_pe ? wave_sum(pe) : 0.0;
  const int x = sums4x(xi[0], xi[1], xi[2], 0);
  const float m = maxs2x(maxd2, step2);
  const int st = __any(status != 0) ? wave_min(status) : 0;
  Part& p = NW == 1 ? parts[part] : sh.w[wv];
  const int q = ((row & 1) << 1) | (row >> 1);     // which of four values this row holds
  if ((ln & 15) == 0) {
    p.V[q] = v0;
    if (q < 3) p.xi[q] = x;
    if ((row & 1) == 0) p.V[4 + (row >> 1)] = v1;
    if (row == 0) { p.pe = e; p.maxd2 = m; p.status = st; }
    if (row == 2) p.step2 = m;
  }
  if constexpr (NW > 1) {
    __syncthreads();
    if (threadIdx.x == 0) {
      Part r = sh.w[0];
      for (int w = 1; w < NW; ++w) {
        const Part& o = sh.w[w];
#pragma unroll
        for (int k = 0; k < 6; ++k) r.V[k] += o.V[k];
        r.pe += o.pe;
#pragma unroll
        for (int k = 0; k < 3; ++k) r.xi[k] += o.xi[k];
        r.maxd2 = fmaxf(r.maxd2, o.maxd2);
        r.step2 = fmaxf(r.step2, o.step2);
        r.status = min(r.status, o.status);
      }
      parts[part] = r;
    }
  }
}

// The per-atom stress contribution of the MD modes, W - K (K only where the kinetic term is
// included), or in statics the FIRE sums carried in K
__device__ __forceinline__ void part_values(const MDArgs& a, int mode, const double W[6], const double K[6], double V[6]) {
  const double kin = a.include_kinetic ? 1.0 : 0.0;
#pragma unroll
  for (int q = 0; q < 6; ++q) V[q] = mode == MODE_STATIC ? K[q] : W[q] - kin * K[q];
}

// Twice the pair virial of one listed pair, g d (x) d / r with gr = g / r, accumulated in FP64 from
// the FP64 separation (halved once after the loop, exact in binary).
__device__ __forceinline__ void add_virial(double w[6], double gr, const double dd[3]) {
  const double t0 = gr * dd[0], t1 = gr * dd[1], t2 = gr * dd[2];
  w[0] = fma(t0, dd[0], w[0]); w[1] = fma(t1, dd[1], w[1]); w[2] = fma(t2, dd[2], w[2]);
  w[3] = fma(t0, dd[1], w[3]); w[4] = fma(t0, dd[2], w[4]); w[5] = fma(t1, dd[2], w[5]);
}

// an empty list, by the kernel that runs before the one that fills it
__device__ __forceinline__ void work_clear(unsigned long long* pack) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *pack = 0;
}
__device__ __forceinline__ void work_clear(const MDArgs& a) { work_clear(a.work_pack); }
// ------------------------------------------------------------------ force kernels
// List entries of one trip: UNR consecutive entries of one list block, as 32-bit words loaded with
// one vector load (the trip's first entry is a multiple of UNR, so they are aligned).
template <class LT>
struct ListVec {
  static constexpr int W = UNR * (int)sizeof(LT) / 4;
  static_assert(W == 1 || W == 2 || W == 4, "one vector load per trip");
  uint32_t w[W];
  __device__ void load(const LT* p) {
    if constexpr (W == 1) {
      w[0] = *(const uint32_t*)p;
    } else if constexpr (W == 2) {
      const uint2 v = *(const uint2*)p;
      w[0] = v.x; w[1] = v.y;
    } else {
      const uint4 v = *(const uint4*)p;
      w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
    }
  }
  // the entries are waited for here whether or not they are used, so that the compiler does not put
  // off their request until it has seen the list's length
  __device__ void arrived() {
#pragma unroll
    for (int q = 0; q < W; ++q) asm volatile("" : "+v"(w[q]));
  }
  __device__ int get(int u) const {
    if constexpr (sizeof(LT) == 2) return (int)((w[u >> 1] >> ((u & 1) * 16)) & 0xffffu);
    else return (int)w[u];
  }
};
static_assert(8 % UNR == 0, "a trip's entries must lie in one list block");

// One lane's walk over atom i's list.  Per trip the lane takes UNR consecutive entries (one vector
// load) and the TPA lanes of the atom take consecutive groups of UNR.  The next trip's entries are
// requested right after this trip's gathers are issued, so a trip waits for one memory round trip
// (the gathers), not two.  Entries at or past the end gather the cell's first atom and come back with
// ok = false: the pair loops run straight-line code and mask those slots out.  sc points at the
// cell's first atom.
template <class P, int TPA, class LT>
struct NbrWalk {
  const LT* list;
  unsigned np, ii;
  int nn, k0, lb;
  ListVec<LT> nx;
  __device__ NbrWalk(const MDArgs& a, long long i, int lane)
      : list((const LT*)a.nbr), np((unsigned)a.npad), ii((unsigned)i), nn(a.nn[i]), k0(lane * UNR), lb(a.lblk), nx{} {
    // not waiting for the length
    if (k0 < a.maxnb) nx.load(list + list_index((unsigned)k0, np, ii, lb));
  }
  __device__ bool more() const { return k0 < nn; }
  __device__ void next(const typename P::S* sc, typename P::S sj[UNR], bool ok[UNR], int j[UNR]) {
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      ok[u] = k0 + u < nn;
      j[u] = ok[u] ? nx.get(u) : 0;
      sj[u] = P::load_rel(sc, j[u]);
    }
    k0 += UNR * TPA;
    if (k0 < nn) nx.load(list + list_index((unsigned)k0, np, ii, lb));
  }
};

// The pruned list: of the full list's entries, which reach to rc + skin, those that were within
// sqrt(prune_rc2) when a pass last walked the full list, kept for each of the atom's TPA lanes apart and
// in order.  A lane therefore adds the same pairs in the same order from either list - the entries left
// out add exact zeros - and the forces do not depend on which list a step walked.  Trip t of lane l of
// atom i: UNR entries at ((t npad + i) TPA + l) UNR, so a wave reads its trips in one piece.
// A pair left out was at least sqrt(prune_rc2) apart, so the list is complete while no atom has moved
// further than (sqrt(prune_rc2) - rc) / 2 since: every step adds its largest displacement to the
// cell's pmove, and past prune_move the cell's next pass prunes again (reduce_cell).
// Kremer-Grest lists shrink from ~21 entries to ~9 this way, copper's from 237 to ~140.  Traced, a pass over 5.1 M
// Kremer-Grest beads (skin 0.7) takes 261 us on the pruned list and 400 where it writes it, 321 on the average of
// a run, against 376 without a pruned list; copper's two passes over 512 000 atoms 84 + 133 us and 212 + 138
// where the first writes, 98 + 140 on average, against 117 + 175.  A cell whose fastest atom uses the margin up
// in every step pays for writing each time, 6 % of such a Kremer-Grest pass.
// Pruning in a walk of its own before the forces (FP32 distances only) was slower.
template <class P, int TPA, class LT>
struct PruneWalk {
  const LT* p;
  size_t stride;
  int n, k;
  ListVec<LT> nx;
  __device__ PruneWalk(const MDArgs& a, long long i, int lane)
      : p((const LT*)a.pl + ((size_t)i * TPA + lane) * UNR), stride((size_t)a.npad * TPA * UNR), n(a.pn[(size_t)i * TPA + lane]), k(0), nx{} {
    nx.load(p);                    // not waiting for the length
  }
  __device__ bool more() const { return k < n; }
  __device__ void next(const typename P::S* sc, typename P::S sj[UNR], bool ok[UNR], int j[UNR]) {
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      ok[u] = k + u < n;
      j[u] = ok[u] ? nx.get(u) : 0;
      sj[u] = P::load_rel(sc, j[u]);
    }
    k += UNR;
    p += stride;
    if (k < n) nx.load(p);
  }
};
// The writer: a lane's kept entries are collected in LDS, four trips deep, and go out as whole trips
// when some lane of the wave has three of them (a branch and a store per entry took copper's density
// pass from 127 to 319 us where it prunes).
template <int NT, class LT>
struct PruneBuf { LT e[4][NT][UNR]; };
template <int TPA, class LT>
struct PruneWriter {
  static constexpr int NT = TILE * TPA;
  PruneBuf<NT, LT>& buf;
  LT* p;
  size_t stride;
  unsigned n = 0, out = 0;         // entries kept, trips stored
  __device__ PruneWriter(const MDArgs& a, long long i, int lane, PruneBuf<NT, LT>& b)
      : buf(b), p((LT*)a.pl + ((size_t)i * TPA + lane) * UNR), stride((size_t)a.npad * TPA * UNR) {}
  __device__ void keep(bool yes, int j) {
    if (yes) buf.e[(n / UNR) & 3][threadIdx.x][n % UNR] = (LT)j;
    n += yes ? 1u : 0u;
  }
  __device__ void store() {
    struct alignas(sizeof(LT) * UNR) Trip { LT e[UNR]; };
    *(Trip*)p = *(const Trip*)buf.e[out & 3][threadIdx.x];
    p += stride;
    ++out;
  }
  // after a trip: at most 2 whole trips and 3 entries stay, and the next adds at most UNR
  __device__ void trip() {
    if (__any(n / UNR - out >= 3u))
      while (n / UNR > out) store();
  }
  __device__ void done(const MDArgs& a, long long i, int lane) {
    a.pn[(size_t)i * TPA + lane] = (unsigned short)n;
    while (n > out * UNR) store();               // the last one perhaps partly filled
  }
};
struct NoWriter {
  __device__ void keep(bool, int) {}
  __device__ void trip() {}
};
// whether this pass over a cell walks the full list and writes the pruned one
__device__ __forceinline__ bool prune_now(const MDArgs& a, const CellDev& C) {
  return a.pl && (a.prune_mode == 0 ? C.prune != 0 : a.prune_mode == 1);
}
// The end of both force passes: the lanes' sums of each atom, its integration tail (first lane) and the
// tile's Part.
template <class P, int TPA>
__device__ __forceinline__ void finish_atoms(const MDArgs& a, const CellK<P>& ck, const Tile& t, int tb, long long i, int lane,
                                             bool active, int mode, const typename P::R f[3], const double w[6], double PE,
                                             const TailIn& in, int status, PartShared<TPA>& psh) {
  double W[6], K[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int q = 0; q < 6; ++q) W[q] = 0.5 * lane_sum<TPA>(w[q]);
  const double fc0 = (double)lane_sum<TPA>(f[0]), fc1 = (double)lane_sum<TPA>(f[1]), fc2 = (double)lane_sum<TPA>(f[2]);
  TailOut o;
  o.maxd2 = o.step2 = 0.f;
  o.xi[0] = o.xi[1] = o.xi[2] = 0;
  if (lane != 0) {
#pragma unroll
    for (int q = 0; q < 6; ++q) W[q] = 0.0;
    PE = 0.0;
  }
  if (active && lane == 0) {
    atom_tail<P>(a, ck, t.cell, i, fc0, fc1, fc2, mode, o, in);
#pragma unroll
    for (int q = 0; q < 6; ++q) K[q] = o.K[q];
  }
  double V[6];
  part_values(a, mode, W, K, V);
  write_part<TILE * TPA>(a.parts, tb, V, PE, mode != MODE_STEP, o.xi, o.maxd2, o.step2, status, psh);
  work_clear(a);                   // here and not earlier: a store ahead of the loads would keep them off the scalar cache
}

// Kremer-Grest: LJ truncated and shifted at rc on every listed pair + FENE on bonds; then the
// integration tail.  TPA lanes share one atom's neighbour list.  MID: the middle steps of a run
// (MODE_STEP), where no energy is reported: neither its terms nor the logarithm of the bonds are
// evaluated.
template <class P, int TPA, class LT, bool MID>
__global__ __launch_bounds__(TILE * TPA) void k_force_kg(MDArgs a, int mode_) {
  using R = typename P::R;
  constexpr int NT = TILE * TPA;
  __shared__ PartShared<NT / 64> psh;
  __shared__ __attribute__((aligned(16))) PruneBuf<NT, LT> pbuf;
  const int mode = MID ? (int)MODE_STEP : mode_;
  const int tb = block_tile_xcd(a.ntiles, blockIdx.x);
  if (tb >= a.ntiles) return;
  const Tile t = a.tiles[tb];
  const CellDev& C = a.cells[t.cell];
  const CellK<P> ck(C);
  const int coff = C.off;
  const bool prune = prune_now(a, C);
  const int slot = threadIdx.x / TPA, lane = threadIdx.x % TPA;
  const bool skip = !MID && ((mode == MODE_PRIME && !C.pending) || (mode == MODE_STATIC && C.fdone));
  const bool active = slot < t.count && !skip;
  const long long i = (long long)t.begin + slot;
  R f[3] = {0, 0, 0}, pe = 0;
  double w[6] = {0, 0, 0, 0, 0, 0};
  TailIn in;
  int status = 0;
  if (active) {
    // the atom's own fixed-point coordinates are recomputed from its position (they are stored only
    // for the neighbours' gathers): the position is read here for the drift anyway
    in.x[0] = a.x[i]; in.x[1] = a.y[i]; in.x[2] = a.z[i];
    const R rc2 = (R)a.rc2, rp2 = (R)a.prune_rc2, sig2 = (R)a.lj_sig2, e24 = (R)(24.0 * a.lj_eps), e4 = (R)(4.0 * a.lj_eps), sh = (R)a.lj_shift;
    const typename P::Geo& g = ck.g;
    const typename P::S* sc = (const typename P::S*)a.s_cur + coff;
    typename P::S si;
    // the walk comes with its length and first entries requested, beside the position: one round trip
    auto pairs = [&](auto&& walk, auto&& out) {
      si = fixed_pos<P>(ck, in.x[0], in.x[1], in.x[2]);
      walk.nx.arrived();
      while (walk.more()) {
        typename P::S sj[UNR];
        bool ok[UNR];
        int j[UNR];
        walk.next(sc, sj, ok, j);
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
          R d[3];
          double dd[3];
          P::sep2(sj[u], si, g, d, dd);
          const R r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
          out.keep(ok[u] && r2 < rp2, j[u]);
          const bool in = ok[u] && r2 < rc2;
          const R r2i = P::rcp(r2);
          const R s2 = sig2 * r2i;
          const R s6 = s2 * s2 * s2;
          const R gr = in ? -e24 * (s6 * ((R)2 * s6 - (R)1)) * r2i : (R)0;   // (dU/dr) / r
          f[0] += gr * d[0]; f[1] += gr * d[1]; f[2] += gr * d[2];
          add_virial(w, (double)gr, dd);
          if constexpr (!MID) pe += in ? (R)0.5 * (e4 * s6 * (s6 - (R)1) - sh) : (R)0;
        }
        out.trip();
      }
    };
    if (prune) {
      PruneWriter<TPA, LT> out(a, i, lane, pbuf);
      pairs(NbrWalk<P, TPA, LT>(a, i, lane), out);
      out.done(a, i, lane);
    } else if (a.pl) {
      pairs(PruneWalk<P, TPA, LT>(a, i, lane), NoWriter());
    } else {
      pairs(NbrWalk<P, TPA, LT>(a, i, lane), NoWriter());
    }
    if (lane == 0) {
      const int li = (int)(i - coff);
      int bp[4];
      in.load(a, i, mode == MODE_STEP);
      if constexpr (sizeof(LT) == 2) {
        const uint2 b = ((const uint2*)a.bond)[i];
        bp[0] = (int)(b.x & 0xffffu); bp[1] = (int)(b.x >> 16); bp[2] = (int)(b.y & 0xffffu); bp[3] = (int)(b.y >> 16);
      } else {
        const int4 b = ((const int4*)a.bond)[i];
        bp[0] = b.x; bp[1] = b.y; bp[2] = b.z; bp[3] = b.w;
      }
      const R K = (R)a.fene_K, R02 = (R)a.fene_R02;
      auto fene = [&](int b, const typename P::S& sb) {
        if (b == li) return;                     // empty slot
        R d[3];
        double dd[3];
        P::sep2(sb, si, g, d, dd);
        const R r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
        const R tt = r2 / R02;
        if (!(tt < (R)1)) { status = ST_BOND; return; }
        const R gr = K / ((R)1 - tt);
        f[0] += gr * d[0]; f[1] += gr * d[1]; f[2] += gr * d[2];
        add_virial(w, (double)gr, dd);
        if constexpr (!MID) pe += (R)(-0.25 * a.fene_K * a.fene_R02) * (R)log((double)((R)1 - tt));
      };
      // both partners of a chain's bead requested together (an empty slot reads the atom itself);
      // branch points have more
      const typename P::S b0 = P::load_rel(sc, bp[0]), b1 = P::load_rel(sc, bp[1]);
      fene(bp[0], b0);
      fene(bp[1], b1);
      if (bp[2] != li || bp[3] != li) {
        const typename P::S b2 = P::load_rel(sc, bp[2]), b3 = P::load_rel(sc, bp[3]);
        fene(bp[2], b2);
        fene(bp[3], b3);
      }
    }
  }
  finish_atoms<P, TPA>(a, ck, t, tb, i, lane, active, mode, f, w, MID ? 0.0 : (double)lane_sum<TPA>(pe), in, status, psh);
}

// Sutton-Chen with n = 9, m = 6 is evaluated in powers of s3 = r^-3: with t = a / r,
// t^6 = a^6 s3^2 and t^9 = a^9 s3^3, and the pair scalar of pass 2 becomes
//   g / r = -r^-2 s3^2 (eps n a^9 s3 + m a^6 (F'_i + F'_j)),
// so pass 1 stores F' scaled by m a^6 (sc_fscale); other exponents store F' itself.
template <int SN, int SM>
__device__ __forceinline__ double sc_fscale(const MDArgs& a) {
  if constexpr (SN == 9 && SM == 6) {
    const double a3 = a.sc_a * a.sc_a * a.sc_a;
    return (double)a.sc_m * a3 * a3;
  } else {
    return 1.0;
  }
}

// Sutton-Chen pass 1: host density rho_i and F'(rho_i) = -eps c / (2 sqrt(rho_i)), stored in s.w
// (times sc_fscale).  Where the cell prunes, this pass writes the pruned list that pass 2 walks.
template <class P, int TPA, int SN, int SM, class LT>
__global__ __launch_bounds__(TILE * TPA) void k_eam_rho(MDArgs a, int mode) {
  using R = typename P::R;
  __shared__ __attribute__((aligned(16))) PruneBuf<TILE * TPA, LT> pbuf;
  const int tb = block_tile_xcd(a.ntiles, blockIdx.x);
  if (tb >= a.ntiles) return;
  const Tile t = a.tiles[tb];
  const CellDev& C = a.cells[t.cell];
  const int slot = threadIdx.x / TPA, lane = threadIdx.x % TPA;
  const bool active = slot < t.count && !(mode == MODE_PRIME && !C.pending) && !(mode == MODE_STATIC && C.fdone);
  const long long i = (long long)t.begin + slot;
  R rho = 0;
  if (active) {
    const typename P::S si = P::load(a.s_cur, i);
    const double a3 = a.sc_a * a.sc_a * a.sc_a;
    const R rc2 = (R)a.rc2, rp2 = (R)a.prune_rc2, sa = (R)a.sc_a, sa6 = (R)(a3 * a3), rhoc = (R)a.sc_rhoc;
    const typename P::Geo g = P::geo(C);
    const typename P::S* sc = (const typename P::S*)a.s_cur + C.off;
    auto pairs = [&](auto&& walk, auto&& out) {
      while (walk.more()) {
        typename P::S sj[UNR];
        bool ok[UNR];
        int j[UNR];
        walk.next(sc, sj, ok, j);
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
          R d[3];
          P::sep(sj[u], si, g, d);
          const R r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
          out.keep(ok[u] && r2 < rp2, j[u]);
          R tm;
          if constexpr (SN == 9 && SM == 6) {
            const R ri = P::rsq(r2), s3 = ri * ri * ri;
            tm = sa6 * (s3 * s3);
          } else {
            R tn;
            sc_powers<SN, SM>(sa * P::rsq(r2), a.sc_n, a.sc_m, tn, tm);
          }
          rho += (ok[u] && r2 < rc2) ? tm - rhoc : (R)0;
        }
        out.trip();
      }
    };
    if (prune_now(a, C)) {
      PruneWriter<TPA, LT> out(a, i, lane, pbuf);
      pairs(NbrWalk<P, TPA, LT>(a, i, lane), out);
      out.done(a, i, lane);
    } else if (a.pl) {
      pairs(PruneWalk<P, TPA, LT>(a, i, lane), NoWriter());
    } else {
      pairs(NbrWalk<P, TPA, LT>(a, i, lane), NoWriter());
    }
  }
  rho = lane_sum<TPA>(rho);
  if (active && lane == 0) {
    const R fp = rho > (R)0 ? (R)(-0.5 * a.sc_eps * a.sc_c * sc_fscale<SN, SM>(a)) / sqrt(rho) : (R)0;
    P::store_w(a.s_cur, i, fp);
  }
}

// Sutton-Chen pass 2: pair scalar g = eps phi'(r) + (F'_i + F'_j) rho'(r), then the tail.  MID: the
// middle steps of a run, where no energy is reported.
template <class P, int TPA, int SN, int SM, class LT, bool MID>
__global__ __launch_bounds__(TILE * TPA) void k_force_eam(MDArgs a, int mode_) {
  using R = typename P::R;
  constexpr int NT = TILE * TPA;
  __shared__ PartShared<NT / 64> psh;
  const int mode = MID ? (int)MODE_STEP : mode_;
  const int tb = block_tile_xcd(a.ntiles, blockIdx.x);
  if (tb >= a.ntiles) return;
  const Tile t = a.tiles[tb];
  const CellDev& C = a.cells[t.cell];
  const CellK<P> ck(C);
  const int slot = threadIdx.x / TPA, lane = threadIdx.x % TPA;
  const bool skip = !MID && ((mode == MODE_PRIME && !C.pending) || (mode == MODE_STATIC && C.fdone));
  const bool active = slot < t.count && !skip;
  const long long i = (long long)t.begin + slot;
  R f[3] = {0, 0, 0}, pe = 0;
  double w[6] = {0, 0, 0, 0, 0, 0};
  R fpi = 0;
  TailIn in;
  if (active) {
    const typename P::S si = P::load(a.s_cur, i);
    fpi = P::get_w(si);
    const double a3 = a.sc_a * a.sc_a * a.sc_a;
    const R rc2 = (R)a.rc2, sa = (R)a.sc_a, en = (R)(a.sc_eps * a.sc_n), m = (R)a.sc_m;
    const R eh = (R)(0.5 * a.sc_eps), phic = (R)a.sc_phic;
    const R en9 = (R)(a.sc_eps * a.sc_n * a3 * a3 * a3), eh9 = (R)(0.5 * a.sc_eps * a3 * a3 * a3);
    const typename P::Geo& g = ck.g;
    const typename P::S* sc = (const typename P::S*)a.s_cur + C.off;
    auto pairs = [&](auto&& walk, auto&& out) {
      while (walk.more()) {
        typename P::S sj[UNR];
        bool ok[UNR];
        int j[UNR];
        walk.next(sc, sj, ok, j);
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
          R d[3];
          double dd[3];
          P::sep2(sj[u], si, g, d, dd);
          const R r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
          const bool in = ok[u] && r2 < rc2;
          const R ri = P::rsq(r2);
          R g0, tn;                                                             // g / r, t^n
          if constexpr (SN == 9 && SM == 6) {
            const R ri2 = ri * ri, s3 = ri2 * ri, s6 = s3 * s3;
            g0 = -(ri2 * s6) * (en9 * s3 + (fpi + P::get_w(sj[u])));
            if constexpr (!MID) tn = s6 * s3;                                 // t^9 / a^9
          } else {
            R tm;
            sc_powers<SN, SM>(sa * ri, a.sc_n, a.sc_m, tn, tm);
            g0 = -(ri * ri) * (en * tn + (fpi + P::get_w(sj[u])) * m * tm);
          }
          const R gr = in ? g0 : (R)0;
          f[0] += gr * d[0]; f[1] += gr * d[1]; f[2] += gr * d[2];
          add_virial(w, (double)gr, dd);
          if constexpr (!MID) {
            if constexpr (SN == 9 && SM == 6) pe += in ? eh9 * tn - eh * phic : (R)0;
            else pe += in ? eh * (tn - phic) : (R)0;
          }
        }
      }
    };
    if (a.pl) pairs(PruneWalk<P, TPA, LT>(a, i, lane), NoWriter());      // pass 1 has just brought it up to date
    else pairs(NbrWalk<P, TPA, LT>(a, i, lane), NoWriter());
    if (lane == 0) {
      in.load(a, i, mode == MODE_STEP);
      if (mode == MODE_STEP) { in.x[0] = a.x[i]; in.x[1] = a.y[i]; in.x[2] = a.z[i]; }
    }
  }
  double PE = MID ? 0.0 : (double)lane_sum<TPA>(pe);
  if (!MID && active && lane == 0) {
    // embedding energy -eps c sqrt(rho) = (eps c)^2 / (2 F'(rho)), zero where rho = 0
    const double ec = a.sc_eps * a.sc_c;
    if (fpi != (R)0) PE += ec * ec * sc_fscale<SN, SM>(a) / (2.0 * (double)fpi);
  }
  finish_atoms<P, TPA>(a, ck, t, tb, i, lane, active, mode, f, w, PE, in, 0, psh);
}

// First half kick and drift of a run (the remaining ones are fused into the force kernels).
template <class P>
__global__ __launch_bounds__(TILE) void k_start(MDArgs a) {
  __shared__ PartShared<1> psh;
  work_clear(a);
  const int tb = block_tile(a.ntiles, blockIdx.x);
  if (tb >= a.ntiles) return;
  const Tile t = a.tiles[tb];
  const CellDev& C = a.cells[t.cell];
  const long long i = (long long)t.begin + threadIdx.x;
  int xi[3] = {0, 0, 0};
  float maxd2 = 0.f, step2 = 0.f;
  if ((int)threadIdx.x < t.count) {
    const double f0 = (double)((const typename P::Fst*)a.fx)[i];
    const double f1 = (double)((const typename P::Fst*)a.fy)[i];
    const double f2 = (double)((const typename P::Fst*)a.fz)[i];
    const double vx = a.vx[i] + a.h * f0, vy = a.vy[i] + a.h * f1, vz = a.vz[i] + a.h * f2;
    const double x = a.x[i] + a.dt * vx, y = a.y[i] + a.dt * vy, z = a.z[i] + a.dt * vz;
    a.vx[i] = vx; a.vy[i] = vy; a.vz[i] = vz;
    a.x[i] = x; a.y[i] = y; a.z[i] = z;
    const typename P::S sn = fixed_pos<P>(C, x, y, z);
    P::store_xyz(a.s_cur, i, sn);
    typename P::R d[3];
    P::disp(sn, a.sb[i], P::geo(C), d);
    maxd2 = (float)(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
    step2 = drift2(a.dt, vx, vy, vz);
    if (a.gamma_on) noise_units(a, a.gid[i], t.cell, C.step + 1, xi);
  }
  const double Z[6] = {0, 0, 0, 0, 0, 0};
  write_part<TILE>(a.parts, tb, Z, 0.0, false, xi, maxd2, step2, 0, psh);
}

// ------------------------------------------------------------------ initial velocities
// Maxwell-Boltzmann velocities for the cells created without them (flag[cell] != 0), one block of
// MB_NT threads per cell, before the first neighbour build (atoms still in their original order):
// three normal variates per atom by the Box-Muller transform of four Philox4x32-10 uniforms
// u = (w + 1/2) 2^-32 (counter: atom, cell, and an all-ones step, a domain the Langevin noise never
// reaches; key: the seed), times sqrt(kB T / m); then the centre-of-mass velocity is removed and the
// velocities are scaled so that sum m v^2 = (3N - 3) kB T exactly.  The two sums run in a fixed tree.
constexpr int MB_NT = 256;
__global__ __launch_bounds__(MB_NT) void k_mb_velocities(MDArgs a, const int* flag, double sd, double dof_kt_m) {
  __shared__ double sh[MB_NT];
  const int c = blockIdx.x;
  if (!flag[c]) return;                           // uniform over the block
  const CellDev& C = a.cells[c];
  const int n = C.n;
  double s[3] = {0.0, 0.0, 0.0};
  for (int l = threadIdx.x; l < n; l += MB_NT) {
    uint32_t w[4];
    philox((uint32_t)l, (uint32_t)c, 0xFFFFFFFFu, 0xFFFFFFFFu, a.key0, a.key1, w);
    double u[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) u[q] = ((double)w[q] + 0.5) * 0x1.0p-32;
    const double r0 = sqrt(-2.0 * log(u[0])), r1 = sqrt(-2.0 * log(u[2]));
    const double t0 = 2.0 * M_PI * u[1], t1 = 2.0 * M_PI * u[3];
    const long long i = (long long)C.off + l;
    a.vx[i] = sd * r0 * cos(t0);
    a.vy[i] = sd * r0 * sin(t0);
    a.vz[i] = sd * r1 * cos(t1);
    s[0] += a.vx[i]; s[1] += a.vy[i]; s[2] += a.vz[i];
  }
  double mean[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) mean[q] = block_sum<MB_NT>(s[q], sh) / (double)n;
  double k2 = 0.0;
  for (int l = threadIdx.x; l < n; l += MB_NT) {
    const long long i = (long long)C.off + l;
    const double vx = a.vx[i] - mean[0], vy = a.vy[i] - mean[1], vz = a.vz[i] - mean[2];
    a.vx[i] = vx; a.vy[i] = vy; a.vz[i] = vz;
    k2 += vx * vx + vy * vy + vz * vz;
  }
  k2 = block_sum<MB_NT>(k2, sh);
  const double scale = (n > 1 && k2 > 0.0) ? sqrt(dof_kt_m * (double)(3 * n - 3) / k2) : 0.0;
  for (int l = threadIdx.x; l < n; l += MB_NT) {
    const long long i = (long long)C.off + l;
    a.vx[i] *= scale; a.vy[i] *= scale; a.vz[i] *= scale;
  }
}

// ------------------------------------------------------------------ molecular statics (FIRE)
// Start of a relaxation: FIRE state of every cell, empty stress window, zero velocities.
__global__ void k_fire_cells(CellDev* cells, int ncells, double dt) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= ncells) return;
  CellDev& C = cells[c];
  C.fdt = dt; C.falpha = 0.1; C.fa = 1.0; C.fb = 0.0;
  C.fcount = 0; C.fdone = 0; C.ffreeze = 1; C.fiter = 0;
  for (int q = 0; q < 6; ++q) C.wsum[q] = 0.0;
  C.wcount = 0;
}

__global__ __launch_bounds__(TILE) void k_zero_v(MDArgs a) {
  const int tb = block_tile(a.ntiles, blockIdx.x);
  if (tb >= a.ntiles) return;
  const Tile t = a.tiles[tb];
  if ((int)threadIdx.x >= t.count) return;
  const long long i = (long long)t.begin + threadIdx.x;
  a.vx[i] = 0.0; a.vy[i] = 0.0; a.vz[i] = 0.0;
}

// One FIRE move of the atoms of unconverged cells: velocity mixing (or zero), v += dt f / m,
// x += dt v, new fixed-point coordinates and the displacement since the last build.
template <class P>
__global__ __launch_bounds__(TILE) void k_fire_move(MDArgs a) {
  __shared__ PartShared<1> psh;
  work_clear(a);
  const int tb = block_tile(a.ntiles, blockIdx.x);
  if (tb >= a.ntiles) return;
  const Tile t = a.tiles[tb];
  const CellDev& C = a.cells[t.cell];
  const long long i = (long long)t.begin + threadIdx.x;
  float maxd2 = 0.f, step2 = 0.f;
  if ((int)threadIdx.x < t.count && !C.fdone) {
    const double f0 = (double)((const typename P::Fst*)a.fx)[i];
    const double f1 = (double)((const typename P::Fst*)a.fy)[i];
    const double f2 = (double)((const typename P::Fst*)a.fz)[i];
    double vx = 0.0, vy = 0.0, vz = 0.0;
    if (!C.ffreeze) {
      vx = C.fa * a.vx[i] + C.fb * f0;
      vy = C.fa * a.vy[i] + C.fb * f1;
      vz = C.fa * a.vz[i] + C.fb * f2;
    }
    const double k = C.fdt * (2.0 * a.h / a.dt);    // dt / (m mvv2e)
    vx += k * f0; vy += k * f1; vz += k * f2;
    const double x = a.x[i] + C.fdt * vx, y = a.y[i] + C.fdt * vy, z = a.z[i] + C.fdt * vz;
    a.vx[i] = vx; a.vy[i] = vy; a.vz[i] = vz;
    a.x[i] = x; a.y[i] = y; a.z[i] = z;
    const typename P::S sn = fixed_pos<P>(C, x, y, z);
    P::store_xyz(a.s_cur, i, sn);
    typename P::R d[3];
    P::disp(sn, a.sb[i], P::geo(C), d);
    maxd2 = (float)(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
    step2 = drift2(C.fdt, vx, vy, vz);
  }
  const double Z[6] = {0, 0, 0, 0, 0, 0};
  const int xi[3] = {0, 0, 0};
  write_part<TILE>(a.parts, tb, Z, 0.0, false, xi, maxd2, step2, 0, psh);
}

__global__ void k_fire_iters(const CellDev* cells, int ncells, int* iters, int* done) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= ncells) return;
  iters[c] = cells[c].fiter;
  done[c] = cells[c].fdone;
}

// one thread enters a cell into the work list: one atomic hands out its place and its first tile
// together, so both arrays increase together whatever order the cells come in
__device__ __forceinline__ void work_add(const MDArgs& a, int cell, int ntile) {
  const unsigned long long old = atomicAdd(a.work_pack, (1ull << 32) | (unsigned)ntile);
  a.work_cells[old >> 32] = cell;
  a.work_tstart[old >> 32] = (int)(unsigned)old;
}
// Per-cell reduction of the tile partials: one wave per cell.  Lane t sums every 64th tile in
// order; the 64 lane sums of each of the 10 summed quantities (V, pe, xi) are then added through
// LDS in a fixed two-level order (four groups of 16 lanes, then the four group sums in order), so
// the result is deterministic for a given tile count.  The cell fields that the update reads are
// loaded at the start, beside the partials, so that none of them waits behind the reduction.
// Every thread of the block calls it (it holds two block barriers); threads from RED_NT on only
// take part in the barriers.
constexpr int RED_NT = 64;
constexpr int RED_Q = 10;         // V[6], pe, xi[3]
struct RedShared {
  double col[RED_Q][RED_NT + 1];
  double grp[4][RED_Q];
};
__device__ __forceinline__ void reduce_cell(const MDArgs& a, int cell, int mode, RedShared& sh, int fill) {
  CellDev& C = a.cells[cell];
  auto& col = sh.col;
  auto& grp = sh.grp;
  const int t = threadIdx.x;
  const int ntile = C.ntile, tile_off = C.tile_off;
  const int pending = C.pending, fdone = C.fdone;
  const int cstatus = C.status, crebuild = C.rebuild, cn = C.n, cprune = C.prune;
  const float chs2 = C.hs2, cpmove = C.pmove;
  const double cV = C.V;
  const long long cnreb = C.nrebuild, cwcount = C.wcount, cstep = C.step;
  double cw[6];
#pragma unroll
  for (int q = 0; q < 6; ++q) cw[q] = C.wsum[q];
  double V[6] = {0, 0, 0, 0, 0, 0}, pe = 0;
  long long xi[3] = {0, 0, 0};
  float m = 0.f, m2 = 0.f;
  int st = 0;
  for (int k = t; k < (t < RED_NT ? ntile : 0); k += RED_NT) {
    const Part& p = a.parts[tile_off + k];
#pragma unroll
    for (int q = 0; q < 6; ++q) V[q] += p.V[q];
    pe += p.pe;
    xi[0] += p.xi[0]; xi[1] += p.xi[1]; xi[2] += p.xi[2];
    m = fmaxf(m, p.maxd2);
    m2 = fmaxf(m2, p.step2);
    st = min(st, p.status);
  }
  if (mode == RED_PRIME && !pending) return;                              // uniform over the block
  if ((mode == RED_STATIC || mode == RED_MOVE) && fdone) return;
  if (t < RED_NT) {
#pragma unroll
    for (int q = 0; q < 6; ++q) col[q][t] = V[q];
    col[6][t] = pe;
#pragma unroll
    for (int q = 0; q < 3; ++q) col[7 + q][t] = __longlong_as_double(xi[q]);
  }
  const float md = wave_max(m), md2 = wave_max(m2);
  st = wave_min(st);
  __syncthreads();
  if (t < RED_NT) {
    const int q = t % 16, g = t / 16;
    const double* c = &col[q < RED_Q ? q : 0][g * 16];
    if (q < 7) {
      double s = 0.0;
#pragma unroll
      for (int k = 0; k < 16; ++k) s += c[k];
      grp[g][q] = s;
    } else if (q < RED_Q) {
      long long s = 0;
#pragma unroll
      for (int k = 0; k < 16; ++k) s += __double_as_longlong(c[k]);
      grp[g][q] = __longlong_as_double(s);
    }
  }
  __syncthreads();
  if (t != 0) return;
  double r[7];
#pragma unroll
  for (int q = 0; q < 7; ++q) r[q] = ((grp[0][q] + grp[1][q]) + grp[2][q]) + grp[3][q];
  long long xs[3];
#pragma unroll
  for (int q = 0; q < 3; ++q)
    xs[q] = __double_as_longlong(grp[0][7 + q]) + __double_as_longlong(grp[1][7 + q]) +
            __double_as_longlong(grp[2][7 + q]) + __double_as_longlong(grp[3][7 + q]);
  const long long x0 = xs[0], x1 = xs[1], x2 = xs[2];
  if (st != 0 && cstatus == 0) C.status = st;
  // the pruned list: a force pass just run has rewritten it if it was asked to; a drift uses up its margin
  const bool moved = mode == RED_MOVE || mode == RED_START || mode == RED_STEP;
  const bool passed = mode != RED_MOVE && mode != RED_START;
  float pm = passed && cprune ? 0.f : cpmove;
  if (moved) pm += 1.000001f * sqrtf(md2);
  C.pmove = pm;
  C.prune = (!passed && cprune) || pm > a.prune_move || (moved && md > chs2);
  if (fill && md > chs2) work_add(a, cell, ntile);
  if (mode == RED_MOVE) {                // statics: positions moved; rebuild when they left the skin
    C.rebuild = md > chs2;
    C.dmax2 = md;
    return;
  }
  if (mode == RED_STATIC) {              // statics: one FIRE decision per cell (same order as the oracle)
    C.pe = r[6];
    const double P = r[0], F2 = r[1], V2 = r[2];
    if ((double)md <= a.fire_ftol2 || st != 0 || C.fiter >= a.fire_max_iter) { C.fdone = 1; C.rebuild = 0; return; }
    if (P > 0.0) {
      if (++C.fcount > 5) { C.fdt = fmin(1.1 * C.fdt, 10.0 * a.dt); C.falpha *= 0.99; }
      C.fa = 1.0 - C.falpha;
      C.fb = C.falpha * sqrt(V2 / F2);
      C.ffreeze = 0;
    } else {
      C.fdt *= 0.5;
      C.falpha = 0.1;
      C.fcount = 0;
      C.ffreeze = 1;
    }
    C.fiter += 1;
    return;
  }
  if (crebuild) C.nrebuild = cnreb + 1;
  if (mode == RED_START) {
    C.rebuild = md > chs2;
    C.dmax2 = md;
    C.xi_mean[0] = (double)x0 / (double)cn;
    C.xi_mean[1] = (double)x1 / (double)cn;
    C.xi_mean[2] = (double)x2 / (double)cn;
    return;
  }
  double s[6];
#pragma unroll
  for (int q = 0; q < 6; ++q) s[q] = r[q] / cV;
  if (mode != RED_STEP) C.pe = r[6];      // the middle steps of a run do not sum the energy
  if (mode == RED_PRIME) {
#pragma unroll
    for (int q = 0; q < 6; ++q) C.last[q] = s[q];
    C.rebuild = 0;
    C.pending = 0;
    return;
  }
#pragma unroll
  for (int q = 0; q < 6; ++q) { C.wsum[q] = cw[q] + s[q]; C.last[q] = s[q]; }
  C.wcount = cwcount + 1;
  C.step = cstep + 1;
  if (mode == RED_STEP) {
    C.rebuild = md > chs2;
    C.dmax2 = md;
    C.xi_mean[0] = (double)x0 / (double)cn;
    C.xi_mean[1] = (double)x1 / (double)cn;
    C.xi_mean[2] = (double)x2 / (double)cn;
  } else {
    C.rebuild = 0;
  }
}

// fill: the reductions that flag rebuilds (RED_START, RED_STEP, RED_MOVE) enter them into the work list
__global__ __launch_bounds__(RED_NT) void k_reduce(MDArgs a, int mode, int fill) {
  __shared__ RedShared sh;
  reduce_cell(a, blockIdx.x, mode, sh, fill);
}

// ------------------------------------------------------------------ neighbour build
// Neighbour build of the cells flagged for a rebuild, in phases:
//   k_bin        per atom: wrap into the box, fixed-point S and the build reference, bin index
//                in scaled space, histogram (tiles)
//   k_bin_scan   exclusive scan of the histogram (one block per cell)
//   k_bin_fill   scatter of cell-local and original indices into their bins (tiles)
//   k_reorder_gather, k_build_list   the atoms in (bin, original index) order, so that the neighbour
//                lists and the force sums built from them are deterministic, then the lists
// atomicAdd(ctr + key, 1) for every valid lane of the wave, one atomic per run of equal keys in
// consecutive lanes: the atoms of a tile are stored in bin order from the last build and have
// mostly stayed in their bins, so neighbouring lanes usually share a key.  The run's first lane
// adds the run length and shares the old value; a lane's slot is that value plus its rank in the
// run (distinct slots, as with one atomic per lane).  Every lane of the wave calls this.
__device__ __forceinline__ int wave_run_add(int* ctr, int key, bool valid) {
  const int lane = (int)(threadIdx.x & 63u);
  const int pkey = __shfl_up(key, 1), pvalid = __shfl_up((int)valid, 1);
  const bool brk = !valid || lane == 0 || !pvalid || pkey != key;
  const unsigned long long breaks = __ballot(brk);
  const unsigned long long le = (2ull << lane) - 1ull;           // lanes <= this one (all for 63)
  const int head = 63 - __clzll(breaks & le);
  const unsigned long long gt = breaks & ~le;
  const int end = gt ? __ffsll((long long)gt) - 1 : 64;
  int old = 0;
  if (valid && head == lane) old = atomicAdd(ctr + key, end - lane);
  return __shfl(old, head) + (lane - head);
}

// an atom wrapped into the box (x updated), its fixed-point coordinates and packed bin; returns the bin
template <class P>
__device__ __forceinline__ int place_atom(const CellDev& C, double x[3], typename P::S& sv, int& packed) {
  const double s0 = C.Hi[0] * x[0] + C.Hi[1] * x[1] + C.Hi[2] * x[2], s1 = C.Hi[4] * x[1] + C.Hi[5] * x[2], s2 = C.Hi[8] * x[2];
  const double k0 = floor(s0), k1 = floor(s1), k2 = floor(s2);
  if (k0 != 0.0 || k1 != 0.0 || k2 != 0.0) {       // x -= H k (a lattice vector), H upper triangular
    x[0] -= C.H[0] * k0 + C.H[1] * k1 + C.H[2] * k2;
    x[1] -= C.H[4] * k1 + C.H[5] * k2;
    x[2] -= C.H[8] * k2;
  }
  double f[3];
  scaled_frac(C, x[0], x[1], x[2], f);
  sv = P::make(f[0], f[1], f[2]);
  int b[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) b[q] = min((int)(f[q] * C.nb[q]), C.nb[q] - 1);
  packed = b[0] | (b[1] << BIN_BITS) | (b[2] << (2 * BIN_BITS));
  return (b[0] * C.nb[1] + b[1]) * C.nb[2] + b[2];
}
template <class P>
__device__ __forceinline__ int bin_one(const MDArgs& a, const CellDev& C, long long i) {
  double x[3] = {a.x[i], a.y[i], a.z[i]};
  typename P::S sv;
  int packed;
  const int bin = place_atom<P>(C, x, sv, packed);
  a.x[i] = x[0]; a.y[i] = x[1]; a.z[i] = x[2];
  P::store_xyz(a.s_cur, i, sv);
  a.sb[i] = P::quant(sv);
  a.abin[i] = packed;
  return bin;
}

template <class P>
__device__ __forceinline__ void bin_atom(const MDArgs& a, const CellDev& C, long long i, bool valid) {
  int bin = -1;
  if (valid) bin = bin_one<P>(a, C, i);
  (void)wave_run_add(a.bcount + C.bin_off, bin, valid);
}

// Tile phases of a rebuild walk the work list: WORK_WAVES tiles per block, one wave per tile,
// block-strided over the tiles of the rebuilding cells, so a step in which few cells rebuild
// launches a small grid instead of one block per tile of the batch.
constexpr int WORK_WAVES = 4;
__device__ __forceinline__ int work_cells_n(const MDArgs& a) { return (int)(*a.work_pack >> 32); }
__device__ __forceinline__ int work_tiles_n(const MDArgs& a) { return (int)(unsigned)*a.work_pack; }
// The last k with start[k] <= w in a strictly increasing array of n entries from 0, for a w common to
// the wave: every lane looks at one entry of 64 (one round trip up to 64 cells, where bisection takes
// one per halving).
__device__ __forceinline__ int work_find(const int* start, int n, int w) {
  const int lane = (int)(threadIdx.x & 63u);
  int lo = 0;
  while (n > 1) {
    const int step = (n + 63) / 64, e = lane * step;
    const int below = __builtin_popcountll(__builtin_amdgcn_ballot_w64(e < n && start[lo + min(e, n - 1)] <= w)) - 1;
    lo += below * step;
    n = min(step, n - below * step);
  }
  return lo;
}
// batch tile index of the w-th tile of the rebuild work list
__device__ __forceinline__ int work_tile(const MDArgs& a, int w) {
  const int k = work_find(a.work_tstart, work_cells_n(a), w);
  return a.cells[a.work_cells[k]].tile_off + (w - a.work_tstart[k]);
}
template <class Fn>
__device__ __forceinline__ void for_work_tiles(const MDArgs& a, Fn&& fn) {
  const int lane = threadIdx.x & 63;
  const XcdLoop L(work_tiles_n(a), WORK_WAVES, threadIdx.x >> 6);
  for (int k = L.k; k < L.end; k += L.step) {
    const Tile t = a.tiles[work_tile(a, k)];
    if (lane < t.count) fn(t, (long long)t.begin + lane);
  }
}
// the same walk with every lane of the wave calling fn (valid: the lane holds an atom of the tile)
template <class Fn>
__device__ __forceinline__ void for_work_tiles_wave(const MDArgs& a, Fn&& fn) {
  const int lane = threadIdx.x & 63;
  const XcdLoop L(work_tiles_n(a), WORK_WAVES, threadIdx.x >> 6);
  for (int k = L.k; k < L.end; k += L.step) {
    const Tile t = a.tiles[work_tile(a, k)];
    const bool valid = lane < t.count;
    fn(t, (long long)t.begin + (valid ? lane : 0), valid);
  }
}

template <class P>
__global__ __launch_bounds__(TILE * WORK_WAVES) void k_bin(MDArgs a) {
  for_work_tiles_wave(a, [&](const Tile& t, long long i, bool valid) { bin_atom<P>(a, a.cells[t.cell], i, valid); });
}

// The displacement threshold for displacements measured against the 16-bit build reference: a
// measured displacement is within qeps of the true one, so the list stays complete while the
// measured one is at most the true bound (squared: hs2) minus qeps.
__device__ __forceinline__ float measured_threshold(double hs2, float qeps) {
  const double h = sqrt(fmax(hs2, 0.0)) - (double)qeps;
  return h > 0.0 ? (float)(h * h) : -1.0f;
}

constexpr int SCAN_NT = 1024;
// Exclusive scan of one value per thread over a block of SCAN_NT threads: an inclusive scan inside
// each wave, the 16 wave totals through LDS (wsum: 16 ints) scanned again by every wave, two barriers.  Returns the exclusive prefix; *total receives the block's sum.
__device__ __forceinline__ int block_exscan(int v, int* wsum, int* total) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int inc = wave_inclusive_scan(v);
  if (lane == 63) wsum[wv] = inc;
  __syncthreads();
  // every wave scans the wave totals for itself
  const int w = wave_inclusive_scan(lane < SCAN_NT / 64 ? wsum[lane] : 0);
  const int before = wv > 0 ? __builtin_amdgcn_readlane(w, wv - 1) : 0;
  *total = __builtin_amdgcn_readlane(w, SCAN_NT / 64 - 1);
  __syncthreads();                 // wsum is reused by the next call
  return before + inc - v;
}

// The bins along z whose lists a wave builds together (build_span): as many as have their candidates, those of
// span + 2 f bins in each column of the stencil, in one register tile, and fewer than half the box.
constexpr float SPAN_CAND = 165.f;  // of 64 BLD_ROUNDS: a span has a few more than the average now and then
// A span leaves the waves enough to do: as many bins as the set has bins per SPAN_TILES atoms' worth of tiles,
// four times as many of half bins.  Longer spans make short work too serial (16 cells of 4000 beads, skin 0.55,
// 1008 tiles: 24 us bin by bin, 34 in spans of two), shorter ones cost rounds (4 such cells in half bins, skin
// 0.4, 252 tiles: 13.7 us, 20 in spans of a quarter of the length).
constexpr float SPAN_TILES = 256.f;
__device__ __forceinline__ void list_span(const MDArgs& a, CellDev& C) {
  const int f = a.bin_factor;
  const float per_atom = (float)(C.nb[0] * C.nb[1] * C.nb[2]) * __builtin_amdgcn_rcpf((float)C.n);
  const int fit = (int)fminf((f == 1 ? SPAN_CAND / 9.f : SPAN_CAND / 25.f) * per_atom, 1024.f) - 2 * f;
  C.span = min(C.nb[0], C.nb[1]) < 2 * f + 3 ? 1 : max(1, min(fit, (C.nb[2] - 1) / 2 - f));
  C.span_rate = (float)(f * f) / SPAN_TILES * per_atom;
}

// Bounds on |d|^2 for the list build's FP32 test (build_span).  A candidate's or an atom's offset from
// the span's first atom is at most pm in each component (three bins in x and y, f + span in z) and is rounded
// once, their difference once more, so a component of d is off by at most 3 2^-24 pm and |d|^2 by at most
// 2 sqrt(3) (rc + skin) times that, plus its own rounding; doubled.
__device__ __forceinline__ void list_band(const MDArgs& a, CellDev& C) {
  const double b0 = 3.0 / C.nb[0], b1 = 3.0 / C.nb[1], b2 = (double)(a.bin_factor + C.span) / C.nb[2];
  const double px = fabs(C.H[0]) * b0 + fabs(C.H[1]) * b1 + fabs(C.H[2]) * b2;
  const double py = fabs(C.H[4]) * b1 + fabs(C.H[5]) * b2, pm = fmax(px, fmax(py, fabs(C.H[8]) * b2));
  const double band = 0x1.0p-23 * (10.4 * sqrt(a.rcs2) * pm + 4.0 * a.rcs2);
  C.list_lo2 = (float)(a.rcs2 - band);
  C.list_hi2 = (float)(a.rcs2 + band);
}

// the cell's fields for a list about to be built, which will hold every pair within rc + skin
__device__ __forceinline__ void begin_build(const MDArgs& a, CellDev& C) {
  const int up[6] = {0, 1, 2, 4, 5, 8};
  for (int q = 0; q < 6; ++q) C.Hb[q] = C.H[up[q]];
  C.hs2 = measured_threshold(a.half_skin2, C.qeps);
  C.dmax2 = 0.f;
  list_span(a, C);
  list_band(a, C);
}

// exclusive scan of one cell's histogram by a block of SCAN_NT threads (sh: at least 16 ints of LDS)
__device__ __forceinline__ void scan_cell(const MDArgs& a, CellDev& C, int* sh) {
  const int nbins = C.nb[0] * C.nb[1] * C.nb[2];
  const int t = threadIdx.x;
  if (t == 0) begin_build(a, C);
  int carry = 0;
  for (int base = 0; base < nbins; base += SCAN_NT) {   // coalesced chunks of SCAN_NT bins
    const int b = base + t;
    const int c = b < nbins ? a.bcount[C.bin_off + b] : 0;
    int tot;
    const int ex = block_exscan(c, sh, &tot);
    if (b < nbins) {
      a.bstart[C.bin_off + b] = carry + ex;
      a.bnum[C.bin_off + b] = c;
      a.bfill[C.bin_off + b] = 0;
      a.bcount[C.bin_off + b] = 0;                        // ready for the next build
    }
    carry += tot;
  }
  __syncthreads();                 // the starts are read by other threads of a fused caller
}

// one block per rebuilding cell, block-strided over the work list
__global__ __launch_bounds__(SCAN_NT) void k_bin_scan(MDArgs a) {
  __shared__ int sh[SCAN_NT / 64];
  const XcdLoop L(work_cells_n(a));
  for (int k = L.k; k < L.end; k += L.step) scan_cell(a, a.cells[a.work_cells[k]], sh);
}

// The work list of a rebuild outside the MD steps (in a step the reduction that flags a cell enters
// it): the cells flagged for one, in cell order.  One block of SCAN_NT threads: exclusive scans of the
// flags and tile counts.
__global__ __launch_bounds__(SCAN_NT) void k_rebuild_work(MDArgs a) {
  __shared__ int sh[SCAN_NT / 64];
  int bc = 0, bt = 0;
  for (int c0 = 0; c0 < a.ncells; c0 += SCAN_NT) {
    const int c = c0 + threadIdx.x;
    int fl = 0, nt = 0;
    if (c < a.ncells && a.cells[c].rebuild) {
      fl = 1;
      nt = a.cells[c].ntile;
    }
    int tc, tt;
    const int ec = block_exscan(fl, sh, &tc);
    const int et = block_exscan(nt, sh, &tt);
    if (fl) {
      a.work_cells[bc + ec] = c;
      a.work_tstart[bc + ec] = bt + et;
    }
    bc += tc; bt += tt;
  }
  if (threadIdx.x == 0) *a.work_pack = ((unsigned long long)bc << 32) | (unsigned)bt;
}

// a bin's index in its cell from its packed coordinates
__device__ __forceinline__ int bin_index(const CellDev& C, int pk) {
  return ((pk & BIN_MASK) * C.nb[1] + ((pk >> BIN_BITS) & BIN_MASK)) * C.nb[2] + (pk >> (2 * BIN_BITS));
}

__device__ __forceinline__ void fill_atom(const MDArgs& a, const CellDev& C, long long i, bool valid) {
  const int bin = valid ? bin_index(C, a.abin[i]) : -1;
  const int slot = wave_run_add(a.bfill + C.bin_off, bin, valid);
  if (valid) {
    const long long q = C.off + a.bstart[C.bin_off + bin] + slot;
    a.binned[q] = (int)(i - C.off);
    a.bkey[q] = a.gid[i];
  }
}

__global__ __launch_bounds__(TILE * WORK_WAVES) void k_bin_fill(MDArgs a) {
  for_work_tiles_wave(a, [&](const Tile& t, long long i, bool valid) { fill_atom(a, a.cells[t.cell], i, valid); });
}

// Reorder the atoms of every rebuilding cell by (bin, original index), so that the order depends only
// on positions, not on earlier reorders.  Phase 1 moves positions, velocities, the fixed-point
// coordinates, bin coordinates and original indices into the scratch rows and records pos_of; phase 2
// copies them back (also as the build reference) and rewrites the bond partners from bond0 through
// pos_of (inside the list build, or as the last phase of the one-block-per-cell preparation).
// The stored total force is not moved: the prime or last step of the run writes it afterwards.
template <class P>
struct Reorder {
  double *x, *y, *z, *vx, *vy, *vz;
  typename P::S* s;
  int *abin, *gid;
  __device__ explicit Reorder(const MDArgs& a) {
    const long long np = a.npad;
    x = (double*)a.pscr; y = x + np; z = y + np; vx = z + np; vy = vx + np; vz = vy + np;
    s = (typename P::S*)(vz + np);
    abin = (int*)(s + np); gid = abin + np;
  }
};

// the four partner slots of the atom at position i (cell-local positions, its own for an empty slot)
__device__ __forceinline__ void store_bonds(const MDArgs& a, long long i, int b0, int b1, int b2, int b3) {
  if (a.bond16)
    ((uint2*)a.bond)[i] = make_uint2((unsigned)b0 | ((unsigned)b1 << 16), (unsigned)b2 | ((unsigned)b3 << 16));
  else
    ((int4*)a.bond)[i] = make_int4(b0, b1, b2, b3);
}

// the atom `src` (batch position) to the scratch row q
template <class P>
__device__ __forceinline__ void reorder_gather_atom(const MDArgs& a, const CellDev& C, long long src, long long q) {
  const Reorder<P> r(a);
  r.x[q] = a.x[src]; r.y[q] = a.y[src]; r.z[q] = a.z[src];
  r.vx[q] = a.vx[src]; r.vy[q] = a.vy[src]; r.vz[q] = a.vz[src];
  r.s[q] = P::load(a.s_cur, src);
  r.abin[q] = a.abin[src];
  const int g = a.gid[src];
  r.gid[q] = g;
  a.pos_of[C.off + g] = (int)(q - C.off);
}

// Phase 1 over the bin slots, in whatever order the fill left a bin's atoms: a slot's place in its bin
// is the number of smaller keys (original indices, distinct) there.  Every lane ranks its own atom, a
// handful of key reads that its neighbours in the bin share, where one lane per bin took a serial
// sort of the whole bin in a launch of its own: 12.6 us per MD step for 100 cells of 10^4 beads at ~5
// atoms per bin, 48 us for 50 glassy cells at ~19, against nothing and +1 us of this kernel.
template <class P>
__device__ __forceinline__ void rank_gather_atom(const MDArgs& a, const CellDev& C, long long q) {
  const long long src = C.off + a.binned[q];
  const int v = a.bkey[q];
  const int bin = C.bin_off + bin_index(C, a.abin[src]);
  const int beg = a.bstart[bin], m = a.bnum[bin];
  const int* key = a.bkey + C.off + beg;
  int rank = 0;
  for (int e = 0; e < m; ++e) rank += key[e] < v;
  reorder_gather_atom<P>(a, C, src, (long long)C.off + beg + rank);
}
template <class P>
__global__ __launch_bounds__(TILE * WORK_WAVES) void k_reorder_gather(MDArgs a) {
  for_work_tiles(a, [&](const Tile& t, long long q) { rank_gather_atom<P>(a, a.cells[t.cell], q); });
}

template <class P>
__device__ __forceinline__ void reorder_scatter_atom(const MDArgs& a, const CellDev& C, long long q) {
  const Reorder<P> r(a);
  a.x[q] = r.x[q]; a.y[q] = r.y[q]; a.z[q] = r.z[q];
  a.vx[q] = r.vx[q]; a.vy[q] = r.vy[q]; a.vz[q] = r.vz[q];
  const typename P::S sq = r.s[q];
  P::store_xyz(a.s_cur, q, sq);
  a.sb[q] = P::quant(sq);
  a.abin[q] = r.abin[q];
  const int g = r.gid[q];
  a.gid[q] = g;
  const int4 b0 = a.bond0[C.off + g];
  const int self = (int)(q - C.off);
  store_bonds(a, q, b0.x < 0 ? self : a.pos_of[C.off + b0.x], b0.y < 0 ? self : a.pos_of[C.off + b0.y],
              b0.z < 0 ? self : a.pos_of[C.off + b0.z], b0.w < 0 ? self : a.pos_of[C.off + b0.w]);
}


// The preparation phases of a rebuild for cells of at most PREP_ATOMS atoms: one block per cell, so a step
// in which no cell rebuilds costs one launch instead of five.  Same results as the phase kernels: the
// order is by (bin, original index), so it depends only on positions.
//
// A block keeps a cell to itself: its histogram, sort keys and new places are in LDS and every thread holds
// its (up to four) atoms in registers from the one read of their rows to the one write, straight to
// their new places once every thread has read.  What bounds it is the round trip of those rows through one CU.
// Through global memory (prep_cell_many_bins) the reduction with a rebuilt cell of 4000 beads took ~62 us,
// 22.1 us averaged over the steps of four such cells; so ~22 and 10.1 us.  First build of 256 copper cells
// of 4000 atoms: 670 / 37 us.
constexpr int PREP_ATOMS = 4096, PREP_BINS = 4096, PREP_SLOTS = PREP_ATOMS / SCAN_NT;
struct PrepShared {
  int scan[SCAN_NT / 64];
  int start[PREP_BINS + 1];        // counts, then first places
  int key[PREP_ATOMS];             // original indices by bin, unordered inside a bin
  unsigned short pos[PREP_ATOMS];  // new place by original index
};
template <class P>
__device__ __forceinline__ void prep_cell(const MDArgs& a, int cell, PrepShared& sh) {
  CellDev& C = a.cells[cell];
  const int n = C.n, t = threadIdx.x, off = C.off, boff = C.bin_off;
  const int nbins = C.nb[0] * C.nb[1] * C.nb[2];
  for (int b = t; b < nbins; b += SCAN_NT) sh.start[b] = 0;
  if (t == 0) begin_build(a, C);
  double x[PREP_SLOTS][3], v[PREP_SLOTS][3];
  int gid[PREP_SLOTS], bin[PREP_SLOTS], slot[PREP_SLOTS], pk[PREP_SLOTS];
#pragma unroll
  for (int e = 0; e < PREP_SLOTS; ++e) {
    const long long i = off + min(t + e * SCAN_NT, n - 1);
    x[e][0] = a.x[i]; x[e][1] = a.y[i]; x[e][2] = a.z[i];
    v[e][0] = a.vx[i]; v[e][1] = a.vy[i]; v[e][2] = a.vz[i];
    gid[e] = a.gid[i];
  }
  __syncthreads();
  typename P::S s[PREP_SLOTS];
#pragma unroll
  for (int e = 0; e < PREP_SLOTS; ++e) {
    bin[e] = place_atom<P>(C, x[e], s[e], pk[e]);
    slot[e] = t + e * SCAN_NT < n ? atomicAdd(&sh.start[bin[e]], 1) : 0;
  }
  __syncthreads();
  // exclusive scan of the counts, consecutive bins per thread
  const int per = (nbins + SCAN_NT - 1) / SCAN_NT, b0 = min(t * per, nbins), b1 = min(b0 + per, nbins);
  int mine = 0, tot;
  for (int b = b0; b < b1; ++b) mine += sh.start[b];
  int at = block_exscan(mine, sh.scan, &tot);
  for (int b = b0; b < b1; ++b) {
    const int c = sh.start[b];
    sh.start[b] = at;
    a.bstart[boff + b] = at;
    a.bnum[boff + b] = c;
    at += c;
  }
  if (t == 0) sh.start[nbins] = n;
  __syncthreads();
#pragma unroll
  for (int e = 0; e < PREP_SLOTS; ++e)
    if (t + e * SCAN_NT < n) sh.key[sh.start[bin[e]] + slot[e]] = gid[e];
  __syncthreads();
  int dest[PREP_SLOTS];
#pragma unroll
  for (int e = 0; e < PREP_SLOTS; ++e) {
    const int beg = sh.start[bin[e]], end = sh.start[bin[e] + 1];
    int rank = 0;
    for (int q = beg; q < end; ++q) rank += sh.key[q] < gid[e];
    dest[e] = beg + rank;
    if (t + e * SCAN_NT < n) sh.pos[gid[e]] = (unsigned short)dest[e];
  }
  __syncthreads();                 // every row has been read, every place is known
#pragma unroll
  for (int e = 0; e < PREP_SLOTS; ++e) {
    if (t + e * SCAN_NT >= n) continue;
    const long long q = off + dest[e];
    a.x[q] = x[e][0]; a.y[q] = x[e][1]; a.z[q] = x[e][2];
    a.vx[q] = v[e][0]; a.vy[q] = v[e][1]; a.vz[q] = v[e][2];
    P::store_xyz(a.s_cur, q, s[e]);
    a.sb[q] = P::quant(s[e]);
    a.abin[q] = pk[e];
    a.gid[q] = gid[e];
    a.pos_of[off + gid[e]] = dest[e];
    const int4 p = a.bond0[off + gid[e]];
    store_bonds(a, q, p.x < 0 ? dest[e] : sh.pos[p.x], p.y < 0 ? dest[e] : sh.pos[p.y],
                p.z < 0 ? dest[e] : sh.pos[p.z], p.w < 0 ? dest[e] : sh.pos[p.w]);
  }
}

// The same through global memory, for a cell with more bins than fit in LDS.
template <class P>
__device__ __forceinline__ void prep_cell_many_bins(const MDArgs& a, int cell, PrepShared& sh) {
  CellDev& C = a.cells[cell];
  const int n = C.n, t = threadIdx.x;
  for (int l0 = 0; l0 < n; l0 += SCAN_NT) {     // whole waves: the bin counts aggregate over lanes
    const bool v = l0 + t < n;
    bin_atom<P>(a, C, (long long)C.off + (v ? l0 + t : 0), v);
  }
  __syncthreads();
  scan_cell(a, C, sh.scan);                  // ends with a barrier
  for (int l0 = 0; l0 < n; l0 += SCAN_NT) {
    const bool v = l0 + t < n;
    fill_atom(a, C, (long long)C.off + (v ? l0 + t : 0), v);
  }
  __syncthreads();
  for (int q = t; q < n; q += SCAN_NT) rank_gather_atom<P>(a, C, (long long)C.off + q);
  __syncthreads();
  for (int q = t; q < n; q += SCAN_NT) reorder_scatter_atom<P>(a, C, (long long)C.off + q);
}
template <class P>
__device__ __forceinline__ void prep_any(const MDArgs& a, int cell, PrepShared& sh) {
  const CellDev& C = a.cells[cell];
  if (C.nb[0] * C.nb[1] * C.nb[2] <= PREP_BINS) prep_cell<P>(a, cell, sh);
  else prep_cell_many_bins<P>(a, cell, sh);
}

template <class P>
__global__ __launch_bounds__(SCAN_NT) void k_cell_prep(MDArgs a) {
  __shared__ PrepShared sh;
  if (!a.cells[blockIdx.x].rebuild) return;
  if (threadIdx.x == 0) work_add(a, blockIdx.x, a.cells[blockIdx.x].ntile);
  prep_any<P>(a, blockIdx.x, sh);
}

// The per-cell reduction of a time step followed, in the same block, by the rebuild preparation
// of a cell that it flags (cells of at most PREP_ATOMS atoms): one launch instead of two per MD
// step.  The flag is read back through the device-coherent path after the barrier.
template <class P>
__global__ __launch_bounds__(SCAN_NT) void k_reduce_prep(MDArgs a, int mode) {
  __shared__ RedShared rsh;
  __shared__ PrepShared sh;
  reduce_cell(a, blockIdx.x, mode, rsh, 1);
  __syncthreads();
  if (!__hip_atomic_load(&a.cells[blockIdx.x].rebuild, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
  prep_any<P>(a, blockIdx.x, sh);
}

// Original order for the atoms of cells [first, first + count) (create, set_state): gid and
// pos_of the identity, bonds as given.  Grid over all tiles.
__global__ __launch_bounds__(TILE) void k_reset_order(MDArgs a, int first, int count) {
  const int tb = block_tile(a.ntiles, blockIdx.x);
  if (tb >= a.ntiles) return;
  const Tile t = a.tiles[tb];
  if (t.cell < first || t.cell >= first + count || (int)threadIdx.x >= t.count) return;
  const long long i = (long long)t.begin + threadIdx.x;
  const int li = (int)(i - a.cells[t.cell].off);
  a.gid[i] = li;
  a.pos_of[i] = li;
  const int4 b0 = a.bond0[i];
  store_bonds(a, i, b0.x < 0 ? li : b0.x, b0.y < 0 ? li : b0.y, b0.z < 0 ? li : b0.z, b0.w < 0 ? li : b0.w);
}

// Verlet list of every atom (after the reorder, so positions are in bin order): cell-local j with
// |d| < rc + skin over the neighbour bins b - f ... b + f of every dimension (bins at least
// (rc + skin) / f wide), in candidate order: the (x, y) columns of the stencil in turn, each column's
// z-neighbour bins one contiguous range of positions (two at the periodic edge in z), because the atoms
// are stored in bin order and bins are numbered with z fastest.  The lists come out nearly sorted by
// position (the force pass's gathers hit few cache lines) and deterministic.
//
// The atoms of one bin have the same candidates, so a wave takes a bin at a time: its lanes hold the
// candidates (64 per round, up to BLD_ROUNDS rounds in registers), read once with coalesced loads
// and turned into Cartesian offsets from the bin's first atom, and every atom of the bin in turn is
// broadcast against them.  The 64-bit mask of a comparison is the accepted candidates in order: an
// accepted lane's place is the running count plus the accepted lanes below it.  No lane waits for a
// longer range of its neighbours', and a cell of 10^4 beads gives ~2200 waves instead of 157.
//
// A wave's cost is per round of 64 candidates and per bin, so bins with few atoms (half bins, short skins) are
// taken several at a time (list_span): `span` bins consecutive in z share the columns of their stencils, which
// are span + 2 f bins long together.  An atom meets candidates beyond its own f bins too, which the distance
// test turns down, and its own in the same order: the lists are the same.  Bin by bin such sets took longer than
// one lane per atom walking its candidates.  16 of 128 cells of 40 000 beads, us, one lane per atom / bin by bin / spans:
// skin 0.4 164 / 193 / 157, 0.55 189 / 177 / 161, 0.4 with half bins 195 / 608 / 202; all 128 of the last
// 2002 / 5320 / 1765.  At skin 0.7 (5.8 beads per bin) a bin fills the register tile: 221 / 178 / 178.  The bar of
// 256 cells of 40 000 beads with some 19 of them rebuilding in every step: 226 / 273 / 220 per step.
constexpr int MAX_BIN_FACTOR = 2;
struct BuildGeo {                  // the stencil of a span of bins: bins per dimension and the z ranges
  int lo[3], cnt[3], nb[3];        // first neighbour bin (unwrapped) and count per dimension
  int zr[2][2], nzr;               // z bins [z0, z1] of every column, or two such ranges
  int ncol, nrange;
};
__device__ __forceinline__ void build_geo(const CellDev& C, const int bb[3], int z1, int fb, BuildGeo& G) {
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    G.nb[q] = C.nb[q];
    // a pair within rc + skin is at most f bins apart in every dimension; a dimension with fewer
    // than 2 f + 1 bins is scanned whole
    if (G.nb[q] >= 2 * fb + 1) { G.lo[q] = bb[q] - fb; G.cnt[q] = 2 * fb + 1; }
    else { G.lo[q] = 0; G.cnt[q] = G.nb[q]; }
  }
  const int nbz = G.nb[2];
  G.zr[0][0] = 0; G.zr[0][1] = nbz - 1; G.zr[1][0] = 0; G.zr[1][1] = 0; G.nzr = 1;
  if (nbz >= 2 * fb + 1) {
    const int lo = bb[2] - fb, hi = z1 + fb;
    if (lo < 0) { G.zr[0][0] = 0; G.zr[0][1] = hi; G.zr[1][0] = lo + nbz; G.zr[1][1] = nbz - 1; G.nzr = 2; }
    else if (hi >= nbz) { G.zr[0][0] = lo; G.zr[0][1] = nbz - 1; G.zr[1][0] = 0; G.zr[1][1] = hi - nbz; G.nzr = 2; }
    else { G.zr[0][0] = lo; G.zr[0][1] = hi; }
  }
  G.ncol = G.cnt[0] * G.cnt[1];
  G.nrange = G.ncol * G.nzr;
}
// a lane's value, in every lane
__device__ __forceinline__ float lane_value(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
template <class P>
__device__ __forceinline__ typename P::S lane_value_s(const typename P::S& v, int l) {
  typename P::S r;
  int w[sizeof(v) / 4];
  __builtin_memcpy(w, &v, sizeof(v));
#pragma unroll
  for (int q = 0; q < (int)(sizeof(v) / 4); ++q) w[q] = __builtin_amdgcn_readlane(w[q], l);
  __builtin_memcpy(&r, w, sizeof(v));
  return r;
}
// whether a pair is listed: |d|^2 below (rc + skin)^2, from the separation that the pair passes form
template <class P>
__device__ __forceinline__ bool exact_in(const typename P::S& sj, const typename P::S& si, const typename P::Geo& g,
                                         typename P::R rcs2) {
  typename P::R d[3];
  P::sep(sj, si, g, d);
  return d[0] * d[0] + d[1] * d[1] + d[2] * d[2] < rcs2;
}

// range r of the stencil (column-major over x, y, then the z parts): first position and count
__device__ __forceinline__ int2 build_range(const MDArgs& a, const CellDev& C, const BuildGeo& G, int r) {
  const int col = G.nzr == 2 ? r >> 1 : r, part = G.nzr == 2 ? r & 1 : 0;
  // col / cnt[1] for col < 64 and cnt[1] <= 2 MAX_BIN_FACTOR + 1
  const int inv = G.cnt[1] == 1 ? 65536 : G.cnt[1] == 2 ? 32768 : G.cnt[1] == 3 ? 21846 : G.cnt[1] == 4 ? 16384 : 13108;
  const int u0 = (col * inv) >> 16, u1 = col - u0 * G.cnt[1];
  int x = G.lo[0] + u0, y = G.lo[1] + u1;
  x = x < 0 ? x + G.nb[0] : (x >= G.nb[0] ? x - G.nb[0] : x);
  y = y < 0 ? y + G.nb[1] : (y >= G.nb[1] ? y - G.nb[1] : y);
  const int bc = C.bin_off + (x * G.nb[1] + y) * G.nb[2];
  const int bf = bc + (part ? G.zr[1][0] : G.zr[0][0]), bl = bc + (part ? G.zr[1][1] : G.zr[0][1]);
  const int beg = a.bstart[bf];
  return make_int2(beg, a.bstart[bl] + a.bnum[bl] - beg);
}

constexpr int BLD_WAVES = 4;       // waves per block of the list build
constexpr int BLD_ROUNDS = 3;      // rounds of 64 candidates held in registers
constexpr int BLD_RUN_TILES = 1024;  // rebuild sets of at least so many tiles: runs of spans per wave
struct BinRanges {                 // one span's candidate ranges, by lane
  int off[64];                     // first candidate of each range (past the last range: INT_MAX)
  int delta[64];                   // position of candidate c of range r: c + delta[r]
};
struct BinHead {                   // a span's atoms and stencil, and this lane's range of it
  int m, first, nrange;
  int2 rng;
};

// bins (x, y, z0) to (x, y, z1) of cell C: their atoms, and the candidate range of every lane below nrange
template <bool SPANS>
__device__ __forceinline__ BinHead bin_head(const MDArgs& a, const CellDev& C, int x, int y, int z0, int z1) {
  const int lane = (int)(threadIdx.x & 63u), col = C.bin_off + (x * C.nb[1] + y) * C.nb[2];
  BinHead h;
  h.first = a.bstart[col + z0];
  if constexpr (SPANS) {           // (the last bin's start and count instead take a wave per SIMD, in registers)
    const bool last = x + 1 == C.nb[0] && y + 1 == C.nb[1] && z1 + 1 == C.nb[2];
    h.m = (last ? C.n : a.bstart[col + z1 + 1]) - h.first;
  } else {
    h.m = a.bnum[col + z0];
  }
  BuildGeo G;
  const int bb[3] = {x, y, z0};
  build_geo(C, bb, z1, a.bin_factor, G);
  h.nrange = G.nrange;
  h.rng = lane < G.nrange ? build_range(a, C, G, lane) : make_int2(0, 0);
  return h;
}

// The lists of the atoms of one span: the wave's share of them, atoms part, part + nparts, ... .
// s: the reordered coordinates of the batch.
//
// LOCAL (at least 2 f + 3 bins in x and y, 2 (f + span) + 1 in z): a candidate (within f bins of the span) lies
// less than half the box from the span's first atom, as every atom of the span does, so the difference of the
// two offsets is the minimum image: the test takes 3 subtractions and 3 multiply-adds in FP32 (issued at nearly
// twice the rate of FP64 and conversions here) on offsets rounded once from FP64.  A candidate whose
// |d|^2 lies between the cell's list_lo2 and list_hi2 takes the exact test, so the lists are those of the exact
// test alone.  With fewer bins every test is the exact one.
template <class P, class LT, bool LOCAL>
__device__ __forceinline__ void build_span(const MDArgs& a, int cell, const BinHead& h, int part, int nparts,
                                          const typename P::S* s, BinRanges& rg) {
  using R = typename P::R;
  const CellDev& C = a.cells[cell];
  const int lane = (int)(threadIdx.x & 63u);
  const int m = __builtin_amdgcn_readfirstlane(h.m), first = __builtin_amdgcn_readfirstlane(h.first);
  if (m <= part) return;
  const typename P::S* sc = s + C.off;
  const int incl = wave_inclusive_scan(h.rng.y);
  const int total = __builtin_amdgcn_readlane(incl, 63), off = incl - h.rng.y;
  __builtin_amdgcn_wave_barrier();                // the last bin's ranges have been read
  rg.off[lane] = lane < h.nrange ? off : 0x7fffffff;
  rg.delta[lane] = h.rng.x - off;
  // candidate index of the span's first atom: its range is the one that holds its position
  const unsigned long long own = __builtin_amdgcn_ballot_w64((unsigned)(first - h.rng.x) < (unsigned)h.rng.y);
  const int self0 = first - __builtin_amdgcn_readlane(h.rng.x - off, __builtin_ctzll(own));
  __builtin_amdgcn_wave_barrier();
  const typename P::Geo g = P::geo(C);
  const R rcs2 = (R)a.rcs2;
  const float lo2 = C.list_lo2, hi2 = C.list_hi2;
  LT* const list = (LT*)a.nbr;
  const unsigned row = (unsigned)a.npad << a.lblk, bm = (1u << a.lblk) - 1u;   // list_index, by rows of blocks
  const int cap = a.maxnb;
  const typename P::S sref = sc[first];
  for (int g0 = 0; g0 < m; g0 += 64) {            // the span's atoms, by lane (one group unless m > 64)
    const int ng = min(64, m - g0);
    const typename P::S so = sc[first + g0 + min(lane, ng - 1)];
    R po[3] = {0, 0, 0};
    if constexpr (LOCAL) P::sep(so, sref, g, po);
    int cnt_reg = 0;
    for (int ct = 0; ct < total; ct += 64 * BLD_ROUNDS) {
      int pos[BLD_ROUNDS];
      typename P::S sj[BLD_ROUNDS];
      float pj[BLD_ROUNDS][3];
#pragma unroll
      for (int q = 0; q < BLD_ROUNDS; ++q) {
        const int c = ct + q * 64 + lane;
        pos[q] = first;
        if (ct + q * 64 < total) {
          int r = 0;                                  // the last range that begins at or before c
          if (h.nrange > 16) {
            r = rg.off[32] <= c ? 32 : 0;
            r = rg.off[r + 16] <= c ? r + 16 : r;
          }
          r = rg.off[r + 8] <= c ? r + 8 : r;
          r = rg.off[r + 4] <= c ? r + 4 : r;
          r = rg.off[r + 2] <= c ? r + 2 : r;
          r = rg.off[r + 1] <= c ? r + 1 : r;
          pos[q] = c < total ? c + rg.delta[r] : first;
        }
        sj[q] = P::load_rel(sc, pos[q]);
      }
      if constexpr (LOCAL) {
#pragma unroll
        for (int q = 0; q < BLD_ROUNDS; ++q) {
          R d[3];
          P::sep(sj[q], sref, g, d);
          const bool ok = ct + q * 64 + lane < total;
#pragma unroll
          for (int e = 0; e < 3; ++e) pj[q][e] = ok ? (float)d[e] : 1e18f;
        }
      }
      // 64 is a multiple of nparts: the wave's atoms of the group are part, part + nparts, ...
      for (int at = part; at < ng; at += nparts) {
        float ox = 0.f, oy = 0.f, oz = 0.f;
        typename P::S si = so;
        if constexpr (LOCAL) { ox = lane_value((float)po[0], at); oy = lane_value((float)po[1], at); oz = lane_value((float)po[2], at); }
        else si = lane_value_s<P>(so, at);
        LT* const li = list + ((size_t)(unsigned)(C.off + first + g0 + at) << a.lblk);
        const int selfc = self0 + g0 + at - ct;
        int cnt = ct ? __builtin_amdgcn_readlane(cnt_reg, at) : 0;
#pragma unroll
        for (int q = 0; q < BLD_ROUNDS; ++q) {
          if (ct + q * 64 >= total) break;
          unsigned long long mask;
          if constexpr (LOCAL) {
            const float dx = pj[q][0] - ox, dy = pj[q][1] - oy, dz = pj[q][2] - oz;
            const float r2 = dx * dx + dy * dy + dz * dz;
            mask = __builtin_amdgcn_ballot_w64(r2 < lo2);
            const unsigned long long most = __builtin_amdgcn_ballot_w64(r2 < hi2);
            if (mask != most)
              mask |= most & __builtin_amdgcn_ballot_w64(exact_in<P>(P::load_rel(sc, pos[q]), lane_value_s<P>(so, at), g, rcs2));
          } else {
            mask = __builtin_amdgcn_ballot_w64(exact_in<P>(sj[q], si, g, rcs2));
            const int left = total - ct - q * 64;
            if (left < 64) mask &= (1ull << left) - 1ull;
          }
          if ((selfc >> 6) == q) mask &= ~(1ull << (selfc & 63));
          const unsigned k = __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, (unsigned)cnt));
          cnt += __builtin_popcountll(mask);
          if (cnt > cap) mask &= __builtin_amdgcn_ballot_w64((int)k < cap);
          if (__builtin_amdgcn_inverse_ballot_w64(mask)) li[(size_t)(k >> a.lblk) * row + (k & bm)] = (LT)pos[q];
        }
        cnt_reg = lane == at ? cnt : cnt_reg;
      }
    }
    if (lane < ng && (lane & (nparts - 1)) == part) {
      if (cnt_reg > cap) atomicMin(&a.cells[cell].status, (int)ST_CAP);
      a.nn[C.off + first + g0 + lane] = min(cnt_reg, cap);
    }
  }
}

// `run` consecutive spans of one cell from its span b0, of `len` bins each but the last of a column, the next
// span's ranges requested before a span's candidates are tested (SPANS: len may be more than one)
template <class P, class LT, bool SPANS>
__device__ __forceinline__ void build_run(const MDArgs& a, int cell, int b0, int run, int len, int ns, int part, int nparts,
                                          const typename P::S* s, BinRanges& rg) {
  const CellDev& C = a.cells[cell];
  const int nb0 = C.nb[0], nb1 = C.nb[1], nb2 = C.nb[2];
  const bool local = min(min(nb0, nb1), nb2) >= 2 * a.bin_factor + 3;
  int z = b0 % ns * len, t = b0 / ns;
  int y = t % nb1, x = t / nb1;
  auto head = [&] { return bin_head<SPANS>(a, C, x, y, z, SPANS ? min(z + len, nb2) - 1 : z); };
  BinHead cur = head();
  for (int e = 0; e < run; ++e) {
    z += len;
    if (z >= nb2) { z = 0; if (++y == nb1) { y = 0; ++x; } }
    BinHead nxt = cur;
    if (e + 1 < run) nxt = head();
    if (local) build_span<P, LT, true>(a, cell, cur, part, nparts, s, rg);
    else build_span<P, LT, false>(a, cell, cur, part, nparts, s, rg);
    cur = nxt;
  }
}

// The lists of the rebuilding cells, over the work list, block-strided (XcdLoop).  An item is a tile's
// share of its cell's spans, split over 2^lsplit waves: a run of a few consecutive spans whose cell is
// looked up once; where bins hold many atoms (copper: ~60), 2^lparts waves share each bin's atoms.
// scatter: after the phase kernels the reorder's second half is done here too, tile by tile - nothing
// else reads the arrays that it writes, and the candidates come from the scratch rows, which hold the
// same reordered coordinates.  After the one-block-per-cell preparation, which reorders completely,
// they are read from s_cur.
// Measured on one MI355X, per MD step, against one lane per atom (sets of 4096 tiles and more) and eight
// lanes per atom walking the candidate ranges: 100 cells of 10^4 beads 62.6 -> 37.1 us, 50 glassy
// cells 102 -> 54 us, 128 cells of 40 000 beads 205 -> 147 us (all 5.1 M beads at once 2.19 -> 1.57 ms).
// SPANS: batches with a cell whose bins are few atoms (set_build_shape); the others keep the shorter code, 2 % of a
// build of 5.1 M beads.
template <class P, class LT, bool SPANS>
__global__ __launch_bounds__(64 * BLD_WAVES) void k_build_list(MDArgs a, int scatter, int lparts) {
  __shared__ BinRanges rg[BLD_WAVES];
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int nc = work_cells_n(a), ntl = work_tiles_n(a);
  if (ntl == 0) return;
  const Reorder<P> ro(a);
  if (scatter)
    for_work_tiles(a, [&](const Tile& t, long long i) { reorder_scatter_atom<P>(a, a.cells[t.cell], i); });
  const typename P::S* s = scatter ? ro.s : (const typename P::S*)a.s_cur;
  // a tile holds 10-14 bins at Kremer-Grest densities: single spans until every resident wave has two,
  // then runs of three or four (5.1 M beads at once: 1.95 ms by single bins, 1.62 ms by runs of four);
  // 3-4 of the glassy cells' fuller bins (two waves each), one of copper's
  const int lsplit = lparts > 1 ? 0 : lparts == 1 ? 2 : ntl < BLD_RUN_TILES ? 4 : 2;
  const XcdLoop L((ntl << lsplit) << lparts, BLD_WAVES, wave);
  for (int k = L.k; k < L.end; k += L.step) {
    const int it = k >> lparts, part = k & ((1 << lparts) - 1);
    const int w = work_find(a.work_tstart, nc, it >> lsplit);
    const int cell = __builtin_amdgcn_readfirstlane(a.work_cells[w]);
    const int q = it - (__builtin_amdgcn_readfirstlane(a.work_tstart[w]) << lsplit);
    const CellDev& C = a.cells[cell];
    const int nb2 = C.nb[2], cols = C.nb[0] * C.nb[1];
    int len = 1, ns = nb2;
    if constexpr (SPANS) {
      len = max(1, min(C.span, (int)((float)ntl * C.span_rate)));
      if (len > 1) {               // about equal in a column
        ns = (nb2 + len - 1) / len;
        len = (nb2 + ns - 1) / ns;
        ns = (nb2 + len - 1) / len;
      }
    }
    const unsigned nu = (unsigned)(cols * ns), nq = (unsigned)C.ntile << lsplit;
    const int b0 = (int)((unsigned long long)q * nu / nq), b1 = (int)((unsigned long long)(q + 1) * nu / nq);
    if (b1 > b0) build_run<P, LT, SPANS>(a, cell, b0, b1 - b0, len, ns, part, 1 << lparts, s, rg[wave]);
  }
}

// ------------------------------------------------------------------ QR box remap (Eqs. 4, 5, 9)
__device__ inline double det3(const double A[9]) {
  return A[0] * (A[4] * A[8] - A[5] * A[7]) - A[1] * (A[3] * A[8] - A[5] * A[6]) + A[2] * (A[3] * A[7] - A[4] * A[6]);
}
__device__ inline void mat3mul(const double A[9], const double B[9], double C[9]) {
  for (int r = 0; r < 3; ++r)
    for (int c = 0; c < 3; ++c) C[3 * r + c] = A[3 * r] * B[c] + A[3 * r + 1] * B[3 + c] + A[3 * r + 2] * B[6 + c];
}
__device__ inline void upper_inv(const double U[9], double Ui[9]) {   // inverse of an upper-triangular matrix
  const double a = U[0], b = U[1], c = U[2], d = U[4], e = U[5], f = U[8];
  Ui[0] = 1.0 / a; Ui[1] = -b / (a * d); Ui[2] = (b * e - c * d) / (a * d * f);
  Ui[3] = 0.0; Ui[4] = 1.0 / d; Ui[5] = -e / (d * f);
  Ui[6] = 0.0; Ui[7] = 0.0; Ui[8] = 1.0 / f;
}
__device__ inline void box_widths(const double H[9], double w[3]) {  // w_k = V / |a_i x a_j| for columns of H
  const double V = fabs(det3(H));
  for (int k = 0; k < 3; ++k) {
    const int i = (k + 1) % 3, j = (k + 2) % 3;
    const double u0 = H[i], u1 = H[3 + i], u2 = H[6 + i], v0 = H[j], v1 = H[3 + j], v2 = H[6 + j];
    const double cx = u1 * v2 - u2 * v1, cy = u2 * v0 - u0 * v2, cz = u0 * v1 - u1 * v0;
    w[k] = V / sqrt(cx * cx + cy * cy + cz * cz);
  }
}

// F = Q R by classical Gram-Schmidt on the columns of F with one re-orthogonalisation pass;
// R_jj = |v_j| > 0.  Returns 0 or ST_BAD_F (non-finite F, det F <= 0, R_jj < 1e-12 |F|_F).
__device__ inline int qr_gs(const double F[9], double Q[9], double R[9]) {
  double fn = 0.0;
  for (int k = 0; k < 9; ++k) {
    if (!isfinite(F[k])) return ST_BAD_F;
    fn += F[k] * F[k];
    R[k] = 0.0;
  }
  fn = sqrt(fn);
  if (!(det3(F) > 0.0)) return ST_BAD_F;
  double q[3][3];
  for (int j = 0; j < 3; ++j) {
    double v0 = F[j], v1 = F[3 + j], v2 = F[6 + j];
    for (int pass = 0; pass < 2; ++pass)
      for (int i = 0; i < j; ++i) {
        const double s = q[i][0] * v0 + q[i][1] * v1 + q[i][2] * v2;
        R[3 * i + j] += s;
        v0 -= s * q[i][0]; v1 -= s * q[i][1]; v2 -= s * q[i][2];
      }
    const double nv = sqrt(v0 * v0 + v1 * v1 + v2 * v2);
    if (!(nv >= 1e-12 * fn)) return ST_BAD_F;
    R[3 * j + j] = nv;
    q[j][0] = v0 / nv; q[j][1] = v1 / nv; q[j][2] = v2 / nv;
  }
  for (int r = 0; r < 3; ++r)
    for (int c = 0; c < 3; ++c) Q[3 * r + c] = q[c][r];
  return 0;
}

// keep |yz| <= ly/2, |xz| <= lx/2, |xy| <= lx/2 by subtracting integer multiples of box edges
__device__ inline void tilt_reduce(double H[9]) {
  if (fabs(H[5]) > 0.5 * H[4]) { const double k = floor(H[5] / H[4] + 0.5); H[2] -= k * H[1]; H[5] -= k * H[4]; }
  if (fabs(H[2]) > 0.5 * H[0]) { const double k = floor(H[2] / H[0] + 0.5); H[2] -= k * H[0]; }
  if (fabs(H[1]) > 0.5 * H[0]) { const double k = floor(H[1] / H[0] + 0.5); H[1] -= k * H[0]; }
}

// stage everything a deformation needs; no state is modified (bw: the bin width, (rc + skin) / f)
__device__ inline void qr_stage_cell(const double* Fall, const CellDev& C, Stage& S, int c, double rcs, double bw) {
  for (int k = 0; k < 9; ++k) S.F[k] = Fall[9 * c + k];
  S.status = qr_gs(S.F, S.Q, S.R);
  if (S.status) return;
  double Ri[9];
  upper_inv(C.Rprev, Ri);
  mat3mul(S.R, Ri, S.dR);                       // Eq. (9)
  S.dR[3] = S.dR[6] = S.dR[7] = 0.0;
  mat3mul(S.dR, C.H, S.Hn);                     // H <- Delta R H
  S.Hn[3] = S.Hn[6] = S.Hn[7] = 0.0;
  tilt_reduce(S.Hn);
  S.J = S.R[0] * S.R[4] * S.R[8];
  double w[3];
  box_widths(S.Hn, w);
  S.wmin = fmin(w[0], fmin(w[1], w[2]));
  if (rcs > 0.5 * S.wmin) { S.status = ST_BOX; return; }
  for (int q = 0; q < 3; ++q) S.nb[q] = min(BIN_MASK, max(1, (int)floor(w[q] / bw)));
  S.nbins = S.nb[0] * S.nb[1] * S.nb[2];
  S.density = (double)C.n / fabs(det3(S.Hn));
}

// The results that the host decides by go straight to its memory (pinned), next to the ones that the commit
// behind this kernel reads: a cell whose F is refused, that needs more bins than it has or is denser
// than the lists are sized for holds the whole batch back.
__global__ void k_qr_stage(const double* Fall, const CellDev* cells, Stage* st, int ncells, double rcs, double bw,
                           double dens_ok, int* status, int* nbins, double* density) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= ncells) return;
  Stage& S = st[c];
  S.nbins = 0; S.density = 0.0;
  qr_stage_cell(Fall, cells[c], S, c, rcs, bw);
  S.hold = S.status != 0 || S.nbins > cells[c].bin_cap || S.density > dens_ok;
  status[c] = S.status; nbins[c] = S.nbins; density[c] = S.density;
}

// fill the derived box fields of a cell from C.H (bw: the bin width)
__device__ inline void set_box_fields(CellDev& C, double bw) {
  upper_inv(C.H, C.Hi);
  C.V = det3(C.H);
  const int up[6] = {0, 1, 2, 4, 5, 8};
  for (int q = 0; q < 6; ++q) {
    const double hs = C.H[up[q]] * TWOM32;
    C.Hm[q] = hs;
    C.Hd[q] = hs * TWOM32;
  }
  // the 16-bit build reference is within 2^-17 of the position in each scaled coordinate, so a
  // measured displacement is within |H|_F sqrt(3) 2^-17 of the true one (with a relative margin for
  // the FP32 arithmetic of the check)
  double hf = 0.0;
  for (int q = 0; q < 6; ++q) hf += C.H[up[q]] * C.H[up[q]];
  C.qeps = (float)(1.001 * sqrt(3.0 * hf) * 0x1.0p-17);
  double w[3];
  box_widths(C.H, w);
  for (int q = 0; q < 3; ++q) C.nb[q] = min(BIN_MASK, max(1, (int)floor(w[q] / bw)));
  // never exceed the bins allocated to this cell: coarser bins are still valid (>= the bin width)
  while (C.nb[0] * C.nb[1] * C.nb[2] > max(C.bin_cap, 1)) {
    int q = 0;
    if (C.nb[1] > C.nb[q]) q = 1;
    if (C.nb[2] > C.nb[q]) q = 2;
    C.nb[q] -= 1;
  }
}

// Whether the neighbour list survives a box change.  With A = H Hb^-1 the affine map since the
// last build and u the largest atom displacement since then (measured in the current box), a pair
// left out of the list (|d_build| >= rc + skin) is now at least sigma_min(A) (rc + skin) - 2 u
// apart, and sigma_min(A) >= 1 - |A - I|_F.  The list therefore still holds every pair within rc
// while u <= ((1 - |A - I|_F)(rc + skin) - rc) / 2; that bound becomes the cell's displacement
// threshold.  A rebuild is forced when it is not positive, or when the displacement the atoms
// already have exceeds it: the remap x <- dR x leaves the scaled offsets since the build unchanged,
// so it stretches the last measured displacement by at most |dR|_2 <= 1 + |dR - I|_F.
__device__ inline float kept_list_threshold(const CellDev& C, double rc, double rcs) {
  const double Hb[9] = {C.Hb[0], C.Hb[1], C.Hb[2], 0.0, C.Hb[3], C.Hb[4], 0.0, 0.0, C.Hb[5]};
  double Hbi[9], A[9];
  upper_inv(Hb, Hbi);
  mat3mul(C.H, Hbi, A);
  double e2 = 0.0;
  for (int k = 0; k < 9; ++k) {
    const double d = A[k] - ((k % 4 == 0) ? 1.0 : 0.0);
    e2 += d * d;
  }
  const double hs = 0.5 * ((1.0 - sqrt(e2)) * rcs - rc);
  return hs > 0.0 ? (float)(hs * hs) : -1.0f;
}

__global__ void k_qr_commit(CellDev* cells, Stage* st, int ncells, double rc, double rcs, double bw,
                            int force_build, int checked) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  int hold = 0;
  if (!checked)
    for (int k = threadIdx.x; k < ncells; k += blockDim.x) hold |= st[k].hold;
  hold = __syncthreads_or(hold);
  if (c >= ncells) return;
  CellDev& C = cells[c];
  Stage& S = st[c];
  S.go = !hold;
  if (hold) return;
  for (int k = 0; k < 9; ++k) {
    C.H[k] = S.Hn[k]; C.Q[k] = S.Q[k]; C.R[k] = S.R[k]; C.Rprev[k] = S.R[k]; C.F[k] = S.F[k];
  }
  C.J = S.J;
  const float qeps_old = C.qeps;
  set_box_fields(C, bw);
  for (int q = 0; q < 6; ++q) C.wsum[q] = 0.0;
  C.wcount = 0;
  const float hs2 = kept_list_threshold(C, rc, rcs);
  double e2 = 0.0;
  for (int k = 0; k < 9; ++k) {
    const double d = S.dR[k] - ((k % 4 == 0) ? 1.0 : 0.0);
    e2 += d * d;
  }
  const double grow = 1.0 + sqrt(e2);
  const double u = (sqrt((double)C.dmax2) + (double)qeps_old) * grow;   // bound on the true displacement
  const float hs2m = hs2 > 0.0f ? measured_threshold((double)hs2, C.qeps) : -1.0f;
  const bool moved = !(hs2 > 0.0f) || u * u >= (double)hs2;
  if (force_build || C.rebuild || moved || !(hs2m > 0.0f)) {
    C.rebuild = 1;
  } else {
    C.hs2 = hs2m;
  }
  C.pending = 1;
  C.prune = 1;
}

// x <- Delta R x for every atom (affine remap, Eq. 6 applied incrementally), with the fixed-point
// scaled coordinates of the remapped positions in the committed box (they equal the old ones up
// to rounding: the remap leaves S = H^-1 x unchanged)
template <class P>
__global__ __launch_bounds__(TILE) void k_remap(MDArgs a, const Stage* st) {
  work_clear(a);
  const int tb = block_tile(a.ntiles, blockIdx.x);
  if (tb >= a.ntiles) return;
  const Tile t = a.tiles[tb];
  if ((int)threadIdx.x >= t.count) return;
  if (!st[t.cell].go) return;
  const double* d = st[t.cell].dR;
  const long long i = (long long)t.begin + threadIdx.x;
  const double x = a.x[i], y = a.y[i], z = a.z[i];
  const double xn = d[0] * x + d[1] * y + d[2] * z, yn = d[4] * y + d[5] * z, zn = d[8] * z;
  a.x[i] = xn; a.y[i] = yn; a.z[i] = zn;
  P::store_xyz(a.s_cur, i, fixed_pos<P>(a.cells[t.cell], xn, yn, zn));
}

// set a cell's box from H (create / set_state) and request a rebuild + prime
__global__ void k_set_box(CellDev* cells, int first, int count, double bw, unsigned long long* pack) {
  work_clear(pack);
  const int c = first + blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= first + count) return;
  CellDev& C = cells[c];
  set_box_fields(C, bw);
  for (int q = 0; q < 6; ++q) C.wsum[q] = 0.0;
  C.wcount = 0;
  C.rebuild = 1;
  C.pending = 1;
  C.prune = 1;
}

// ------------------------------------------------------------------ stress return (Eqs. 7, 8)
__global__ void k_stress_out(CellDev* cells, int ncells, double* sig, double* P, double* smd) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= ncells) return;
  CellDev& C = cells[c];
  double sv[6];
  for (int q = 0; q < 6; ++q) sv[q] = C.wcount > 0 ? C.wsum[q] / (double)C.wcount : C.last[q];
  if (smd)
    for (int q = 0; q < 6; ++q) smd[6 * c + q] = sv[q];
  const double s[9] = {sv[0], sv[3], sv[4], sv[3], sv[1], sv[5], sv[4], sv[5], sv[2]};
  double Qt[9], T[9], Sf[9];
  for (int r = 0; r < 3; ++r)
    for (int k = 0; k < 3; ++k) Qt[3 * r + k] = C.Q[3 * k + r];
  mat3mul(C.Q, s, T);
  mat3mul(T, Qt, Sf);                              // sigma_FEM = Q sigma_MD Q^T
  const int ia[6] = {0, 1, 2, 0, 0, 1}, ib[6] = {0, 1, 2, 1, 2, 2};
  bool finite = true;
  for (int q = 0; q < 6; ++q) {
    sig[6 * c + q] = Sf[3 * ia[q] + ib[q]];
    finite = finite && isfinite(Sf[3 * ia[q] + ib[q]]);
  }
  if (!finite && C.status == 0) C.status = -5;
  if (P) {
    const double* F = C.F;
    const double d = det3(F);
    // F^-T: transpose of the adjugate over det
    double FiT[9];
    FiT[0] = (F[4] * F[8] - F[5] * F[7]) / d; FiT[3] = (F[2] * F[7] - F[1] * F[8]) / d; FiT[6] = (F[1] * F[5] - F[2] * F[4]) / d;
    FiT[1] = (F[5] * F[6] - F[3] * F[8]) / d; FiT[4] = (F[0] * F[8] - F[2] * F[6]) / d; FiT[7] = (F[2] * F[3] - F[0] * F[5]) / d;
    FiT[2] = (F[3] * F[7] - F[4] * F[6]) / d; FiT[5] = (F[1] * F[6] - F[0] * F[7]) / d; FiT[8] = (F[0] * F[4] - F[1] * F[3]) / d;
    double Pm[9];
    mat3mul(Sf, FiT, Pm);                          // P = J sigma_FEM F^-T
    for (int q = 0; q < 9; ++q) P[9 * c + q] = C.J * Pm[q];
  }
  for (int q = 0; q < 6; ++q) C.wsum[q] = 0.0;
  C.wcount = 0;
}

// kinetic energy 1/2 sum m v^2 per cell (one block per cell, fixed order)
__global__ __launch_bounds__(RED_NT) void k_kinetic(MDArgs a, double* ke) {
  const CellDev& C = a.cells[blockIdx.x];
  double s = 0.0;
  for (int k = threadIdx.x; k < C.n; k += RED_NT) {
    const long long i = (long long)C.off + k;
    s += a.vx[i] * a.vx[i] + a.vy[i] * a.vy[i] + a.vz[i] * a.vz[i];
  }
  s = wave_sum(s);
  if (threadIdx.x == 0) ke[blockIdx.x] = 0.5 * a.mmv * s;
}

// Eq. (4) for a batch of deformation gradients (no cell state): Q, R, status per F
__global__ void k_qr_batch(const double* F, int n, double* Q, double* R, int* status) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n) return;
  double f[9], q[9], r[9];
  for (int k = 0; k < 9; ++k) f[k] = F[9 * c + k];
  const int st = qr_gs(f, q, r);
  for (int k = 0; k < 9; ++k) { Q[9 * c + k] = st ? 0.0 : q[k]; R[9 * c + k] = st ? 0.0 : r[k]; }
  if (status) status[c] = st;
}

// Eqs. (7), (8) for a batch: sigma_FEM = Q sigma_MD Q^T and P = J sigma_FEM F^-T, with Q and
// J = prod R_ii from the QR of each F (Voigt in and out; non-finite output for a bad F)
__global__ void k_return_batch(const double* F, const double* smd, int n, double* sfem, double* P) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n) return;
  double f[9], Q[9], R[9];
  for (int k = 0; k < 9; ++k) f[k] = F[9 * c + k];
  const int ia[6] = {0, 1, 2, 0, 0, 1}, ib[6] = {0, 1, 2, 1, 2, 2};
  if (qr_gs(f, Q, R)) {
    for (int q = 0; q < 6; ++q) sfem[6 * c + q] = __longlong_as_double(0x7ff8000000000000LL);
    if (P) for (int q = 0; q < 9; ++q) P[9 * c + q] = __longlong_as_double(0x7ff8000000000000LL);
    return;
  }
  const double* sv = smd + 6 * c;
  const double s[9] = {sv[0], sv[3], sv[4], sv[3], sv[1], sv[5], sv[4], sv[5], sv[2]};
  double Qt[9], T[9], Sf[9];
  for (int r = 0; r < 3; ++r)
    for (int k = 0; k < 3; ++k) Qt[3 * r + k] = Q[3 * k + r];
  mat3mul(Q, s, T);
  mat3mul(T, Qt, Sf);
  for (int q = 0; q < 6; ++q) sfem[6 * c + q] = Sf[3 * ia[q] + ib[q]];
  if (P) {
    const double d = det3(f);
    double FiT[9];
    FiT[0] = (f[4] * f[8] - f[5] * f[7]) / d; FiT[3] = (f[2] * f[7] - f[1] * f[8]) / d; FiT[6] = (f[1] * f[5] - f[2] * f[4]) / d;
    FiT[1] = (f[5] * f[6] - f[3] * f[8]) / d; FiT[4] = (f[0] * f[8] - f[2] * f[6]) / d; FiT[7] = (f[2] * f[3] - f[0] * f[5]) / d;
    FiT[2] = (f[3] * f[7] - f[4] * f[6]) / d; FiT[5] = (f[1] * f[6] - f[0] * f[7]) / d; FiT[8] = (f[0] * f[4] - f[1] * f[3]) / d;
    double Pm[9];
    mat3mul(Sf, FiT, Pm);
    const double J = R[0] * R[4] * R[8];
    for (int q = 0; q < 9; ++q) P[9 * c + q] = J * Pm[q];
  }
}

// a new bin width for every cell: bin counts recomputed from the box; the list stays valid and the
// next build uses the new bins
__global__ void k_set_bin_width(CellDev* cells, int ncells, double bw) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c < ncells) set_box_fields(cells[c], bw);
}

__global__ void k_set_pending(CellDev* cells, int first, int count, unsigned long long* pack) {
  work_clear(pack);
  const int c = first + blockIdx.x * blockDim.x + threadIdx.x;
  if (c < first + count) { cells[c].rebuild = 1; cells[c].pending = 1; cells[c].prune = 1; }
}

// the next force pass of every cell prunes (the pruned list's lanes per atom have changed, or it has moved)
__global__ void k_set_prune(CellDev* cells, int ncells) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c < ncells) cells[c].prune = 1;
}

}  // namespace rcell
