// Geometric multigrid V-cycle used as the preconditioner of the PLCG solve
// of M y = sigma_p (the multigrid of the Results section, "Performance and
// scaling": red-black Gauss-Seidel smoothing, 27-point full-weighting
// restriction, trilinear prolongation, and a conjugate-gradient solve on the
// coarsest grid).
//
// Level l has N_l = N / 2^l points per side and solves A_l x = b with
// A_l = c_l (6 I - sum of the six neighbours), c_l = 4^-l: the fine operator
// A = -M rediscretised at spacing 2^l h, in fine-grid units. One V-cycle
// maps a residual r to z = B r:
//
//   for each level going down: x = 0; red then black half-sweep (pre);
//                              residual; full-weighting restriction
//   coarsest level: CG to round-off, mean-zero projection
//   for each level going up:   trilinear prolongation of the coarse
//                              correction; black then red half-sweep (post)
//
// The post-smoother visits the colours in the reverse order of the
// pre-smoother and the restriction is 1/8 of the transpose of the
// prolongation, so B is symmetric and the outer CG stays a CG. Grids are
// N^3 with index (x*N + y)*N + z, z fastest; consecutive threads take
// consecutive z. The vector type T is double, or float for the FP32
// preconditioner of the mixed-precision path.
//
// Every pass of a level is a stencil on one grid, so the cycle is bound by
// the bytes it moves, and each half of a level is one kernel that reads its
// right-hand side once (b below; points with i + j + k even are red):
//
//  - k_mg_down. With x = 0, the red half-sweep gives b / (6 c), the black one
//    t / (6 c) with t = b + (sum of the six red b) / 6. The residual is then
//    zero on black points and the sum of the six black t over 6 on red ones,
//    so the restricted residual of a coarse point is a fixed sum of t around
//    it: 8 on the 6 faces, 3 on the 8 corners and 1 on the 24 points
//    (2, 1, 0) away, over 192. Neither x nor the residual is stored.
//  - k_mg_up. The prolongation adds P e, and the black half-sweep that
//    follows replaces every black value, so it only needs the red ones,
//    b / (6 c) + P e: the smoothed grid is a function of b and e alone.
//
// A workgroup owns R rows of y (and a piece of z on wide grids) and marches
// through planes of x. One thread holds the two points (z even, z + 1) of a
// row, one of each colour; of a plane only one colour is ever a neighbour in
// the next stage, so the LDS planes hold one value per pair. The stages of
// the cycle follow each other by one plane, on double-buffered LDS planes:
// one barrier per plane, the next plane's loads in flight across it.
// The levels of at most kTail points per side run in one workgroup, whole,
// in LDS (k_mg_tail).
//
// 256^3, FP32 cycle on an FP64 residual: level 0 takes 42 us down (142 MB, 3.4
// TB/s) and 47 up (with <r, z>; 209 MB, 4.4 TB/s), where the plain passes took
// 430 us and moved 1.5 GB; the whole cycle 148 us of an iteration's 360.
#include <algorithm>

#include "device_util.h"

namespace maze {

__device__ __forceinline__ int wrapi(int v, int N) { return v < 0 ? v + N : (v >= N ? v - N : v); }

template <typename T> struct Pair;
template <> struct Pair<float> { using type = float2; };
template <> struct Pair<double> { using type = double2; };

// c ? a : b of values: of vector members, the conditional operator would pick
// an address, and the vectors would live in memory.
template <typename T>
__device__ __forceinline__ T pick(bool c, T a, T b) {
  return c ? a : b;
}

constexpr int kMgThreads = 1024;
constexpr int kDownHalo = 5;  // rows of b beyond the R of a tile: 3 before, 2 after
constexpr int kUpHalo = 4;    // 2 before, 2 after
constexpr int kDirHalo = 2;   // 1 before, 1 after

// Tiles of one level: R rows of y (even) by W z-pairs, planes in chunks of cx
// (even). Rows of at most `wide` pairs are taken whole (periodic neighbours
// inside the row), longer ones in pieces with hz halo pairs on each side.
struct MgTile {
  int N, R, W, IW, hz, ny, nz, cx, nchunk, nwg;
};

static MgTile make_tile(int N, int R, int cx, int wide, int hz) {
  MgTile g;
  g.N = N;
  g.R = R;
  g.cx = cx;
  g.hz = N / 2 <= wide ? 0 : hz;
  g.W = g.hz ? wide : N / 2;
  g.IW = g.W + 2 * g.hz;
  g.ny = (N + g.R - 1) / g.R;
  g.nz = (N / 2 + g.W - 1) / g.W;
  g.nchunk = (N + g.cx - 1) / g.cx;
  g.nwg = g.ny * g.nz * g.nchunk;
  return g;
}

// Of a V-cycle: at most 13 rows of 68 pairs, one pair a thread, two workgroups
// a CU. The halo costs (R + 4) / R and (cx + 4) / cx of the loads, so a large
// grid takes long chunks and a small one as many workgroups as it can fill.
// Down / up of 256^3 from an FP64 residual, FP32: 40 / 43 us with 8 rows of 64
// pairs by 32 planes; 42 / 58 with whole rows by 16 planes (two pairs a
// thread), 49 / 47 with 16 whole rows (three), 54 / 57 with 16 planes. 128^3 9.2 /
// 11.1 with 8 rows by 8 planes, 12.7 / 16.8 by 16, 10.5 / 12.4 with 4 rows; 64^3
// 5.4 / 5.4 with 4 rows by 2 planes, 5.5 / 6.2 by 4.
static MgTile mg_tile(int N) {
  const int R = N >= 96 ? 8 : 4, cx = N >= 192 ? 32 : N >= 96 ? 8 : 2;
  return make_tile(N, R, cx, 64, 2);
}

// Of the direction pass: wider pieces, as it holds pairs of doubles and one
// halo row (256^3: 61 us; 63 with 8 rows, 70 with pieces of 64 pairs).
static MgTile dir_tile(int N) {
  return make_tile(N, 4, N >= 192 ? 32 : N >= 96 ? 8 : 4, 128, 1);
}

struct MgPos {
  int x0, y0, m0;  // first plane, row and z-pair of the tile
};
__device__ __forceinline__ MgPos mg_pos(const MgTile& g) {
  const int L = xcd_remap(blockIdx.x, g.nwg);
  const int t = L / g.nz;
  return {(t / g.ny) * g.cx, (t % g.ny) * g.R, (L % g.nz) * g.W};
}

// The pairs beside pair q, column im, of a plane in LDS; a halo pair at the
// edge of a piece stands for its own neighbour, which no result needs.
struct MgAdj {
  int l, r;
};
__device__ __forceinline__ MgAdj mg_adj(const MgTile& g, int q, int im) {
  return {im > 0 ? q - 1 : (g.hz ? q : q + g.IW - 1),
          im < g.IW - 1 ? q + 1 : (g.hz ? q : q - g.IW + 1)};
}

// Down half of a level: bc = restricted residual after one red and one black
// half-sweep from zero, from the level's right-hand side alone.
template <typename T, typename S>
__global__ __launch_bounds__(kMgThreads) void k_mg_down(const S* __restrict__ src,
                                                        T* __restrict__ bc, MgTile g,
                                                        const Scalars* sc) {
  using S2 = typename Pair<S>::type;
  extern __shared__ __align__(16) unsigned char mg_lds[];
  if (ctl_ld(&sc->done) != 0) return;
  const MgPos o = mg_pos(g);
  const int N = g.N, N2 = N / 2, IW = g.IW, R = g.R;
  const int tid = threadIdx.x;
  const int items = (R + kDownHalo) * IW;
  T* const lr = reinterpret_cast<T*>(mg_lds);  // red b of two planes
  T* const lt = lr + 2 * items;                // t of two planes, rows -2 .. R
  const int tn = (R + 3) * IW;

  const int q = min(tid, items - 1);
  const int ir = q / IW, im = q - ir * IW;
  const MgAdj adj = mg_adj(g, q, im);
  const int off = wrapi(o.y0 - 3 + ir, N) * N + 2 * wrapi(o.m0 - g.hz + im, N2);
  const int pr = (ir + 1) & 1;  // parity of the row: the first is y0 - 3, y0 even
  const bool in = ir >= 1 && ir <= R + 3;
  auto load = [&](int x) -> S2 {
    return *reinterpret_cast<const S2*>(src + (long long)wrapi(x, N) * N * N + off);
  };

  // the thread's coarse point (R / 2 rows of W), and its pair in t
  const int Nc = N2, c = min(tid, (R / 2) * g.W - 1);
  const int Jl = c / g.W, J = o.y0 / 2 + Jl, K = o.m0 + c - Jl * g.W;
  const int cb = (2 * Jl + 2) * IW + (c - Jl * g.W) + g.hz;
  const MgAdj ca = mg_adj(g, cb, (c - Jl * g.W) + g.hz);
  const bool cv = tid < (R / 2) * g.W && J < Nc && K < Nc;

  const int x1 = min(N, o.x0 + g.cx);
  const int I0 = o.x0 / 2, I1 = x1 / 2;
  const int p0 = 2 * I0 - 2, p1 = 2 * I1;
  T a0 = (T)0, a1 = (T)0;  // sums of coarse planes I and I + 1
  // red b of plane p - 1 beside the black point; red and black b of plane p;
  // the pair of plane p + 1
  T rp, rc, bk;
  S2 nx;
  {
    const S2 v = load(p0 - 1), w = load(p0);
    nx = load(p0 + 1);
    const bool odd = (pr + p0) & 1;
    rp = (T)pick(odd, v.x, v.y);
    rc = (T)pick(odd, w.y, w.x);
    bk = (T)pick(odd, w.x, w.y);
    lr[(p0 & 1) * items + q] = rc;
  }
  __syncthreads();

  const T s6 = (T)(1.0 / 6.0), s192 = (T)(1.0 / 192.0);
  // adds plane x of t to the coarse sums; an even plane 2 I ends coarse plane
  // I - 1 and begins I + 1
  auto gather = [&](int x) {
    const T* t = lt + (x & 1) * tn;
    const T* u = t + cb;
    const T* v = t + ca.l;
    const T* w = t + ca.r;
    if ((x & 1) == 0) {
      const T f = (u[-IW] + u[IW]) + (v[0] + u[0]);
      const T e = ((v[-2 * IW] + u[-2 * IW]) + (v[2 * IW] + u[2 * IW])) +
                  ((v[-IW] + w[-IW]) + (v[IW] + w[IW]));
      const int I = x / 2 - 1;
      if (I >= I0 && cv) bc[((long long)I * Nc + J) * Nc + K] = (a0 + f) * s192;
      a0 = a1 + ((T)8 * f + e);
      a1 = f;
    } else {
      const T d = (v[-IW] + u[-IW]) + (v[IW] + u[IW]);
      const T e = (u[-2 * IW] + u[2 * IW]) + (v[0] + w[0]);
      const T s = (T)8 * u[0] + ((T)3 * d + e);
      a0 += s;
      a1 += s;
    }
  };
  for (int p = p0; p <= p1; ++p) {
    S2 ld = nx;
    if (p < p1) ld = load(p + 2);
    const T* lc = lr + (p & 1) * items;
    T* ln = lr + ((p + 1) & 1) * items;
    T* to = lt + (p & 1) * tn;
    const bool odd = (pr + p) & 1;  // red point of this plane: z odd
    const T rn = (T)pick(odd, nx.x, nx.y);
    const T bn = (T)pick(odd, nx.y, nx.x);
    ln[q] = rn;
    if (in) {
      const T nb = ((rp + rn) + (lc[q - IW] + lc[q + IW])) + (rc + lc[odd ? adj.l : adj.r]);
      to[q - IW] = bk + nb * s6;
    }
    rp = rc;
    rc = rn;
    bk = bn;
    if (p > p0) gather(p - 1);
    nx = ld;
    __syncthreads();
  }
  gather(p1);
}

// Sum over the workgroup (at most 1024 threads), valid in thread 0.
__device__ __forceinline__ double mg_block_sum(double v, double* red) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < (int)blockDim.x / 64; ++i) s += red[i];
  return s;
}

// Up half of a level: z = the grid after the coarse correction e and one
// black and one red half-sweep, from the right-hand side and e. DOT: the
// workgroup's part of <src, z>.
template <typename T, typename S, bool DOT>
__global__ __launch_bounds__(kMgThreads) void k_mg_up(const S* __restrict__ src,
                                                      const T* __restrict__ e, T* __restrict__ z,
                                                      T inv_c, MgTile g, double* part,
                                                      const Scalars* sc) {
  using S2 = typename Pair<S>::type;
  using T2 = typename Pair<T>::type;
  extern __shared__ __align__(16) unsigned char mg_lds[];
  __shared__ double red[kMgThreads / 64];
  if (ctl_ld(&sc->done) != 0) return;
  const MgPos o = mg_pos(g);
  const int N = g.N, N2 = N / 2, Nc = N2, IW = g.IW, R = g.R;
  const int tid = threadIdx.x;
  const int items = (R + kUpHalo) * IW;
  T* const lu = reinterpret_cast<T*>(mg_lds);  // red values of two planes
  T* const lb = lu + 2 * items;                // black ones

  const int q = min(tid, items - 1);
  const int ir = q / IW, im = q - ir * IW;
  const int row = wrapi(o.y0 - 2 + ir, N), J = row >> 1;
  const int mm = o.m0 - g.hz + im, m = wrapi(mm, N2);
  const MgAdj adj = mg_adj(g, q, im);
  const int off = row * N + 2 * m;
  const bool rodd = (row & 1) != 0;
  const bool inner = ir >= 1 && ir <= R + 2;  // black values are formed
  const bool out = ir >= 2 && ir <= R + 1 && o.y0 - 2 + ir < N && im >= g.hz &&
                   im < g.hz + g.W && mm < N2 && tid < items;
  auto load = [&](int x) -> S2 {
    return *reinterpret_cast<const S2*>(src + (long long)wrapi(x, N) * N * N + off);
  };
  // The prolongation at a pair's red point, from a coarse plane I: on the
  // even plane 2 I it is ea; the odd plane 2 I + 1 takes a quarter of the eh
  // of coarse planes I and I + 1.
  const int e0 = J * Nc + m, ez = J * Nc + wrapi(m + 1, Nc);
  const int dy = rodd ? (J == Nc - 1 ? Nc - Nc * Nc : Nc) : 0;
  T ev[4];
  auto load_e = [&](int I) {
    const T* b = e + (long long)wrapi(I, Nc) * Nc * Nc;
    ev[0] = b[e0];
    ev[1] = b[ez];
    ev[2] = b[e0 + dy];
    ev[3] = b[ez + dy];
  };
  auto even_part = [&]() { return rodd ? (T)0.25 * ((ev[0] + ev[1]) + (ev[2] + ev[3])) : ev[0]; };
  auto odd_part = [&]() { return ev[0] + (rodd ? ev[2] : ev[1]); };

  const int x0 = o.x0, x1 = min(N, x0 + g.cx);
  const T s6 = (T)(1.0 / 6.0), i6 = inv_c * s6;
  T ea, eh;
  S2 cur, nxt;                        // the right-hand side of planes p, p + 1
  S rr = (S)0;                        // that of the red point of plane p - 1
  T up, uc, bq = (T)0, bp = (T)0;     // red of p - 1, p; black of p - 2, p - 1
  {
    const S2 first = load(x0 - 2);
    load_e(x0 / 2 - 1);
    cur = load(x0 - 1);
    nxt = load(x0);
    up = i6 * (T)pick(rodd, first.y, first.x) + even_part();
    eh = odd_part();
    load_e(x0 / 2);
    ea = even_part();
    const T h = odd_part();
    uc = i6 * (T)pick(rodd, cur.x, cur.y) + (T)0.25 * (eh + h);
    eh = h;
    lu[((x0 - 1) & 1) * items + q] = uc;
  }
  __syncthreads();
  double acc = 0.0;
  // one plane: p's black points, then the red points of p - 1
  for (int p = x0 - 1; p <= x1; ++p) {
    T pe = ea;  // the prolongation in plane p + 1
    if ((p & 1) == 0) {
      const T h = odd_part();
      pe = (T)0.25 * (eh + h);
      eh = h;
      ea = even_part();
    }
    S2 ld = nxt;
    if (p < x1) {
      ld = load(p + 2);
      if ((p & 1) != 0) load_e((p + 3) / 2);
    }
    const T* uu = lu + (p & 1) * items;
    T* un_ = lu + ((p + 1) & 1) * items;
    T* bb_ = lb + (p & 1) * items;
    const T* bo = lb + ((p + 1) & 1) * items;
    const bool odd = (row + p) & 1;  // the red point of plane p is z odd
    const int nb_z = odd ? adj.l : adj.r;
    const T un = i6 * (T)pick(odd, nxt.x, nxt.y) + pe;
    un_[q] = un;
    const S cr = pick(odd, cur.y, cur.x), cb = pick(odd, cur.x, cur.y);
    T bb = (T)0;
    if (inner) {
      const T nb = ((up + un) + (uu[q - IW] + uu[q + IW])) + (uc + uu[nb_z]);
      bb = ((T)cb * inv_c + nb) * s6;
      bb_[q] = bb;
    }
    if (out) {
      if (DOT && p >= x0 && p < x1) acc += (double)cb * (double)bb;
      if (p > x0) {
        // plane p - 1: its red point is z even where plane p's is odd
        const T nb = ((bq + bb) + (bo[q - IW] + bo[q + IW])) + (bp + bo[nb_z]);
        const T rv = ((T)rr * inv_c + nb) * s6;
        T2 w;
        w.x = odd ? rv : bp;
        w.y = odd ? bp : rv;
        *reinterpret_cast<T2*>(z + (long long)(p - 1) * N * N + off) = w;
        if (DOT) acc += (double)rr * (double)rv;
      }
    }
    bq = bp;
    bp = bb;
    up = uc;
    uc = un;
    rr = cr;
    cur = nxt;
    nxt = ld;
    __syncthreads();
  }
  if (DOT) {
    const double s = mg_block_sum(acc, red);
    if (tid == 0) part[blockIdx.x] = s;
  }
}

// Direction pass of the outer CG: p = z + beta p_old (beta = 0 on the first
// iteration) and the partials of <p, A p>, A p formed on the fly. Tiles as
// above with one halo row, pair and plane; FP64. Bound by HBM: 335 MB at 256^3
// and FP32 z in 62 us, 5.4 TB/s (121 with one point a thread and two arrays
// loaded for a halo of two rows in four).
template <typename ZT>
__global__ __launch_bounds__(kMgThreads) void k_mg_dir(const ZT* __restrict__ z,
                                                       const double* __restrict__ pold,
                                                       double* __restrict__ pnew, MgTile g,
                                                       double* part, const Scalars* sc) {
  using Z2 = typename Pair<ZT>::type;
  extern __shared__ __align__(16) unsigned char mg_lds[];
  __shared__ double red[kMgThreads / 64];
  if (ctl_ld(&sc->done) != 0 || ctl_ld(&sc->err) != 0) return;
  const double beta = ctl_ld(&sc->mg_beta);
  const MgPos o = mg_pos(g);
  const int N = g.N, N2 = N / 2, IW = g.IW, R = g.R;
  const int tid = threadIdx.x;
  const int items = (R + kDirHalo) * IW;
  double2* const lp = reinterpret_cast<double2*>(mg_lds);
  const int q = min(tid, items - 1);
  const int ir = q / IW, im = q - ir * IW, mm = o.m0 - g.hz + im;
  const MgAdj adj = mg_adj(g, q, im);
  const int off = wrapi(o.y0 - 1 + ir, N) * N + 2 * wrapi(mm, N2);
  const bool out = ir >= 1 && ir <= R && o.y0 - 1 + ir < N && im >= g.hz && im < g.hz + g.W &&
                   mm < N2 && tid < items;
  Z2 zl;
  double2 pl, pv, pc, pn;
  auto load = [&](int x) {
    const long long b = (long long)wrapi(x, N) * N * N;
    zl = *reinterpret_cast<const Z2*>(z + b + off);
    pl = *reinterpret_cast<const double2*>(pold + b + off);
  };
  auto form = [&]() -> double2 {
    return {pick(beta == 0.0, (double)zl.x, (double)zl.x + beta * pl.x),
            pick(beta == 0.0, (double)zl.y, (double)zl.y + beta * pl.y)};
  };
  const int x0 = o.x0, x1 = min(N, x0 + g.cx);
  load(x0 - 1);
  pv = form();
  load(x0);
  pc = form();
  lp[(x0 & 1) * items + q] = pc;
  load(x0 + 1);
  __syncthreads();
  double acc = 0.0;
  for (int x = x0; x < x1; ++x) {
    pn = form();
    if (x + 1 < x1) load(x + 2);
    const double2* l = lp + (x & 1) * items;
    double2* n = lp + ((x + 1) & 1) * items;
    n[q] = pn;
    if (out) {
      const double2 ym = l[q - IW], yp = l[q + IW];
      const double zm = l[adj.l].y, zp = l[adj.r].x;
      const double a0 = 6.0 * pc.x - (((pv.x + pn.x) + (ym.x + yp.x)) + (zm + pc.y));
      const double a1 = 6.0 * pc.y - (((pv.y + pn.y) + (ym.y + yp.y)) + (pc.x + zp));
      *reinterpret_cast<double2*>(pnew + (long long)x * N * N + off) = pc;
      acc += pc.x * a0;
      acc += pc.y * a1;
    }
    pv = pc;
    pc = pn;
    __syncthreads();
  }
  const double s = mg_block_sum(acc, red);
  if (tid == 0) part[blockIdx.x] = s;
}

// Update pass of the outer CG: x += alpha p, r -= alpha A p (A p recomputed),
// and the partials of ||r||^2 and max |r|. Tiles of the direction pass. Bound
// by HBM: 671 MB at 256^3 in 120 us, 5.6 TB/s (135 with one point a thread).
__global__ __launch_bounds__(kMgThreads) void k_mg_upd(const double* __restrict__ p,
                                                       double* __restrict__ x,
                                                       double* __restrict__ r, MgTile g,
                                                       double* part, double* part_max,
                                                       const Scalars* sc) {
  extern __shared__ __align__(16) unsigned char mg_lds[];
  __shared__ double red[kMgThreads / 64];
  if (ctl_ld(&sc->done) != 0 || ctl_ld(&sc->err) != 0) return;
  const double alpha = ctl_ld(&sc->mg_alpha);
  const MgPos o = mg_pos(g);
  const int N = g.N, N2 = N / 2, IW = g.IW, R = g.R;
  const int tid = threadIdx.x;
  const int items = (R + kDirHalo) * IW;
  double2* const lp = reinterpret_cast<double2*>(mg_lds);
  const int q = min(tid, items - 1);
  const int ir = q / IW, im = q - ir * IW, mm = o.m0 - g.hz + im;
  const MgAdj adj = mg_adj(g, q, im);
  const int off = wrapi(o.y0 - 1 + ir, N) * N + 2 * wrapi(mm, N2);
  const bool out = ir >= 1 && ir <= R && o.y0 - 1 + ir < N && im >= g.hz && im < g.hz + g.W &&
                   mm < N2 && tid < items;
  auto load = [&](int xp) -> double2 {
    return *reinterpret_cast<const double2*>(p + (long long)wrapi(xp, N) * N * N + off);
  };
  const int x0 = o.x0, x1 = min(N, x0 + g.cx);
  double2 pv = load(x0 - 1), pc = load(x0), pn = load(x0 + 1);
  lp[(x0 & 1) * items + q] = pc;
  double2 xv = *reinterpret_cast<const double2*>(x + (long long)x0 * N * N + off);
  double2 rv = *reinterpret_cast<const double2*>(r + (long long)x0 * N * N + off);
  __syncthreads();
  double acc = 0.0, mx = 0.0;
  for (int xp = x0; xp < x1; ++xp) {
    double2 ld = pn, xn = xv, rn = rv;
    if (xp + 1 < x1) {
      const long long b = (long long)(xp + 1) * N * N + off;
      ld = load(xp + 2);
      if (out) {
        xn = *reinterpret_cast<const double2*>(x + b);
        rn = *reinterpret_cast<const double2*>(r + b);
      }
    }
    const double2* l = lp + (xp & 1) * items;
    lp[((xp + 1) & 1) * items + q] = pn;
    if (out) {
      const double2 ym = l[q - IW], yp = l[q + IW];
      const double zm = l[adj.l].y, zp = l[adj.r].x;
      const double a0 = 6.0 * pc.x - (((pv.x + pn.x) + (ym.x + yp.x)) + (zm + pc.y));
      const double a1 = 6.0 * pc.y - (((pv.y + pn.y) + (ym.y + yp.y)) + (pc.x + zp));
      const long long b = (long long)xp * N * N + off;
      xv.x += alpha * pc.x;
      xv.y += alpha * pc.y;
      rv.x -= alpha * a0;
      rv.y -= alpha * a1;
      *reinterpret_cast<double2*>(x + b) = xv;
      *reinterpret_cast<double2*>(r + b) = rv;
      acc += rv.x * rv.x;
      acc += rv.y * rv.y;
      mx = fmax(mx, fmax(fabs(rv.x), fabs(rv.y)));
    }
    pv = pc;
    pc = pn;
    pn = ld;
    xv = xn;
    rv = rn;
    __syncthreads();
  }
  const double s = mg_block_sum(acc, red);
  mx = wave_max(mx);
  __syncthreads();
  if ((tid & 63) == 0) red[tid >> 6] = mx;
  __syncthreads();
  if (tid == 0) {
    for (int i = 1; i < (int)blockDim.x / 64; ++i) mx = fmax(mx, red[i]);
    part[blockIdx.x] = s;
    part_max[blockIdx.x] = mx;
  }
}

// The levels of at most kTail points per side, in one workgroup: down to the
// coarsest grid, its solve, and up again; the smaller levels' grids stay in
// LDS. src: the right-hand side of the first of them (S), xo: its solution.
constexpr int kTail = 16;
constexpr int kTailThreads = 1024;
constexpr int kTailLevels = 3;    // of at most 16 points per side: 16, 8, 4
constexpr int kCoarseMax = 1728;  // 12^3, points of the coarsest grid

struct MgTail {
  int levels;
  int N[kTailLevels];
  double c[kTailLevels];
  int b[kTailLevels], x[kTailLevels];  // LDS offsets, elements of T
};

// CG on c (6 x - sum of neighbours) = b - mean(b) to round-off (FP64), x -
// mean(x) into xs. WAVE: by the first wavefront alone, without barriers; K:
// points per thread. ps: LDS copy of the direction.
template <typename T, bool WAVE, int K>
__device__ __forceinline__ void mg_coarse(const T* b, T* xs, double* ps, double* red, int N,
                                          double c) {
  constexpr int NT = WAVE ? 64 : kTailThreads;
  const int G = N * N * N, tid = threadIdx.x;
  auto sync = [&]() {
    if (WAVE) __threadfence_block();
    else __syncthreads();
  };
  auto sum = [&](double v) -> double {
    if (WAVE) {
#pragma unroll
      for (int s = 32; s > 0; s >>= 1) v += __shfl_xor(v, s, 64);
      return v;
    }
    v = mg_block_sum(v, red);
    if (tid == 0) red[0] = v;
    __syncthreads();
    return red[0];
  };
  double x[K], r[K], p[K], w[K];
  int nb[K][6];
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int g = min(tid + k * NT, G - 1);
    const int kz = g % N, j = (g / N) % N, i = g / (N * N);
    nb[k][0] = wrapi(i - 1, N) * N * N + j * N + kz;
    nb[k][1] = wrapi(i + 1, N) * N * N + j * N + kz;
    nb[k][2] = i * N * N + wrapi(j - 1, N) * N + kz;
    nb[k][3] = i * N * N + wrapi(j + 1, N) * N + kz;
    nb[k][4] = i * N * N + j * N + wrapi(kz - 1, N);
    nb[k][5] = i * N * N + j * N + wrapi(kz + 1, N);
    x[k] = 0.0;
    r[k] = tid + k * NT < G ? (double)b[g] : 0.0;
    s += r[k];
  }
  const double mean = sum(s) / (double)G;
  double rr = 0.0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    r[k] = tid + k * NT < G ? r[k] - mean : 0.0;
    p[k] = r[k];
    rr += r[k] * r[k];
  }
  rr = sum(rr);
  const double stop = rr * 1e-28;
  for (int it = 0; it < 4 * G && rr > stop && rr > 0.0; ++it) {
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (tid + k * NT < G) ps[tid + k * NT] = p[k];
    sync();
    double pw = 0.0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const double a = ((ps[nb[k][0]] + ps[nb[k][1]]) + (ps[nb[k][2]] + ps[nb[k][3]])) +
                       (ps[nb[k][4]] + ps[nb[k][5]]);
      w[k] = tid + k * NT < G ? c * (6.0 * p[k] - a) : 0.0;
      pw += p[k] * w[k];
    }
    pw = sum(pw);
    if (!(pw > 0.0)) break;
    const double al = rr / pw;
    double rn = 0.0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      x[k] += al * p[k];
      r[k] -= al * w[k];
      rn += r[k] * r[k];
    }
    rn = sum(rn);
    const double be = rn / rr;
    rr = rn;
#pragma unroll
    for (int k = 0; k < K; ++k) p[k] = r[k] + be * p[k];
  }
  s = 0.0;
#pragma unroll
  for (int k = 0; k < K; ++k) s += x[k];  // zero beyond the grid
  const double xm = sum(s) / (double)G;
#pragma unroll
  for (int k = 0; k < K; ++k)
    if (tid + k * NT < G) xs[tid + k * NT] = (T)(x[k] - xm);
}

template <typename T, typename S, bool DOT>
__global__ __launch_bounds__(kTailThreads) void k_mg_tail(const S* __restrict__ src,
                                                          T* __restrict__ xo, MgTail m,
                                                          double* part, const Scalars* sc) {
  __shared__ double ps[kCoarseMax], red[kTailThreads / 64];
  extern __shared__ __align__(16) unsigned char mg_lds[];
  if (ctl_ld(&sc->done) != 0) return;
  T* const lds = reinterpret_cast<T*>(mg_lds);
  const int tid = threadIdx.x;
  const int G0 = m.N[0] * m.N[0] * m.N[0];
  const T s6 = (T)(1.0 / 6.0);
  for (int g = tid; g < G0; g += kTailThreads) lds[m.b[0] + g] = (T)src[g];
  __syncthreads();
  // sum of v at the six neighbours of point (i, j, k)
  auto six = [](const T* v, int N, int i, int j, int k) {
    const int a = i * N * N, b = j * N;
    return ((v[wrapi(i - 1, N) * N * N + b + k] + v[wrapi(i + 1, N) * N * N + b + k]) +
            (v[a + wrapi(j - 1, N) * N + k] + v[a + wrapi(j + 1, N) * N + k])) +
           (v[a + b + wrapi(k - 1, N)] + v[a + b + wrapi(k + 1, N)]);
  };
  // q / n for q < 2^13 and n <= 16, by a product
  auto inv = [](int n) { return (65535 + n) / n; };
  auto quo = [](int q, int v) { return (q * v) >> 16; };
  for (int l = 0; l + 1 < m.levels; ++l) {
    const int N = m.N[l], Nc = N / 2, vN = inv(N), vc = inv(Nc);
    const T* b = lds + m.b[l];
    T* t = lds + m.x[l];
    for (int q = tid; q < N * N * Nc; q += kTailThreads) {
      const int row = quo(q, vc), i = quo(row, vN), j = row - i * N, h = q - row * Nc;
      const int k = 2 * h + (((i + j) & 1) ^ 1);  // black
      t[(i * N + j) * N + k] = b[(i * N + j) * N + k] + six(b, N, i, j, k) * s6;
    }
    __syncthreads();
    T* bc = lds + m.b[l + 1];
    for (int c = tid; c < Nc * Nc * Nc; c += kTailThreads) {
      const int row = quo(c, vc), I = quo(row, vc), J = row - I * Nc, K = c - row * Nc;
      int x[5], y[5], z[5];
#pragma unroll
      for (int d = 0; d < 5; ++d) {
        x[d] = wrapi(2 * I + d - 2, N) * N * N;
        y[d] = wrapi(2 * J + d - 2, N) * N;
        z[d] = wrapi(2 * K + d - 2, N);
      }
      T s = (T)0;
#pragma unroll
      for (int a = 0; a < 5; ++a)
#pragma unroll
        for (int d = 0; d < 5; ++d)
#pragma unroll
          for (int f = 0; f < 5; ++f) {
            const int n = (a - 2) * (a - 2) + (d - 2) * (d - 2) + (f - 2) * (f - 2);
            const int wt = n == 1 ? 8 : n == 3 ? 3 : n == 5 ? 1 : 0;
            if (wt != 0) s += (T)wt * t[x[a] + y[d] + z[f]];
          }
      bc[c] = s * (T)(1.0 / 192.0);
    }
    __syncthreads();
  }
  const int lc = m.levels - 1;
  {
    const int N = m.N[lc];
    const T* b = lds + m.b[lc];
    T* x = lds + m.x[lc];
    // a grid of a few points per lane is solved by one wavefront: the sums
    // are shuffles, nothing waits for a barrier
    if (N * N * N <= 64) {
      if (tid < 64) mg_coarse<T, true, 1>(b, x, ps, red, N, m.c[lc]);
    } else if (N * N * N <= 6 * 64) {
      if (tid < 64) mg_coarse<T, true, 6>(b, x, ps, red, N, m.c[lc]);
    } else {
      mg_coarse<T, false, (kCoarseMax + kTailThreads - 1) / kTailThreads>(b, x, ps, red, N,
                                                                          m.c[lc]);
    }
    __syncthreads();
  }
  for (int l = lc - 1; l >= 0; --l) {
    const int N = m.N[l], Nc = N / 2, vN = inv(N), vc = inv(Nc);
    const T inv_c = (T)(1.0 / m.c[l]);
    const T* b = lds + m.b[l];
    const T* e = lds + m.x[l + 1];
    T* x = lds + m.x[l];
    // red: the first half-sweep's value and the prolongation, an average over
    // the coarse points on both sides along each odd axis
    for (int q = tid; q < N * N * Nc; q += kTailThreads) {
      const int row = quo(q, vc), i = quo(row, vN), j = row - i * N, h = q - row * Nc;
      const int k = 2 * h + ((i + j) & 1);
      const int i0 = (i >> 1) * Nc * Nc, i1 = wrapi((i >> 1) + (i & 1), Nc) * Nc * Nc;
      const int j0 = (j >> 1) * Nc, j1 = wrapi((j >> 1) + (j & 1), Nc) * Nc;
      const int k0 = k >> 1, k1 = wrapi((k >> 1) + (k & 1), Nc);
      const T pe = (T)0.125 * (((e[i0 + j0 + k0] + e[i0 + j0 + k1]) +
                                (e[i0 + j1 + k0] + e[i0 + j1 + k1])) +
                               ((e[i1 + j0 + k0] + e[i1 + j0 + k1]) +
                                (e[i1 + j1 + k0] + e[i1 + j1 + k1])));
      const int g = (i * N + j) * N + k;
      x[g] = b[g] * (inv_c * s6) + pe;
    }
    __syncthreads();
#pragma unroll 1
    for (int color = 1; color >= 0; --color) {
      for (int q = tid; q < N * N * Nc; q += kTailThreads) {
        const int row = quo(q, vc), i = quo(row, vN), j = row - i * N, h = q - row * Nc;
        const int k = 2 * h + (((i + j) & 1) ^ color);
        const int g = (i * N + j) * N + k;
        x[g] = (b[g] * inv_c + six(x, N, i, j, k)) * s6;
      }
      __syncthreads();
    }
  }
  double acc = 0.0;
  for (int g = tid; g < G0; g += kTailThreads) {
    const T v = lds[m.x[0] + g];
    xo[g] = v;
    if (DOT) acc += (double)src[g] * (double)v;
  }
  if (DOT) {
    const double s = mg_block_sum(acc, red);
    if (tid == 0) part[0] = s;
  }
}

// ---- launches ------------------------------------------------------------------

// Raises a kernel's dynamic LDS limit where a launch may need more than the
// default; always to the same value, so concurrent callers agree.
static hipError_t lds_limit(const void* f, size_t lds) {
  if (lds <= 32 * 1024) return hipSuccess;
  return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024);
}

// Threads of a tile of `items` pairs.
static dim3 mg_threads(int items) { return dim3((items + 63) / 64 * 64); }

template <typename T, typename S>
static hipError_t launch_down(const S* src, T* bc, int N, const Scalars* sc, hipStream_t st) {
  const MgTile g = mg_tile(N);
  const size_t lds = sizeof(T) * 2 * ((size_t)(g.R + kDownHalo) + g.R + 3) * g.IW;
  hipLaunchKernelGGL((k_mg_down<T, S>), dim3(g.nwg), mg_threads((g.R + kDownHalo) * g.IW), lds, st,
                     src, bc, g, sc);
  return hipGetLastError();
}

template <typename T, typename S, bool DOT>
static hipError_t launch_up(const S* src, const T* e, T* z, double c, int N, double* part,
                            const Scalars* sc, hipStream_t st) {
  const MgTile g = mg_tile(N);
  const size_t lds = sizeof(T) * 4 * (size_t)(g.R + kUpHalo) * g.IW;
  hipLaunchKernelGGL((k_mg_up<T, S, DOT>), dim3(g.nwg), mg_threads((g.R + kUpHalo) * g.IW), lds,
                     st, src, e, z, (T)(1.0 / c), g, part, sc);
  return hipGetLastError();
}

bool mg_dir_ok(int N) { return N % 2 == 0; }
int mg_dir_count(int N) { return dir_tile(N).nwg; }

hipError_t launch_mg_dir_pairs(const DeviceState& d, const void* z, bool fp32, const double* pold,
                               double* pnew, hipStream_t st) {
  const MgTile g = dir_tile(d.N);
  if (!mg_dir_ok(d.N) || g.nwg > d.part_stride) return hipErrorInvalidValue;
  const int items = (g.R + kDirHalo) * g.IW;
  const size_t lds = sizeof(double2) * 2 * (size_t)items;
  double* part = d.part + (size_t)SL_MU0 * d.part_stride;
  if (fp32)
    hipLaunchKernelGGL(k_mg_dir<float>, dim3(g.nwg), mg_threads(items), lds, st,
                       reinterpret_cast<const float*>(z), pold, pnew, g, part,
                       (const Scalars*)d.sc);
  else
    hipLaunchKernelGGL(k_mg_dir<double>, dim3(g.nwg), mg_threads(items), lds, st,
                       reinterpret_cast<const double*>(z), pold, pnew, g, part,
                       (const Scalars*)d.sc);
  return hipGetLastError();
}

hipError_t launch_mg_upd_pairs(const DeviceState& d, const double* p, double* x, hipStream_t st) {
  const MgTile g = dir_tile(d.N);
  if (!mg_dir_ok(d.N) || g.nwg > d.part_stride) return hipErrorInvalidValue;
  const int items = (g.R + kDirHalo) * g.IW;
  hipLaunchKernelGGL(k_mg_upd, dim3(g.nwg), mg_threads(items), sizeof(double2) * 2 * (size_t)items,
                     st, p, x, d.r, g, d.part + (size_t)SL_RR0 * d.part_stride,
                     d.part + (size_t)SL_RMAX0 * d.part_stride, (const Scalars*)d.sc);
  return hipGetLastError();
}

static int first_tail(const MgHierarchy& m) {
  int l = 0;
  while (m.N[l] > kTail && l + 1 < m.levels) ++l;
  return l;
}

template <typename T, typename S, bool DOT>
static hipError_t launch_tail(const MgHierarchy& m, int l0, const S* src, T* x, double* part,
                              const Scalars* sc, hipStream_t st) {
  MgTail t{};
  t.levels = m.levels - l0;
  if (t.levels > kTailLevels) return hipErrorInvalidValue;
  int n = 0;
  for (int l = 0; l < t.levels; ++l) {
    t.N[l] = m.N[l0 + l];
    t.c[l] = m.c[l0 + l];
    t.b[l] = n;
    t.x[l] = n + (int)m.G[l0 + l];
    n += 2 * (int)m.G[l0 + l];
  }
  const size_t lds = sizeof(T) * (size_t)n;
  const hipError_t e = lds_limit(reinterpret_cast<const void*>(k_mg_tail<T, S, DOT>), lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_mg_tail<T, S, DOT>), dim3(1), dim3(kTailThreads), lds, st, src, x, t, part,
                     sc);
  return hipGetLastError();
}

template <typename T>
static hipError_t vcycle_t(const DeviceState& d, const MgHierarchy& m, const double* r, void* z,
                           hipStream_t st) {
  T* const* X = reinterpret_cast<T* const*>(m.x);
  T* const* B = reinterpret_cast<T* const*>(m.b);
  T* const x0 = reinterpret_cast<T*>(z);
  double* part = d.part + (size_t)SL_MGRZ * d.part_stride;
  const Scalars* sc = d.sc;
  const int lt = first_tail(m);
  if (lt == 0) return launch_tail<T, double, true>(m, 0, r, x0, part, sc, st);
  if (mg_rho_count(m) > d.part_stride) return hipErrorInvalidValue;
  hipError_t e = launch_down<T, double>(r, B[1], m.N[0], sc, st);
  for (int l = 1; l < lt && e == hipSuccess; ++l)
    e = launch_down<T, T>(B[l], B[l + 1], m.N[l], sc, st);
  if (e == hipSuccess) e = launch_tail<T, T, false>(m, lt, B[lt], X[lt], nullptr, sc, st);
  for (int l = lt - 1; l > 0 && e == hipSuccess; --l)
    e = launch_up<T, T, false>(B[l], X[l + 1], X[l], m.c[l], m.N[l], nullptr, sc, st);
  if (e == hipSuccess)
    e = launch_up<T, double, true>(r, X[1], x0, m.c[0], m.N[0], part, sc, st);
  return e;
}

hipError_t launch_mg_vcycle(const DeviceState& d, const MgHierarchy& m, const double* r, void* z,
                            bool fp32, hipStream_t st) {
  return fp32 ? vcycle_t<float>(d, m, r, z, st) : vcycle_t<double>(d, m, r, z, st);
}

int mg_rho_count(const MgHierarchy& m) {
  return first_tail(m) == 0 ? 1 : mg_tile(m.N[0]).nwg;
}

int mg_partials(int N) { return std::max(mg_tile(N).nwg, dir_tile(N).nwg); }

// Levels: halve while the grid stays even and the next grid has at least 4
// points per side; the coarsest grid must fit the one-workgroup solve.
int mg_plan(int N, int* Ns, int max_levels) {
  int L = 0;
  int n = N;
  Ns[L++] = n;
  while (L < max_levels && n % 2 == 0 && n / 2 >= 4) {
    n /= 2;
    Ns[L++] = n;
  }
  if ((long long)n * n * n > kCoarseMax) return 0;
  return L;
}

}  // namespace maze
