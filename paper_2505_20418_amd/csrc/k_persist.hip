// Resident form of the PLCG solve (Appendix B; equations "SHAKEy" and
// "linearproblem") for grids whose CG vectors fit on the chip: one launch
// runs every iteration of a solve.
//
// The N^3 grid is cut into bricks of bx by by rows of N points (whole rows in
// z), one brick per workgroup, at most one workgroup per CU. A thread owns
// one (y, z) column of its brick, bx points in x, whose x, r, p and w = A p
// stay in its registers for the whole solve: the x neighbours of a point are
// the thread's own, the y and z neighbours come from an LDS copy of p. Per
// iteration a workgroup
//   1. reads the five sums of every workgroup for the iteration before
//      (||r||^2, max |r|, <p, w>, <r, w>, <w, w>) and takes alpha, beta and
//      the stopping decision from them, as the fused sweep does;
//   2. forms x, r, p on its brick and r, p on the rows around it, which it
//      carries along (of its neighbours' rows it needs w of the iteration
//      before, nothing else), and w = A p;
//   3. sends w of its boundary rows to its neighbours, then its five sums to
//      everybody.
// The per-point arithmetic and its order are the fused sweep's (k_cg.hip),
// so are the iterates up to the rounding of the sums' order.
//
// What bounds it: on small grids the exchange. Every iteration ends in one
// all-to-all of the workgroups' sums, a store that has to reach the level shared by the
// XCDs and a load that finds it there. The launched form pays a kernel's
// start and end, the halo planes of its march and six or more dependent
// plane steps instead. At 128^3 FP64 (8.4 us an iteration) vector instructions
// take 63% of the SIMDs' issue, at 64^3 FP32 (3.6 us) about half.
//
// Exchange. All data that crosses workgroups moves through stores and loads
// with agent-scope cache policy, which bypass the caches private to an XCD,
// and is its own flag: a place that has not been written holds a bit pattern
// that the data cannot take (a signalling NaN: arithmetic returns quiet
// ones), and a reader loads until it finds something else. So nothing waits
// for a store to complete before the next is issued.
//   - Sums: one slot per workgroup, in four sets used by iteration mod 4.
//     Once the sums of k - 1 have arrived everybody has read those of k - 2;
//     a workgroup then empties its own slots of that set, which k + 2 uses.
//   - Rows: every workgroup has an inbox with a place for each point of the
//     rows around its brick, in three sets used by iteration mod 3, which its
//     neighbours write and which it empties as it reads. A set emptied in
//     iteration k is written again in k + 2 by a workgroup that has the sums
//     of k + 1.
// In both cases the emptying stores of iteration k have completed (vmcnt)
// when the workgroup passes the wait of iteration k + 1, so before it posts the
// sums of k + 1, which whoever writes or polls the place again has seen.
// A solve leaves its inboxes empty, and of the slots the set of its last sums
// full, as if the iterations went on: the next solve goes on counting from
// there (Scalars::res_iter).
//
// The workgroups of a solve wait for each other, so they have to be resident
// together: a launch never exceeds what the device holds, and launches of one
// process overlap on a device only as far as it holds them all (resident_gate.h).
// Should they be kept from running together all the same (another process's
// kernels), every wait is bounded: a workgroup that has polled `spin` times
// sets err = kErrAborted and leaves, as in turn do all others, and the host
// repeats the solve with the launched kernels; the exchange is emptied before the
// session's next resident solve.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "device_util.h"

namespace maze {

namespace {

// Brick of workgroup L: rows [x0, x0 + bx) x [y0, y0 + by), split as evenly
// as possible.
struct Brick {
  int cx, cy, x0, y0, bx, by;
};
__device__ __forceinline__ Brick brick_of(const PersistGeom& g, int L) {
  Brick b;
  b.cx = L / g.ncy;
  b.cy = L - b.cx * g.ncy;
  b.x0 = b.cx * g.N / g.ncx;
  b.y0 = b.cy * g.N / g.ncy;
  b.bx = (b.cx + 1) * g.N / g.ncx - b.x0;
  b.by = (b.cy + 1) * g.N / g.ncy - b.y0;
  return b;
}

// Buffer loads and stores addressed by a scalar resource, a scalar offset and
// a 32-bit byte offset per lane, so a point's address takes one register.
// kAgent: the cache policy of agent-scope atomics (sc1).
constexpr int kAgent = 16;
constexpr uint32_t kDrop = 0x80000000u;  // past the records of every buffer
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(void* base, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(base, 0, (int)(uint32_t)bytes, 0x00020000);
}
template <typename T, int AUX = kAgent>
__device__ __forceinline__ T ldx(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff = 0) {
  if constexpr (sizeof(T) == 4)
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, off, soff, AUX));
  else
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, off, soff, AUX));
}
template <typename T, int AUX = kAgent>
__device__ __forceinline__ void stx(__amdgpu_buffer_rsrc_t r, uint32_t off, T v, uint32_t soff = 0) {
  if constexpr (sizeof(T) == 4)
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, off, soff, AUX);
  else
    __builtin_amdgcn_raw_buffer_store_b64(
        __builtin_bit_cast(__attribute__((ext_vector_type(2))) unsigned int, v), r, off, soff, AUX);
}

// The empty pattern of an inbox place, and whether a value is it.
__device__ __forceinline__ float empty_of(float) { return __builtin_bit_cast(float, kPersistEmpty32); }
__device__ __forceinline__ double empty_of(double) { return __builtin_bit_cast(double, kPersistEmpty); }
__device__ __forceinline__ bool is_empty(float v) {
  return __builtin_bit_cast(uint32_t, v) == kPersistEmpty32;
}
__device__ __forceinline__ bool is_empty(double v) {
  return __builtin_bit_cast(unsigned long long, v) == kPersistEmpty;
}

// Whether x is kept in LDS instead of registers: 1024 threads have 128
// registers each, which do not hold eight points of four doubles.
constexpr bool x_in_lds(size_t bytes, int nt, int k) { return bytes == 8 && nt == 1024 && k >= 8; }

// Hides how v was formed, so that the addresses derived from it are formed
// where they are used instead of being kept in registers through the solve.
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// The lane that a DPP control names, per 32-bit half.
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  using I2 = int __attribute__((ext_vector_type(2)));
  I2 w = __builtin_bit_cast(I2, v);
  w.x = __builtin_amdgcn_update_dpp(0, w.x, CTRL, 0xF, 0xF, true);
  w.y = __builtin_amdgcn_update_dpp(0, w.y, CTRL, 0xF, 0xF, true);
  return __builtin_bit_cast(double, w);
}
__device__ __forceinline__ double lane_of(double v, int l) {
  using I2 = int __attribute__((ext_vector_type(2)));
  I2 w = __builtin_bit_cast(I2, v);
  w.x = __builtin_amdgcn_readlane(w.x, l);
  w.y = __builtin_amdgcn_readlane(w.y, l);
  return __builtin_bit_cast(double, w);
}
template <bool MAX>
__device__ __forceinline__ double join(double a, double b) {
  return MAX ? fmax(a, b) : a + b;
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kHalfMirror = 0x141, kMirror = 0x140;

// Sum (or max) over the wavefront, the same in every lane: lanes of a row of
// 16 by DPP, then the four rows.
template <bool MAX>
__device__ __forceinline__ double wave_join(double v) {
  v = join<MAX>(v, dpp<kXor1>(v));
  v = join<MAX>(v, dpp<kXor2>(v));
  v = join<MAX>(v, dpp<kHalfMirror>(v));
  v = join<MAX>(v, dpp<kMirror>(v));
  return join<MAX>(join<MAX>(lane_of(v, 0), lane_of(v, 16)),
                   join<MAX>(lane_of(v, 32), lane_of(v, 48)));
}

// C per-thread values (CM of them, the last ones, are maxima) over the WV
// wavefronts of the workgroup, in a fixed order. One barrier: each wavefront
// leaves its own in sm (C * WV <= 128 doubles), and reads all of them after
// it, entry i * WV + w value i of wavefront w, 64 a read; WV lanes then join
// a value. ALL: every lane gets every value, else value i is in lane
// i * WV % 64 of v[i * WV / 64].
template <int C, int CM, bool ALL, int WV>
__device__ __forceinline__ void reduce_c(double (&v)[C], double* sm) {
  static_assert((WV == 4 || WV == 8 || WV == 16) && C * WV <= kPersistRed, "lanes per value");
#pragma unroll
  for (int i = 0; i < C; ++i) v[i] = (i >= C - CM) ? wave_join<true>(v[i]) : wave_join<false>(v[i]);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (lane == 0) {
#pragma unroll
    for (int i = 0; i < C; ++i) sm[i * WV + w] = v[i];
  }
  __syncthreads();
  constexpr int R = (C * WV + 63) / 64;
  double s[R];
#pragma unroll
  for (int q = 0; q < R; ++q) {
    s[q] = sm[q * 64 + lane];
    const bool mx = q * 64 + lane >= (C - CM) * WV;
    auto step = [mx](double x, double y) { return mx ? fmax(x, y) : x + y; };
    s[q] = step(s[q], dpp<kXor1>(s[q]));
    s[q] = step(s[q], dpp<kXor2>(s[q]));
    if (WV >= 8) s[q] = step(s[q], dpp<kHalfMirror>(s[q]));
    if (WV >= 16) s[q] = step(s[q], dpp<kMirror>(s[q]));
  }
  if (ALL) {
#pragma unroll
    for (int i = 0; i < C; ++i) v[i] = lane_of(s[i * WV / 64], i * WV % 64);
  } else {
#pragma unroll
    for (int q = 0; q < R; ++q) v[q] = s[q];
  }
}

// The slots of workgroup L in a set: its values side by side in one 64-byte
// line (two for more than eight), which one store fills.
template <int C>
__device__ __forceinline__ double* slot_of(double* slots, int set, int L) {
  constexpr int W = (C + 7) / 8 * 8;
  return slots + ((size_t)(set & 3) * kPersistMaxWg + L) * W;
}

// Posts the first C of the values that reduce_c<C1, ., false, WV> left in
// the lanes of the first wavefront.
template <int C, int C1, int WV>
__device__ __forceinline__ void post_sums(double* slots, int set, int L, const double (&v)[C1]) {
  if (threadIdx.x >= 64) return;
  const int c = threadIdx.x;
  double s = __shfl(v[0], (c * WV) % 64);
#pragma unroll
  for (int h = 1; h < (C * WV + 63) / 64; ++h) {
    const double o = __shfl(v[h], (c * WV) % 64);
    s = (c * WV / 64 == h) ? o : s;
  }
  if (c < C) ctl_st(slot_of<C>(slots, set, L) + c, s);
}
template <int C>
__device__ __forceinline__ void empty_sums(double* slots, int set, int L) {
  if (threadIdx.x < C)
    ctl_st(reinterpret_cast<unsigned long long*>(slot_of<C>(slots, set, L)) + threadIdx.x,
           kPersistEmpty);
}

// Waits for the C sums of every workgroup of the solve; thread t receives
// those of workgroup t (zero past the last). False if the wait was given up.
template <int C>
__device__ __forceinline__ bool poll_sums(double* slots, int set, int nwg, unsigned spin, double* v) {
#pragma unroll
  for (int c = 0; c < C; ++c) v[c] = 0.0;
  const int t = threadIdx.x;
  if (t >= nwg) return true;
  const double* p = slot_of<C>(slots, set, t);
  for (unsigned n = 0;; ++n) {
    bool all = true;
#pragma unroll
    for (int c = 0; c < C; ++c) v[c] = ctl_ld(p + c);
#pragma unroll
    for (int c = 0; c < C; ++c) all = all && !is_empty(v[c]);
    if (all) return true;
    if (n >= spin) return false;
    __builtin_amdgcn_s_sleep(1);
  }
}

__device__ __forceinline__ float fused(float x, float y, float z) { return __builtin_fmaf(x, y, z); }
__device__ __forceinline__ double fused(double x, double y, double z) { return __builtin_fma(x, y, z); }

}  // namespace

// One workgroup (logical index L) of a resident sweep solve: NT threads, K
// points per thread in x, KY inbox places per thread of the rows around it
// in y.
template <typename T, int NT, int K, int KY>
__device__ __forceinline__ void persist_sweep_wg(const SweepArgs<T>& a, const PersistGeom& g,
                                                 int L, unsigned spin, unsigned char* smem) {
// products and sums are fused where fused() says so, as in the launched sweep
#pragma clang fp contract(off)
  constexpr int C = kPersistSweepSums, WV = NT / 64, kAhead = NT == 1024 ? 2 : 4;
  constexpr bool XL = x_in_lds(sizeof(T), NT, K);
  double* red = reinterpret_cast<double*>(smem);  // two reductions' wavefront sums
  int* lost = reinterpret_cast<int*>(red + 2 * kPersistRed);
  // x of the thread where it is kept in LDS, then p
  T* X = reinterpret_cast<T*>(red + 2 * kPersistRed + 2) + threadIdx.x;
  T* P = reinterpret_cast<T*>(red + 2 * kPersistRed + 2) + (XL ? NT * K : 0);
  Scalars* sc = a.sc;
  if (wg_flags_set(&sc->done, &sc->err, reinterpret_cast<int32_t*>(smem))) return;
  const int tid = threadIdx.x;
  const bool leader = L == 0 && tid == 0;
  const int N = g.N;
  const Brick b = brick_of(g, L);
  if (tid == 0) *lost = 0;

  // the thread's column
  const bool on = tid < b.by * N;
  const int ly = on ? tid / N : 0, z = on ? tid - ly * N : 0;
  const uint32_t place = (uint32_t)sizeof(T);
  const size_t gb = (size_t)N * N * N * sizeof(T);
  const auto gx = rsrc(a.x, gb), gr = rsrc(a.r[0], gb);
  const uint32_t plane = (uint32_t)(N * N) * place;
  const uint32_t g0 = (uint32_t)((b.x0 * N + b.y0 + ly) * N + z) * place;
  // LDS: rows -1 .. by of K planes, [lx][ly + 1][z]; a point past the brick
  // (lx >= bx) carries zeros and is nobody's neighbour
  const int es = (b.by + 2) * N;  // plane stride
  const int e0 = (ly + 1) * N + z, ezm = z == 0 ? e0 + N - 1 : e0 - 1,
            ezp = z == N - 1 ? e0 - N + 1 : e0 + 1;

  // Inbox of a workgroup: three sets of places for w: the rows below and above
  // in x (my rows each), then in y (mx rows each).
  double* slots = reinterpret_cast<double*>(a.res);
  const uint32_t fx = (uint32_t)(g.my * N) * place, fy = (uint32_t)(g.mx * N) * place;
  const uint32_t val = 2 * (fx + fy), box = 3 * val;
  const auto inbox = rsrc(static_cast<char*>(a.res) + kPersistSlotBytes, (size_t)g.nwg * box);
  const uint32_t own = (uint32_t)L * box;
  const int cxm = b.cx == 0 ? g.ncx - 1 : b.cx - 1, cxp = b.cx + 1 == g.ncx ? 0 : b.cx + 1;
  const int cym = b.cy == 0 ? g.ncy - 1 : b.cy - 1, cyp = b.cy + 1 == g.ncy ? 0 : b.cy + 1;
  // this brick's faces in its neighbours' inboxes
  const uint32_t to_xm = (uint32_t)(cxm * g.ncy + b.cy) * box + fx;
  const uint32_t to_xp = (uint32_t)(cxp * g.ncy + b.cy) * box;
  const uint32_t to_ym = (uint32_t)(b.cx * g.ncy + cym) * box + 2 * fx + fy;
  const uint32_t to_yp = (uint32_t)(b.cx * g.ncy + cyp) * box + 2 * fx;
  // The thread's own places: below and above its column in x, and KY of the
  // rows around the brick in y with their LDS index. A thread without one
  // loads zeros from, and stores nothing to, an offset past every buffer.
  const uint32_t in_lo = on ? own + (uint32_t)(ly * N + z) * place : kDrop;  // above: fx further
  uint32_t hy[KY], gy[KY];
  int ey[KY];
#pragma unroll
  for (int j = 0; j < KY; ++j) {
    const int h = tid + j * NT, m = b.bx * N;
    const int f = h >= m ? 1 : 0, q = h - f * m;
    const int lx = q / N, zz = q - lx * N;
    const bool have = h < 2 * m;
    ey[j] = have ? lx * es + (f ? b.by + 1 : 0) * N + zz : -1;
    hy[j] = have ? own + 2 * fx + (f ? fy : 0) + (uint32_t)(lx * N + zz) * place : kDrop;
    int y = f ? b.y0 + b.by : b.y0 - 1;
    y = y < 0 ? y + N : (y >= N ? y - N : y);
    gy[j] = have ? (uint32_t)(((b.x0 + lx) * N + y) * N + zz) * place : kDrop;
  }

  const T c6 = (T)(1.0 / 6.0);
  T x[XL ? 1 : K], r[K], p[K], w[K];
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const bool have = on && i < b.bx;
    r[i] = have ? ldx<T, 0>(gr, g0 + i * plane) : (T)0;
    const T xi = (have && !a.zero_x) ? ldx<T, 0>(gx, g0 + i * plane) : (T)0;
    if constexpr (XL) X[i * NT] = xi;
    else x[i] = xi;
    p[i] = w[i] = (T)0;
  }
  T rx[2], px[2], ry[KY], py[KY];  // r and p around the brick, in x and in y
  {
    const int xm = b.x0 == 0 ? N - 1 : b.x0 - 1, xp = b.x0 + b.bx == N ? 0 : b.x0 + b.bx;
    const uint32_t o = (uint32_t)((b.y0 + ly) * N + z) * place;
    rx[0] = ldx<T, 0>(gr, on ? (uint32_t)xm * plane + o : kDrop);
    rx[1] = ldx<T, 0>(gr, on ? (uint32_t)xp * plane + o : kDrop);
#pragma unroll
    for (int j = 0; j < KY; ++j) ry[j] = ldx<T, 0>(gr, gy[j]);
  }
  const double thr = ctl_ld(&sc->thr);
  const bool absmax = ctl_ld(&sc->norm) == MAZE_NORM_ABSMAX;
  const int imax = ctl_ld(&sc->max_iter);
  const int k0 = ctl_ld(&sc->res_iter);  // iterations of the solves before

  // Iteration k; FIRST: k = 0, p = r / 6. Returns whether the solve goes on;
  // code: why it stopped (-1: a wait was given up).
  int code = 0, it = 0;
  auto iterate = [&](auto first, const int k) __attribute__((always_inline)) -> bool {
    constexpr bool FIRST = decltype(first)::value;
    const int kk = k0 + k;
    // ---- sums of the kernel before (k = 0) or of iteration k - 1 ------------
    // <p, w>, <r, w>, <w, w>, ||r||^2, then the maxima: max |r|, wait given up
    double v[C + 1];
    v[C] = 0.0;
    const uint32_t set = (uint32_t)((unsigned)(kk + 2) % 3u) * val;  // inbox of k - 1
    T wx[2], wy[KY];
    if constexpr (FIRST) {
#pragma unroll
      for (int c = 0; c < C; ++c) v[c] = 0.0;
      for (int i = tid; i < a.nprev_first; i += NT) {
        v[3] += a.part[(size_t)SL_RR0 * a.pstride + i];
        v[4] = fmax(v[4], a.part[(size_t)SL_RMAX0 * a.pstride + i]);
      }
    } else {
      if (!poll_sums<C>(slots, kk - 1, g.nwg, spin, v))
        v[C] = 1.0;
      __builtin_amdgcn_s_waitcnt(0);  // places and slots emptied in k - 1 are empty
      // the rows around the brick arrive with the sums: fetch them behind those
      wx[0] = ldx<T>(inbox, in_lo, set);
      wx[1] = ldx<T>(inbox, in_lo + fx, set);
#pragma unroll
      for (int j = 0; j < KY; ++j) wy[j] = ldx<T>(inbox, hy[j], set);
    }
    reduce_c<C + 1, 2, true, WV>(v, red);
    if (v[C] != 0.0) {
      code = -1;
      return false;
    }
    if constexpr (!FIRST) {
      empty_sums<C>(slots, kk + 2, L);  // last read for k - 2, used next by k + 2
      auto settle = [&](uint32_t o, T& w_h) {
        for (unsigned n = 0; is_empty(w_h); ++n) {
          if (n >= spin) {
            *lost = 1;
            break;
          }
          w_h = ldx<T>(inbox, o, set);
        }
        stx<T>(inbox, o, empty_of(T{}), set);
      };
      settle(in_lo, wx[0]);
      settle(in_lo + fx, wx[1]);
#pragma unroll
      for (int j = 0; j < KY; ++j) settle(hy[j], wy[j]);
    }
    // alpha and beta are formed beside the stopping test, not behind it
    it = FIRST ? 0 : k - 1;
    const double mu = v[0], gam = v[3], rn = sqrt(gam);
    const double al = gam / (6.0 * mu);
    const double gnext = gam - 2.0 * al * v[1] + al * al * v[2];
    const T alpha = (T)al, beta = (T)((gnext > 0.0) ? gnext / gam : 0.0);
    const bool conv = absmax ? (v[4] <= thr) : (rn <= thr);
    if (leader && it < a.hist_cap) a.hist[it] = rn;
    if (conv || !isfinite(gam)) {
      code = conv ? 1 : 2;
      return false;
    }
    if (!FIRST && it >= imax) {
      code = 3;
      return false;
    }
    if (!FIRST && (!(mu > 0.0) || !isfinite(mu))) {
      code = 2;
      return false;
    }

    // ---- x, r, p of the brick and p around it ---------------------------------
    // The sweep's operations and roundings, each product and sum as fused there.
    auto advance = [&](T& ri, T& pi, T wi) {
      if constexpr (FIRST) {
        pi = c6 * ri;
      } else {
        ri = fused(-alpha, wi, ri);
        pi = fused(beta, pi, c6 * ri);
      }
    };
    double acc[C + 1] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    T* Pw = P + opaque(e0);
#pragma unroll
    for (int i = 0; i < K; ++i) {
      if (i > 0 && i % kAhead == 0) __builtin_amdgcn_sched_barrier(0);
      if constexpr (!FIRST) {
        if constexpr (XL) X[i * NT] = fused(alpha, p[i], X[i * NT]);
        else x[i] = fused(alpha, p[i], x[i]);
      }
      advance(r[i], p[i], w[i]);
      if (on) Pw[i * es] = p[i];
      const double rd = (double)r[i];
      acc[3] = fused(rd, rd, acc[3]);
      acc[4] = fmax(acc[4], fabs(rd));
    }
#pragma unroll
    for (int j = 0; j < KY; ++j) {
      advance(ry[j], py[j], wy[j]);
      if (ey[j] >= 0) P[ey[j]] = py[j];
    }
    advance(rx[0], px[0], wx[0]);
    advance(rx[1], px[1], wx[1]);
    __syncthreads();
    if (*lost) {
      code = -1;
      return false;
    }

    // ---- w = A p, its sums, and the rows for the neighbours --------------------
    const uint32_t out = (uint32_t)((unsigned)kk % 3u) * val;
    auto send = [&](uint32_t o, int i) { stx<T>(inbox, o, w[i], out); };
    const T *Pc = P + opaque(e0), *Pm = P + opaque(ezm), *Pp = P + opaque(ezp);
#pragma unroll
    for (int i = 0; i < K; ++i) {
      // bounds the LDS reads in flight, so the registers
      if (i > 0 && i % kAhead == 0) __builtin_amdgcn_sched_barrier(0);
      const T xm = (i == 0) ? px[0] : p[i > 0 ? i - 1 : 0];
      const T xp = (i + 1 < b.bx) ? p[i + 1 < K ? i + 1 : i] : px[1];
      const T ym = Pc[i * es - N], yp = Pc[i * es + N];
      const T zm = Pm[i * es], zp = Pp[i * es];
      const T wn = fused((T)6, p[i], -(((xm + xp) + (ym + yp)) + (zm + zp)));
      w[i] = (on && i < b.bx) ? wn : (T)0;
      const double wd = (double)w[i];
      acc[0] = fused((double)p[i], wd, acc[0]);
      acc[1] = fused((double)r[i], wd, acc[1]);
      acc[2] = fused(wd, wd, acc[2]);
    }
    if (on) {
      const uint32_t hx = in_lo - own;
      send(to_xm + hx, 0);
#pragma unroll
      for (int i = 0; i < K; ++i)
        if (i == b.bx - 1) send(to_xp + hx, i);
      const uint32_t oz = (uint32_t)opaque(z) * place;
      if (ly == 0) {
#pragma unroll
        for (int i = 0; i < K; ++i)
          if (i < b.bx) send(to_ym + oz + (uint32_t)(i * N) * place, i);
      }
      if (ly == b.by - 1) {
#pragma unroll
        for (int i = 0; i < K; ++i)
          if (i < b.bx) send(to_yp + oz + (uint32_t)(i * N) * place, i);
      }
    }
    reduce_c<C + 1, 2, false, WV>(acc, red + kPersistRed);
    post_sums<C, C + 1, WV>(slots, kk, L, acc);
    return true;
  };
  bool more = iterate(std::true_type{}, 0);
  int k = 1;
  for (; more; ++k) more = iterate(std::false_type{}, k);
  if (code < 0) {
    if (tid == 0) ctl_st(&sc->err, kErrAborted);
    return;
  }

  // ---- stopped: every workgroup has taken the same decision -------------------
  if (on) {
#pragma unroll
    for (int i = 0; i < K; ++i)
      if (i < b.bx) stx<T, 0>(gx, g0 + i * plane, XL ? X[i * NT] : x[XL ? 0 : i]);
  }
  if (leader) {
    ctl_st(&sc->iters, it);
    // the sums of iteration k - 2 were the last posted (none if k = 1)
    ctl_st(&sc->res_iter, (k0 + k - 1) % 12);
    ctl_st(&sc->done, code);
  }
}

template <typename T, int NT, int K, int KY>
__global__ __launch_bounds__(NT) void k_persist_sweep(SweepArgs<T> a, PersistGeom g,
                                                       unsigned spin) {
  extern __shared__ __align__(16) unsigned char smem[];
  persist_sweep_wg<T, NT, K, KY>(a, g, xcd_remap(blockIdx.x, g.nwg), spin, smem);
}

// Batched form: session i owns workgroups [wg_begin[i], wg_begin[i + 1]).
template <typename T, int NT, int K, int KY>
__global__ __launch_bounds__(NT) void k_persist_sweep_batch(const SweepArgs<T>* __restrict__ args,
                                                             const PersistGeom* __restrict__ geoms,
                                                             const int* __restrict__ wg_begin,
                                                             int count, unsigned spin) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int blk = blockIdx.x;
  int lo = 0, hi = count - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (wg_begin[mid] <= blk) lo = mid;
    else hi = mid - 1;
  }
  lo = __builtin_amdgcn_readfirstlane(lo);
  const SweepArgs<T> a = args[lo];
  const PersistGeom g = geoms[lo];
  persist_sweep_wg<T, NT, K, KY>(a, g, blk - wg_begin[lo], spin, smem);
}

// ---- geometry and launch ------------------------------------------------------
namespace {

struct PersistClass {
  int nt, k, ky;
};
// Threads, points per thread in x, inbox places per thread in y.
constexpr PersistClass kClasses[] = {{256, 2, 1}, {256, 4, 2}, {256, 6, 3}, {256, 8, 4},
                                     {512, 2, 1}, {512, 4, 2}, {512, 6, 3}, {512, 8, 4},
                                     {1024, 2, 1}, {1024, 4, 2}, {1024, 6, 2}, {1024, 8, 2}};
constexpr int kNumClasses = (int)(sizeof(kClasses) / sizeof(kClasses[0]));

int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Class of nt threads that holds bricks of at most bx by by rows (-1: none).
int class_of(int N, int nt, int bx, int by) {
  if (by * N > nt) return -1;
  for (int c = 0; c < kNumClasses; ++c)
    if (kClasses[c].nt == nt && kClasses[c].k >= bx && kClasses[c].ky >= ceil_div(2 * bx * N, nt))
      return c;
  return -1;
}

template <typename T, bool BATCH, int C>
const void* kernel_of() {
  constexpr int NT = kClasses[C].nt, K = kClasses[C].k, KY = kClasses[C].ky;
  if constexpr (BATCH && NT > 512) {
    return nullptr;
  } else if constexpr (BATCH) {
    return (const void*)k_persist_sweep_batch<T, NT, K, KY>;
  } else {
    return (const void*)k_persist_sweep<T, NT, K, KY>;
  }
}
template <typename T, bool BATCH, int... C>
const void* kernel_of(int c, std::integer_sequence<int, C...>) {
  const void* f = nullptr;
  ((f = (c == C) ? kernel_of<T, BATCH, C>() : f), ...);
  return f;
}
template <typename T, bool BATCH>
const void* kernel_of(int c) {
  return kernel_of<T, BATCH>(c, std::make_integer_sequence<int, kNumClasses>{});
}
const void* kernel_fn(bool fp32, bool batch, int c) {
  if (fp32) return batch ? kernel_of<float, true>(c) : kernel_of<float, false>(c);
  return batch ? kernel_of<double, true>(c) : kernel_of<double, false>(c);
}

// Dynamic LDS beyond the default limit, raised for the current device.
hipError_t allow_lds(const void* fn, size_t lds) {
  if (lds <= 65536) return hipSuccess;
  hipFuncAttributes fa{};
  if (hipFuncGetAttributes(&fa, fn) == hipSuccess && (size_t)fa.maxDynamicSharedSizeBytes >= lds)
    return hipSuccess;
  return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kPersistMaxLds);
}

}  // namespace

size_t persist_lds_bytes(const PersistGeom& g, bool fp32) {
  const PersistClass& c = kClasses[g.cls];
  const size_t es = fp32 ? 4 : 8;
  return sizeof(double) * (2 * kPersistRed + 2) + es * c.k * (g.my + 2) * (size_t)g.N +
         (x_in_lds(es, c.nt, c.k) ? es * c.nt * c.k : 0);
}

// The brick shape: the least of an iteration's cost in microseconds beyond
// the 2 us that even one workgroup takes, from timings at 20^3 to 128^3 (FP64;
// FP32 is about a tenth below): 0.14 per point of a thread and wavefront of
// a SIMD, 0.01 per workgroup whose sums everybody reads. At 64^3, for
// instance, 4 x 8 rows in 512 threads (128 workgroups) 4.5 us, 4 x 4 in 256
// (256 workgroups) 5.2, 8 x 8 in 512 (64 workgroups) 5.1. 1024 threads pay
// 0.3 more for their barriers (64^3: 2 x 16 rows 5.4, 4 x 16 5.4); a tie goes to
// the larger y face, whose rows travel through LDS anyway.
PersistGeom make_persist_geom(int N, bool fp32) {
  PersistGeom best;
  best.N = N;
  double cost = 1e30;
  for (int nt : {256, 512, 1024}) {
    for (int by = 1; by <= N && by * N <= nt; ++by)
      for (int bx = 1; bx <= 8 && bx <= N; ++bx) {
        PersistGeom g;
        g.N = N;
        g.ncx = ceil_div(N, bx);
        g.ncy = ceil_div(N, by);
        g.nwg = g.ncx * g.ncy;
        g.mx = ceil_div(N, g.ncx);
        g.my = ceil_div(N, g.ncy);
        g.cls = class_of(N, nt, g.mx, g.my);
        if (g.cls < 0 || g.nwg > kPersistMaxWg || persist_lds_bytes(g, fp32) > kPersistMaxLds)
          continue;
        g.cost_us = 2.0 + 0.14 * kClasses[g.cls].k * (nt / 256) + 0.01 * g.nwg +
                    (nt > 512 ? 0.3 : 0.0);
        if (g.cost_us <= cost) {
          cost = g.cost_us;
          best = g;
        }
      }
  }
  return best;
}

size_t persist_bytes(const PersistGeom& g, bool fp32) {
  if (g.nwg == 0) return 0;
  return kPersistSlotBytes + (size_t)g.nwg * 3 * 2 * (g.mx + g.my) * g.N * (fp32 ? 4 : 8);
}

// Empties slots and inboxes before the first solve, and before one that
// follows launched solves or one that gave up; solves that run to their end
// keep them in order.
__global__ __launch_bounds__(kThreads) void k_persist_empty(uint32_t* q, size_t n, int fp32,
                                                            Scalars* sc) {
  const size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x;
  if (i == 0) ctl_st(&sc->res_iter, 0);
  if (i < n)
    q[i] = (fp32 && i >= kPersistSlotBytes / sizeof(uint32_t))
               ? kPersistEmpty32
               : (uint32_t)(kPersistEmpty >> (32 * (i & 1)));
}
hipError_t launch_persist_empty(const DeviceState& d, const PersistGeom& g, bool fp32,
                                hipStream_t st) {
  const size_t n = persist_bytes(g, fp32) / sizeof(uint32_t);
  hipLaunchKernelGGL(k_persist_empty, dim3((unsigned)((n + kThreads - 1) / kThreads)),
                     dim3(kThreads), 0, st, reinterpret_cast<uint32_t*>(d.res), n, fp32 ? 1 : 0, d.sc);
  return hipGetLastError();
}

// Bricks of 1024 threads fill the device by themselves: they are launched one
// session at a time.
bool persist_batched(const PersistGeom& g) { return kClasses[g.cls].nt <= 512; }

int persist_resident(const PersistGeom& g, bool fp32, bool batch, int cus) {
  const void* fn = kernel_fn(fp32, batch, g.cls);
  const size_t lds = persist_lds_bytes(g, fp32);
  int per = 0;
  if (!fn || allow_lds(fn, lds) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fn, kClasses[g.cls].nt, lds) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  return per * cus;
}

// The sweep's arguments and the session's exchange scratch.
template <typename T>
SweepArgs<T> persist_args(const DeviceState& d, T* x, int nprev_first, bool zero_x) {
  SweepArgs<T> a = make_sweep_args<T>(d, x, nprev_first, 0, zero_x);
  a.res = d.res;
  return a;
}
template SweepArgs<float> persist_args<float>(const DeviceState&, float*, int, bool);
template SweepArgs<double> persist_args<double>(const DeviceState&, double*, int, bool);

hipError_t launch_persist(const DeviceState& d, const PersistGeom& g, void* x, bool fp32,
                          bool zero_x, int nprev_first, unsigned spin, hipStream_t st) {
  const void* fn = kernel_fn(fp32, false, g.cls);
  if (!fn || g.nwg < 1 || g.nwg > kPersistMaxWg || g.N != d.N || !d.res) return hipErrorInvalidValue;
  const size_t lds = persist_lds_bytes(g, fp32);
  const hipError_t e = allow_lds(fn, lds);
  if (e != hipSuccess) return e;
  PersistGeom gg = g;
  SweepArgs<float> af;
  SweepArgs<double> ad;
  void* args[3] = {nullptr, &gg, &spin};
  if (fp32) {
    af = persist_args<float>(d, (float*)x, nprev_first, zero_x);
    args[0] = &af;
  } else {
    ad = persist_args<double>(d, (double*)x, nprev_first, zero_x);
    args[0] = &ad;
  }
  return hipLaunchKernel(fn, dim3(g.nwg), dim3(kClasses[g.cls].nt), args, lds, st);
}

hipError_t launch_persist_batch(const void* args_dev, const PersistGeom* geoms, const int* wg_begin,
                                int count, int nwg, int cls, size_t lds, bool fp32, unsigned spin,
                                hipStream_t st) {
  const void* fn = kernel_fn(fp32, true, cls);
  if (cls < 0 || cls >= kNumClasses || !fn || count < 1 || nwg < 1) return hipErrorInvalidValue;
  const hipError_t e = allow_lds(fn, lds);
  if (e != hipSuccess) return e;
  void* args[5] = {(void*)&args_dev, (void*)&geoms, (void*)&wg_begin, &count, &spin};
  return hipLaunchKernel(fn, dim3(nwg), dim3(kClasses[cls].nt), args, lds, st);
}

}  // namespace maze
