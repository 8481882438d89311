// Structural and transport observables of the Results section, and the
// Langevin noise as an entry point of its own.
//
// * maze_langevin_noise: the normal deviates one OVRVO half step draws.
// * maze_rdf_accumulate: pair-distance histograms for g_IJ(r), over cells or
//   over all pairs; each workgroup histograms in LDS (integer atomics, so
//   counts are exact and order-free) and adds its counts to the global
//   histogram.
// * maze_tcf_*: velocity autocorrelation and mean squared displacement per
//   species over a ring of time origins; one workgroup per live origin and
//   sample, reduced in a fixed order.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include "device_util.h"
#include "philox.h"
#include "rdf_plan.h"

namespace maze {

namespace {

constexpr int kRdfMaxBins = 4096;

__global__ __launch_bounds__(kThreads) void k_langevin_noise(uint64_t seed, long long step,
                                                             int half, int n, double* out) {
  const int i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= n) return;
  double z[3];
  langevin_normals(seed, step, half, i, z);
  out[3 * i] = z[0];
  out[3 * i + 1] = z[1];
  out[3 * i + 2] = z[2];
}

// Squared minimum-image distance, rounded as written: each product and sum
// on its own, no fused multiply-add (the bin of a pair is decided on it).
// The image number rint(dx / box) is taken from dx times 1 / box, which
// rounds to the same integer unless it falls within rounding of a half; only
// then is the division made. (A division per axis was most of a pair's work.)
struct RdfBox {
  double box, inv;
};
__device__ __forceinline__ double min_image_r2(double dx, double dy, double dz, const RdfBox& B) {
#pragma clang fp contract(off)
  const double tx = dx * B.inv, ty = dy * B.inv, tz = dz * B.inv;
  double qx = rint(tx), qy = rint(ty), qz = rint(tz);
  const double half = fmax(fmax(fabs(tx - qx), fabs(ty - qy)), fabs(tz - qz));
  const double most = fmax(fmax(fabs(tx), fabs(ty)), fabs(tz));
  if (!(half <= 0.499999) || !(most < 1e8)) {
    qx = rint(dx / B.box);
    qy = rint(dy / B.box);
    qz = rint(dz / B.box);
  }
  dx = dx - B.box * qx;
  dy = dy - B.box * qy;
  dz = dz - B.box * qz;
  return (dx * dx + dy * dy) + dz * dz;
}

// An ion for the pair search: its coordinates in units of 2^-32 of the box,
// whose differences wrap to the nearest image by themselves, and 4 * index +
// 2 * far + species.
struct RdfIon {
  uint32_t x, y, z;
  int n;
};
// far: not finite or over 1e6 boxes away, where 2^-32 is not resolved.
__device__ __forceinline__ uint32_t reduced(double v, double inv, bool& far) {
  const double f = v * inv;
  far = far || !(fabs(f) <= 1e6);
  return (uint32_t)((f - floor(f)) * 4294967296.0);  // saturates at 2^32 - 1
}

// LDS of a workgroup of the pair histogram: the squared edges, its counters
// (3 rows of nbins), the ions taken as i and as j, and per wavefront the
// pairs whose exact distance is still to be formed.
constexpr int kRdfThreads = 1024, kRdfWaves = kRdfThreads / 64;
constexpr int kRdfI = 256, kRdfJ = 2 * kRdfThreads, kRdfQueue = 128;
struct RdfLds {
  RdfIon *I, *J;
  double* E;
  unsigned* H;
  int *queue, *word;
  __device__ RdfLds(unsigned char* smem, int nbins) {
    I = reinterpret_cast<RdfIon*>(smem);
    J = I + kRdfI;
    E = reinterpret_cast<double*>(J + kRdfJ);
    H = reinterpret_cast<unsigned*>(E + (nbins + 1));
    queue = reinterpret_cast<int*>(H + 3 * nbins);
    word = queue + kRdfWaves * kRdfQueue;
  }
};
size_t rdf_lds_bytes(int nbins) {
  return sizeof(RdfIon) * (kRdfI + kRdfJ) + sizeof(double) * ((size_t)nbins + 1) +
         sizeof(unsigned) * 3 * (size_t)nbins +
         sizeof(int) * kRdfWaves * (kRdfQueue + 1);
}

// Counts a pair at squared distance r2 in row `row`: the bin with E[b] <= r2
// < E[b + 1]. The search starts where bins of equal width in r would have it
// (r0, per: their origin and number per length) and walks a few bins, then
// bisects; any ascending edges give the same bin.
__device__ __forceinline__ void count_pair(const RdfLds& s, int nbins, float r0, float per, double r2,
                                           int row) {
  int b = (int)((sqrtf((float)r2) - r0) * per);
  b = min(max(b, 0), nbins - 1);
  int steps = 0;
  for (; steps < 4 && s.E[b] > r2; ++steps) --b;      // E[0] <= r2
  for (; steps < 4 && !(r2 < s.E[b + 1]); ++steps) ++b;  // r2 < E[nbins]
  if (s.E[b] > r2 || !(r2 < s.E[b + 1])) {
    int lo = 0, hi = nbins;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (s.E[mid] <= r2) lo = mid;
      else hi = mid;
    }
    b = lo;
  }
  atomicAdd(&s.H[row * nbins + b], 1u);
}

// What the pair search needs besides its LDS.
struct RdfJob {
  const double* pos;
  RdfBox B;
  int nbins;
  float r0, per;
  double lo_e, hi_e;
  bool any_far;  // whether there are far ions: their pairs are all left in
  float far2;  // squared distance in 2^-32 boxes past which a pair is out of range
};

// The exact distance and bin of `n` queued pairs, one per lane.
__device__ __forceinline__ void count_queue(const RdfLds& s, const RdfJob& q, const int* queue,
                                            int n) {
  const int lane = threadIdx.x & 63;
  if (lane < n) {
    const int pair = queue[lane];
    const int a = s.I[pair & 255].n, b = s.J[pair >> 8].n;
    const double* pa = q.pos + 3 * (size_t)(a >> 2);
    const double* pb = q.pos + 3 * (size_t)(b >> 2);
    const double r2 = min_image_r2(pb[0] - pa[0], pb[1] - pa[1], pb[2] - pa[2], q.B);
    if (r2 >= q.lo_e && r2 < q.hi_e) count_pair(s, q.nbins, q.r0, q.per, r2, (a & 1) + (b & 1));
  }
}

// Pairs of the i ions [0, ni) in LDS with the j ions [0, nj), each unordered
// pair once (`flip`: where i's index is the larger, else where j's is). A
// distance of 24 bits leaves out the pairs that are surely out of range; the rest
// of a wavefront's pairs queue up until there are 64 of them, so the exact
// distances and bins are formed by full wavefronts.
__device__ __forceinline__ void count_block(const RdfLds& s, const RdfJob& q, bool flip, int ni,
                                            int nj) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int* queue = s.queue + w * kRdfQueue;
  int have = 0;
  const RdfShare t = rdf_share(ni, nj, w, kRdfWaves);
  for (int j0 = t.j0; j0 < nj; j0 += kRdfThreads) {
    const int j = j0 + lane;
    const RdfIon b = s.J[min(j, nj - 1)];
    for (int i = t.i0; i < t.i1; ++i) {
      const RdfIon a = s.I[i];
      const float dx = (float)(int)(b.x - a.x), dy = (float)(int)(b.y - a.y),
                  dz = (float)(int)(b.z - a.z);
      const float d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
      const bool once = flip ? (b.n >> 2) < (a.n >> 2) : (b.n >> 2) > (a.n >> 2);
      bool maybe = !(d2 > q.far2);
      if (q.any_far) maybe = maybe || ((a.n | b.n) & 2) != 0;
      const unsigned long long m = __ballot(j < nj && once && maybe);
      if (m == 0) continue;
      if ((m >> lane) & 1ull) queue[have + __popcll(m & ((1ull << lane) - 1ull))] = j << 8 | i;
      have += __popcll(m);
      __builtin_amdgcn_wave_barrier();
      if (have >= 64) {
        have -= 64;
        count_queue(s, q, queue + have, 64);
        __builtin_amdgcn_wave_barrier();
      }
    }
  }
  if (have > 0) count_queue(s, q, queue, have);
}

// Pair histograms. Where the largest distance counted is at most a sixth of
// the box and the ions are many, the box is cut into nc^3 cells no shorter
// than it: a workgroup takes cells in turn, gathers a cell's ions and those
// of the 27 cells around it by scanning the positions (which stay in the
// caches), and counts only pairs of these. Else, or if a position is not
// finite or more than 1e6 boxes away (its cell would be uncertain), or if the
// ions crowd into a few cells (rdf_cell_heavy: the workgroup of such a cell
// would work alone), all pairs, in blocks. The decision rests on the edges and
// the positions alone, so every workgroup takes the same one: the first scan
// counts the ions of every cell. Counts are integers: exact in any order.
// What bounds it: FP64 work. With all pairs tested in FP64 and a division per
// axis, 32768 ions to 12 of 102 A took 1.26 ms (4.3e11 pairs/s), though 0.7%
// of these pairs are in range. The 24-bit test of all pairs takes 0.54 ms; the
// cells (512 here) leave 5% of them and two scans of the positions per cell:
// 0.27 ms. At 13824 ions and 216 cells the scans cost more than they save
// (0.120 against 0.095 ms), so cells start at 16384 ions. 1728 ions: 203 us
// before, 14 now. 32768 ions in a drop of a tenth of the box: 77 ms by cells,
// 2.5 by all pairs (of 0.4 of the box 6.7 and 0.9).
constexpr int kRdfCellsMin = 6, kRdfCellsMax = 16, kRdfIonsMin = 16384, kRdfBlockJ = 64;
// Long side of a block of all pairs: many blocks for few ions, full workgroups
// for many.
__host__ __device__ inline int rdf_long(int n) { return n >= 4096 ? kRdfThreads : 256; }
// Two kernels, since together they need more than the 64 registers that let
// two workgroups of 16 wavefronts share a CU (with 91, one to a CU, all pairs
// of 32768 ions took 0.80 ms): of both launches, the one whose form the edges
// and positions ask for counts.
template <bool CELLS>
__global__ __launch_bounds__(kRdfThreads, 8) void k_rdf(const double* __restrict__ pos,
                                                  const int32_t* __restrict__ species, int n,
                                                  double box, const double* __restrict__ edges2,
                                                  int nbins, unsigned long long* hist) {
  extern __shared__ __align__(16) unsigned char smem[];
  const RdfLds s(smem, nbins);
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int b = tid; b <= nbins; b += kRdfThreads) s.E[b] = edges2[b];
  for (int b = tid; b < 3 * nbins; b += kRdfThreads) s.H[b] = 0u;
  __syncthreads();
  RdfJob q;
  q.pos = pos;
  q.B = RdfBox{box, 1.0 / box};
  q.nbins = nbins;
  q.any_far = false;
  q.lo_e = s.E[0];
  q.hi_e = s.E[nbins];
  q.r0 = sqrtf(fmaxf((float)q.lo_e, 0.f));
  q.per = (float)nbins / fmaxf(sqrtf((float)q.hi_e) - q.r0, 1e-30f);
  // reduced coordinates are off by under 1e-9 boxes, squared distances by under
  // 1e-5 of themselves plus 1e-8 boxes^2
  q.far2 = (float)((q.hi_e / (box * box) * 1.00001 + 1e-8) * 18446744073709551616.0);
  // cells per side: at least 2e-5 longer than the largest distance, which
  // covers the rounding of the coordinates that cells are taken from
  const double fc = floor(box / (sqrt(q.hi_e) * (1.0 + 2e-5)));
  const int nc =
      (n >= kRdfIonsMin && fc >= kRdfCellsMin) ? (int)fmin(fc, (double)kRdfCellsMax) : 0;
  auto flush = [&]() {
    __syncthreads();
    for (int b = tid; b < 3 * nbins; b += kRdfThreads)
      if (s.H[b] != 0u) {
        atomicAdd(&hist[b], (unsigned long long)s.H[b]);
        s.H[b] = 0u;
      }
    __syncthreads();
  };
  // Counts a block, with the counters flushed before one could run over (every
  // thread of the workgroup calls).
  RdfTaken taken;
  auto count = [&](bool flip, int ni, int nj) {
    if (taken.flush_before(ni, nj)) flush();
    count_block(s, q, flip, ni, nj);
  };
  bool far = false;
  auto ion_at = [&](int i, double x, double y, double z) {
    RdfIon a;
    bool f = false;
    a.x = reduced(x, q.B.inv, f);
    a.y = reduced(y, q.B.inv, f);
    a.z = reduced(z, q.B.inv, f);
    a.n = 4 * i + (f ? 2 : 0);
    far = far || f;
    return a;
  };
  auto ion_of = [&](int i) {
    return ion_at(i, pos[3 * (size_t)i], pos[3 * (size_t)i + 1], pos[3 * (size_t)i + 2]);
  };
  // positions of the scan's next ions, fetched while the last are looked at
  double nx = 0, ny = 0, nz = 0;
  auto fetch = [&](int base) {
    const size_t i = 3 * (size_t)min(base + tid, n - 1);
    nx = pos[i];
    ny = pos[i + 1];
    nz = pos[i + 2];
  };
  auto cell1 = [&](uint32_t u) { return (int)__umulhi(u, (uint32_t)nc); };
  // Appends to L, in scan order, those of the ions [base, base + kRdfThreads)
  // for which take(ion) holds; `have` are in it, and of the sequence only
  // [from, from + cap) is kept. Returns the new length of the sequence.
  auto append = [&](int base, int have, RdfIon* L, int from, int cap, auto take) {
    const int i = base + tid;
    if (base == 0) fetch(0);
    RdfIon a = ion_at(i, nx, ny, nz);
    if (base + kRdfThreads < n) fetch(base + kRdfThreads);
    const unsigned long long m = __ballot(i < n && take(a));
    if (lane == 0) s.word[w] = __popcll(m);
    __syncthreads();
    int before = 0, total = 0;
#pragma unroll 4
    for (int v = 0; v < kRdfWaves; ++v) {
      const int k = __builtin_amdgcn_readfirstlane(s.word[v]);
      before += (v < w) ? k : 0;
      total += k;
    }
    const int p = have + before + __popcll(m & ((1ull << lane) - 1ull)) - from;
    if (((m >> lane) & 1ull) && p >= 0 && p < cap) {
      a.n += species[i] ? 1 : 0;  // any nonzero value counts as Cl
      L[p] = a;
    }
    __syncthreads();
    return have + total;
  };
  // Ions per cell, in the place of the j ions (the first scan has none).
  static_assert(sizeof(RdfIon) * kRdfJ >= sizeof(int) * kRdfCellsMax * kRdfCellsMax * kRdfCellsMax,
                "the cells' ions are counted in the place of the j ions");
  int* const cells = reinterpret_cast<int*>(s.J);
  const int ncells = nc * nc * nc;
  auto tally = [&](const RdfIon& a) {
    atomicAdd(&cells[(cell1(a.x) * nc + cell1(a.y)) * nc + cell1(a.z)], 1);
  };
  auto no_cells = [&]() {  // after the scan that tallied: whether all pairs are taken
    __syncthreads();
    // no cell is heavy unless one would be among 27 like itself
    bool heavy = far;
    for (int c = tid; c < ncells; c += kRdfThreads)
      heavy = heavy || rdf_cell_heavy(cells[c], 27ll * cells[c], n);
    if (!__syncthreads_or(heavy ? 1 : 0)) return false;
    heavy = false;
    for (int c = tid; c < ncells; c += kRdfThreads) {
      const int x = c / (nc * nc), y = (c / nc) % nc, z = c % nc;
      int near = 0;
#pragma unroll 1
      for (int k = 0; k < 27; ++k) {
        const int a = x + k / 9 - 1, b = y + (k / 3) % 3 - 1, d = z + k % 3 - 1;
        near += cells[((a < 0 ? nc - 1 : a == nc ? 0 : a) * nc +
                       (b < 0 ? nc - 1 : b == nc ? 0 : b)) * nc +
                      (d < 0 ? nc - 1 : d == nc ? 0 : d)];
      }
      heavy = heavy || rdf_cell_heavy(cells[c], near, n);
    }
    return __syncthreads_or(far || heavy ? 1 : 0) != 0;
  };
  if (ncells > 0) {
    for (int c = tid; c < ncells; c += kRdfThreads) cells[c] = 0;
    __syncthreads();
  }
  if constexpr (CELLS) {
    bool first = true;
    for (int c = blockIdx.x; c < ncells; c += gridDim.x) {
      const int cx = c / (nc * nc), cy = (c / nc) % nc, cz = c % nc;
      for (int from = 0;; from += kRdfI) {  // the cell's ions, kRdfI at a time
        int ni = 0;
        for (int base = 0; base < n; base += kRdfThreads)
          ni = append(base, ni, s.I, from, kRdfI, [&](const RdfIon& a) {
            if (first) tally(a);
            return cell1(a.x) == cx && cell1(a.y) == cy && cell1(a.z) == cz;
          });
        // seen by every workgroup in its first scan: all pairs instead
        if (first && no_cells()) return;
        first = false;
        const int here = min(ni - from, kRdfI);
        int nj = 0;
        for (int base = 0; here > 0 && base < n; base += kRdfThreads) {
          nj = append(base, nj, s.J, 0, kRdfJ, [&](const RdfIon& a) {
            auto near = [&](uint32_t v, int cc) {
              const int d = cell1(v) - cc;
              return d == 0 || d == 1 || d == -1 || d == nc - 1 || d == 1 - nc;
            };
            return near(a.x, cx) && near(a.y, cy) && near(a.z, cz);
          });
          // fewer than kRdfThreads are left over, so the next step's fit
          if (nj >= kRdfThreads || base + kRdfThreads >= n) {
            count(false, here, nj);
            nj = 0;
            __syncthreads();
          }
        }
        if (ni - from <= kRdfI) break;
      }
    }
  } else {
    if (ncells > 0) {
      for (int i = tid; i < n; i += kRdfThreads) tally(ion_of(i));
      if (!no_cells()) return;
    }
    q.any_far = true;  // cheap beside all pairs
    const int wide = rdf_long(n);
    const long long nbi = (n + wide - 1) / wide, nbj = (n + kRdfBlockJ - 1) / kRdfBlockJ;
    for (long long b = blockIdx.x; b < nbi * nbj; b += gridDim.x) {
      // the long side (`wide` ions from i0 on) takes the place of
      // j, the short one that of i
      const int i0 = (int)(b / nbj) * wide, j0 = (int)(b % nbj) * kRdfBlockJ;
      const int ni = min(wide, n - i0), nj = min(kRdfBlockJ, n - j0);
      if (j0 + nj <= i0) continue;  // the short side's ions are all below
      __syncthreads();
      if (tid < ni) {
        s.J[tid] = ion_of(i0 + tid);
        s.J[tid].n += species[i0 + tid] ? 1 : 0;
      }
      if (tid < nj) {
        s.I[tid] = ion_of(j0 + tid);
        s.I[tid].n += species[j0 + tid] ? 1 : 0;
      }
      __syncthreads();
      count(true, nj, ni);
    }
  }
  flush();
}

// One workgroup per origin slot: the slot holds origin q (sample q*every),
// the latest origin with q mod slots == slot; lag = k - q*every. Adds the
// per-species sums of v(origin).v(k) and |r(k) - r(origin)|^2 to lag's row.
__global__ __launch_bounds__(kThreads) void k_tcf_accumulate(
    const double* __restrict__ pos, const double* __restrict__ vel,
    const double* __restrict__ opos, const double* __restrict__ ovel,
    const int32_t* __restrict__ species, int n, long long k, int every, int max_lag, int slots,
    double* sums) {
  __shared__ double red[8];
  const int s = blockIdx.x;
  const long long Q = k / every;
  if (Q < s) return;
  const long long q = Q - ((Q - s) % slots);
  const long long lag = k - q * every;
  if (lag > max_lag) return;
  const double* p0 = opos + (size_t)s * 3 * n;
  const double* v0 = ovel + (size_t)s * 3 * n;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};  // VACF Na, VACF Cl, MSD Na, MSD Cl
  for (int i = threadIdx.x; i < n; i += kThreads) {
    double vv = 0.0, rr = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      vv += v0[3 * i + d] * vel[3 * i + d];
      const double dr = pos[3 * i + d] - p0[3 * i + d];
      rr += dr * dr;
    }
    const int c = species[i] ? 1 : 0;
    acc[c] += vv;
    acc[2 + c] += rr;
  }
  const int L = max_lag + 1;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const double t = block_sum(acc[r], red);
    if (threadIdx.x == 0) sums[(size_t)r * L + lag] += t;
  }
}

__global__ __launch_bounds__(kThreads) void k_fill_zero(double* x, long long m) {
  const long long g = (long long)blockIdx.x * kThreads + threadIdx.x;
  if (g < m) x[g] = 0.0;
}

}  // namespace
}  // namespace maze

using namespace maze;

struct maze_tcf {
  int n = 0, max_lag = 0, every = 1, slots = 0, device = 0;
  long long k = 0;
  hipStream_t stream = nullptr;
  int32_t* species = nullptr;
  double* opos = nullptr;
  double* ovel = nullptr;
  double* sums = nullptr;
  std::vector<int64_t> counts;
};

#define OBS_TRY(x)                    \
  do {                                \
    if ((x) != hipSuccess) {          \
      (void)hipGetLastError();        \
      return MAZE_E_DEVICE;           \
    }                                 \
  } while (0)

extern "C" {

int maze_langevin_noise(uint64_t seed, int64_t step, int32_t half, int32_t n, double* out_dev,
                        void* stream) {
  if (n < 0 || (half != 0 && half != 1) || step < 0 || (n > 0 && !out_dev)) return MAZE_E_INVALID;
  if (n == 0) return MAZE_OK;
  hipLaunchKernelGGL(k_langevin_noise, dim3((n + kThreads - 1) / kThreads), dim3(kThreads), 0,
                     (hipStream_t)stream, seed, (long long)step, (int)half, (int)n, out_dev);
  OBS_TRY(hipGetLastError());
  return MAZE_OK;
}

int maze_rdf_accumulate(const double* pos_dev, const int32_t* species_dev, int32_t n, double box,
                        const double* edges2_dev, int32_t nbins, uint64_t* hist_dev,
                        void* stream) {
  if (n < 0 || nbins < 1 || nbins > kRdfMaxBins || !(box > 0) || !std::isfinite(box) ||
      !edges2_dev || !hist_dev || (n > 0 && (!pos_dev || !species_dev)))
    return MAZE_E_INVALID;
  if (n < 2) return MAZE_OK;
  const int wide = rdf_long(n);
  const long long blocks = (((long long)n + wide - 1) / wide) *
                           (((long long)n + kRdfBlockJ - 1) / kRdfBlockJ);
  const size_t lds = rdf_lds_bytes(nbins);
  if (lds > 64 * 1024) {
    static bool raised = false;
    if (!raised) {
      for (const void* f : {(const void*)k_rdf<true>, (const void*)k_rdf<false>})
        OBS_TRY(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    160 * 1024 - 1024));
      raised = true;
    }
  }
  const dim3 grid((unsigned)std::min(blocks, 1024LL));
  unsigned long long* hist = reinterpret_cast<unsigned long long*>(hist_dev);
  if (n >= kRdfIonsMin) {
    hipLaunchKernelGGL(k_rdf<true>, grid, dim3(kRdfThreads), lds, (hipStream_t)stream, pos_dev,
                       species_dev, (int)n, box, edges2_dev, (int)nbins, hist);
    OBS_TRY(hipGetLastError());
  }
  hipLaunchKernelGGL(k_rdf<false>, grid, dim3(kRdfThreads), lds, (hipStream_t)stream, pos_dev,
                     species_dev, (int)n, box, edges2_dev, (int)nbins, hist);
  OBS_TRY(hipGetLastError());
  return MAZE_OK;
}

int maze_tcf_create(int32_t n, const int32_t* species_dev, int32_t max_lag, int32_t origin_every,
                    void* stream, maze_tcf** out) {
  if (!out) return MAZE_E_INVALID;
  *out = nullptr;
  if (n < 1 || !species_dev || max_lag < 0 || origin_every < 1) return MAZE_E_INVALID;
  maze_tcf* t = new (std::nothrow) maze_tcf;
  if (!t) return MAZE_E_OOM;
  t->n = n;
  t->max_lag = max_lag;
  t->every = origin_every;
  t->slots = max_lag / origin_every + 1;
  t->stream = (hipStream_t)stream;
  t->counts.assign((size_t)max_lag + 1, 0);
  if (hipGetDevice(&t->device) != hipSuccess) {
    (void)hipGetLastError();
    delete t;
    return MAZE_E_DEVICE;
  }
  const size_t per = sizeof(double) * 3 * (size_t)n * (size_t)t->slots;
  const size_t nsum = 4 * ((size_t)max_lag + 1);
  if (hipMalloc(&t->species, sizeof(int32_t) * (size_t)n) != hipSuccess ||
      hipMalloc(&t->opos, per) != hipSuccess || hipMalloc(&t->ovel, per) != hipSuccess ||
      hipMalloc(&t->sums, sizeof(double) * nsum) != hipSuccess) {
    (void)hipGetLastError();
    maze_tcf_destroy(t);
    return MAZE_E_OOM;
  }
  if (hipMemcpyAsync(t->species, species_dev, sizeof(int32_t) * (size_t)n,
                     hipMemcpyDeviceToDevice, t->stream) != hipSuccess) {
    (void)hipGetLastError();
    maze_tcf_destroy(t);
    return MAZE_E_DEVICE;
  }
  hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)((nsum + kThreads - 1) / kThreads)),
                     dim3(kThreads), 0, t->stream, t->sums, (long long)nsum);
  if (hipGetLastError() != hipSuccess) {
    maze_tcf_destroy(t);
    return MAZE_E_DEVICE;
  }
  *out = t;
  return MAZE_OK;
}

int maze_tcf_sample(maze_tcf* t, const double* pos_dev, const double* vel_dev) {
  if (!t || !pos_dev || !vel_dev) return MAZE_E_INVALID;
  OBS_TRY(hipSetDevice(t->device));
  const long long k = t->k;
  const size_t bytes = sizeof(double) * 3 * (size_t)t->n;
  if (k % t->every == 0) {
    const long long slot = (k / t->every) % t->slots;
    OBS_TRY(hipMemcpyAsync(t->opos + (size_t)slot * 3 * t->n, pos_dev, bytes,
                           hipMemcpyDeviceToDevice, t->stream));
    OBS_TRY(hipMemcpyAsync(t->ovel + (size_t)slot * 3 * t->n, vel_dev, bytes,
                           hipMemcpyDeviceToDevice, t->stream));
  }
  hipLaunchKernelGGL(k_tcf_accumulate, dim3(t->slots), dim3(kThreads), 0, t->stream, pos_dev,
                     vel_dev, (const double*)t->opos, (const double*)t->ovel,
                     (const int32_t*)t->species, t->n, k, t->every, t->max_lag, t->slots, t->sums);
  OBS_TRY(hipGetLastError());
  // the same live-origin rule on the host, for the counts
  const long long Q = k / t->every;
  for (long long s = 0; s < t->slots && s <= Q; ++s) {
    const long long q = Q - ((Q - s) % t->slots);
    const long long lag = k - q * t->every;
    if (lag <= t->max_lag) t->counts[(size_t)lag] += 1;
  }
  t->k = k + 1;
  return MAZE_OK;
}

int maze_tcf_read(const maze_tcf* t, double* sums_host, int64_t* counts_host) {
  if (!t) return MAZE_E_INVALID;
  OBS_TRY(hipSetDevice(t->device));
  const size_t L = (size_t)t->max_lag + 1;
  if (sums_host) {
    OBS_TRY(hipMemcpyAsync(sums_host, t->sums, sizeof(double) * 4 * L, hipMemcpyDeviceToHost,
                           t->stream));
  }
  OBS_TRY(hipStreamSynchronize(t->stream));
  if (counts_host) std::memcpy(counts_host, t->counts.data(), sizeof(int64_t) * L);
  return MAZE_OK;
}

void maze_tcf_destroy(maze_tcf* t) {
  if (!t) return;
  (void)hipSetDevice(t->device);
  if (t->stream) (void)hipStreamSynchronize(t->stream);
  else (void)hipDeviceSynchronize();
  if (t->species) (void)hipFree(t->species);
  if (t->opos) (void)hipFree(t->opos);
  if (t->ovel) (void)hipFree(t->ovel);
  if (t->sums) (void)hipFree(t->sums);
  delete t;
}

}  // extern "C"
