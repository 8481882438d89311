// Molecular-dynamics driver kernels around the MaZe step: velocity Verlet
// for the ions (Section 2), its Langevin extension OVRVO for canonical runs
// (Results section), and the Born-Huggins-Mayer short-range term with the
// electrostatic part removed (Results section). Not part of the
// electrostatic hot path; they make a full device-resident MD step.
//
// Scratch layout (md.scratch_dev): [0, 3n) positions before the drift,
// [3n, 6n) electrostatic forces before the drift, then per-workgroup
// partials: 5 slots of `nb` doubles (unused, kinetic energy, work increment,
// unused, unused) followed by 3*nb momentum partials. The short-range
// energy partials go to the session's own buffer (DeviceState::md_epart).
#include <cmath>

#include "device_util.h"
#include "philox.h"

namespace maze {

struct MdParams {
  int n;
  int lgv;             // Langevin half steps on (gamma > 0)
  double dt, accel, cutoff, box, inv_box;
  double tab[15];
  double ou_a, ou_b2;  // v <- a v + sqrt(b2 / m) xi
  uint64_t seed;
  long long step;      // noise counter of this step
};

// The Ornstein-Uhlenbeck half step over dt/2: a = exp(-gamma dt / 2) and
// b2 = (1 - a^2) kT accel, so that sqrt(b2 / m) is the velocity spread
// [A/fs] that the half step adds for an ion of mass m [amu].
static MdParams md_params(const maze_md_state& md, double box, long long step = 0) {
  MdParams p;
  p.n = md.n_ions;
  p.dt = md.dt;
  p.accel = md.accel;
  p.cutoff = md.cutoff;
  p.box = box;
  p.inv_box = 1.0 / box;
  for (int i = 0; i < 15; ++i) p.tab[i] = md.bmh_table[i];
  p.lgv = md.gamma > 0.0 ? 1 : 0;
  p.ou_a = p.lgv ? std::exp(-md.gamma * md.dt / 2.0) : 1.0;
  p.ou_b2 = p.lgv ? (1.0 - p.ou_a * p.ou_a) * md.kT * md.accel : 0.0;
  p.seed = md.seed;
  p.step = step;
  return p;
}

static int md_blocks(int n) { return (n + kThreads - 1) / kThreads; }

__device__ __forceinline__ double bmh_v(const double* row, double r) {
  const double r2 = r * r, r6 = r2 * r2 * r2, r8 = r6 * r2;
  return row[0] * exp(row[1] * (row[2] - r)) - row[3] / r6 - row[4] / r8;
}

__device__ __forceinline__ double bmh_dvdr(const double* row, double r) {
  const double r2 = r * r, r7 = r2 * r2 * r2 * r, r9 = r7 * r2;
  return -row[0] * row[1] * exp(row[1] * (row[2] - r)) + 6.0 * row[3] / r7 + 8.0 * row[4] / r9;
}

// Short range: one wavefront per ion i (four to a workgroup). Its lanes test
// candidates j; the pairs within the cutoff queue up in LDS until there are
// 64, so the pair terms (a root, divisions and exponentials in FP64, most of
// the kernel's instructions) are formed by full wavefronts. Minimum image,
// cutoff, energy shifted to zero at the cutoff. Each pair is evaluated from
// both sides (force on i only), so no atomics are needed; the energy counts
// each pair once (j > i). The terms are added in the order of the candidates,
// one sum per component and class of candidates, so the result does not
// depend on how the pairs fell into wavefronts.
// Bound by latency on small systems (tiles -> ions -> positions): 7 us for 216
// ions in all pairs, 8 for 512 by tiles, 71 for 32768 (one thread an ion in all
// pairs 34, eight lanes an ion 42 and 78: the lanes took a pair term whenever
// one of them had a pair).
constexpr int kBmhWaves = kThreads / 64;
constexpr int kBmhClasses = 8;

struct BmhLds {
  int queue[128];
  uint8_t cls[128];
  double f[64], d[3][64], e[64];
};

struct BmhWave {
  const MdParams& p;
  const double* pos;
  const int32_t* species;
  const double* tab;  // LDS: the 15 coefficients, then the 3 energy shifts
  BmhLds& s;
  int i, si, have;    // the same in every lane
  double xi, yi, zi;
  double acc;         // lane 4 c + k: component k (3: energy) of class c

  __device__ __forceinline__ double separation(double xj, double yj, double zj, double d[3]) const {
    double dx = xi - xj, dy = yi - yj, dz = zi - zj;
    dx -= p.box * rint(dx * p.inv_box);
    dy -= p.box * rint(dy * p.inv_box);
    dz -= p.box * rint(dz * p.inv_box);
    d[0] = dx;
    d[1] = dy;
    d[2] = dz;
    return dx * dx + dy * dy + dz * dz;
  }
  // Candidate j of a class at (x, y, z), if `on`; every lane calls. Classes
  // do not decrease from lane to lane and call to call.
  __device__ __forceinline__ void test(bool on, int j, int cls, double x, double y, double z) {
    double d[3];
    const double r2 = separation(x, y, z, d);
    const bool in = on && j != i && !(r2 >= p.cutoff * p.cutoff);
    const unsigned long long m = __ballot(in);
    const int lane = threadIdx.x & 63;
    if (in) {
      const int at = have + __popcll(m & ((1ull << lane) - 1));
      s.queue[at] = j;
      s.cls[at] = (uint8_t)cls;
    }
    have += __popcll(m);
    if (have >= 64) {
      drain(64);
      have -= 64;
      const int rest = lane < have ? s.queue[64 + lane] : 0;
      const int rc = lane < have ? s.cls[64 + lane] : 0;
      __threadfence_block();
      if (lane < have) {
        s.queue[lane] = rest;
        s.cls[lane] = (uint8_t)rc;
      }
    }
  }
  // Adds the pairs with the first n of the queue.
  __device__ __forceinline__ void drain(int n) {
    const int lane = threadIdx.x & 63;
    __threadfence_block();
    const int cls = lane < n ? s.cls[lane] : kBmhClasses;
    if (lane < n) {
      const int j = s.queue[lane];
      double d[3];
      const double r = sqrt(separation(pos[3 * j], pos[3 * j + 1], pos[3 * j + 2], d));
      const int t = si + species[j];
      const double* row = tab + 5 * t;
      s.f[lane] = -bmh_dvdr(row, r) / r;
      s.d[0][lane] = d[0];
      s.d[1][lane] = d[1];
      s.d[2][lane] = d[2];
      s.e[lane] = j > i ? bmh_v(row, r) - tab[15 + t] : 0.0;
    }
    __threadfence_block();
    // the queue is in order of class: a class's pairs are one run of it
    int b = 0, en = 0;
#pragma unroll
    for (int c = 0; c < kBmhClasses; ++c) {
      const int before = __popcll(__ballot(cls < c)), upto = __popcll(__ballot(cls <= c));
      if (lane >> 2 == c) {
        b = before;
        en = upto;
      }
    }
    const int k = lane & 3;
    for (int q = b; q < en; ++q) acc = k < 3 ? fma(s.f[q], s.d[k][q], acc) : acc + s.e[q];
    __threadfence_block();
  }
  // Ends the ion: its force; its energy is lane 3's.
  __device__ __forceinline__ double finish(double* f_sr) {
    drain(have);
#pragma unroll
    for (int m = 2 * kBmhClasses; m >= 4; m >>= 1) acc += __shfl_xor(acc, m, 64);
    const int lane = threadIdx.x & 63;
    if (lane < 3) f_sr[3 * i + lane] = acc;
    return lane == 3 ? acc : 0.0;
  }
};

// The kernels that end an MD step are queued before the outcome of its solve is
// known; after an error (Scalars::err) they change nothing.

// The coefficients and the shifts into LDS; the caller waits.
__device__ __forceinline__ void bmh_table(const MdParams& p, double* tab) {
  const int t = threadIdx.x;
  if (t < 15) tab[t] = p.tab[t];
  if (t < 3) tab[15 + t] = bmh_v(p.tab + 5 * t, p.cutoff);
}

// All pairs: every j, staged through LDS for the workgroup's four ions.
__global__ __launch_bounds__(kThreads) void k_md_bmh(MdParams p, const double* __restrict__ pos,
                                                     const int32_t* __restrict__ species,
                                                     double* __restrict__ f_sr, double* part_e,
                                                     const Scalars* sc) {
  __shared__ double sx[kThreads], sy[kThreads], sz[kThreads], tab[18], red[8];
  __shared__ BmhLds lds[kBmhWaves];
  if (ctl_ld(&sc->err)) return;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int s = __builtin_amdgcn_readfirstlane(blockIdx.x * kBmhWaves + w);
  const int i = min(s, p.n - 1);
  bmh_table(p, tab);
  BmhWave b{p, pos, species, tab, lds[w], i, species[i], 0, pos[3 * i], pos[3 * i + 1],
            pos[3 * i + 2], 0.0};
  for (int base = 0; base < p.n; base += kThreads) {
    const int j = base + threadIdx.x;
    __syncthreads();
    if (j < p.n) {
      sx[threadIdx.x] = pos[3 * j];
      sy[threadIdx.x] = pos[3 * j + 1];
      sz[threadIdx.x] = pos[3 * j + 2];
    }
    __syncthreads();
    const int m = min(kThreads, p.n - base);
    if (s < p.n)
      for (int k0 = 0; k0 < m; k0 += 64) {
        const int k = min(k0 + lane, m - 1);
        b.test(k0 + lane < m, base + k, 0, sx[k], sy[k], sz[k]);
      }
  }
  const double e = s < p.n ? b.finish(f_sr) : 0.0;
  const double te = block_sum(e, red);
  if (threadIdx.x == 0) part_e[blockIdx.x] = te;
}

// Over the tiles of the MaZe binning (tiles of kTile^3 grid points, filled by
// the assignment of the step at the same positions): each ion visits the
// (2R+1)^3 tiles around its own, R tiles covering the cutoff, in eight classes
// (every eighth tile). A lane looks up a tile; the tiles' ions are listed in
// LDS, kBmhList at a time, and tested 64 at a time.
constexpr int kBmhList = 256;

struct BmhTiles {
  const int32_t* tile_start;
  const int32_t* sorted_idx;
  const int32_t* s_cell;
  int ntx;
  int R;
};

__global__ __launch_bounds__(kThreads) void k_md_bmh_tiles(MdParams p, BmhTiles t,
                                                           const double* __restrict__ pos,
                                                           const int32_t* __restrict__ species,
                                                           double* __restrict__ f_sr,
                                                           double* e_part, const Scalars* sc) {
  __shared__ double tab[18], red[8];
  __shared__ BmhLds lds[kBmhWaves];
  __shared__ int list[kBmhWaves][kBmhList];
  __shared__ uint8_t list_cls[kBmhWaves][kBmhList];
  if (ctl_ld(&sc->err)) return;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int s = __builtin_amdgcn_readfirstlane(blockIdx.x * kBmhWaves + w);
  bmh_table(p, tab);
  __syncthreads();
  double e = 0.0;
  if (s < p.n) {
    const int i = t.sorted_idx[s];
    const int tx = t.s_cell[3 * s] / kTile, ty = t.s_cell[3 * s + 1] / kTile,
              tz = t.s_cell[3 * s + 2] / kTile;
    BmhWave b{p, pos, species, tab, lds[w], i, species[i], 0, pos[3 * i], pos[3 * i + 1],
              pos[3 * i + 2], 0.0};
    int* const l = list[w];
    uint8_t* const lc = list_cls[w];
    const int W = 2 * t.R + 1, ntot = W * W * W;
    // tile c belongs to class c mod 8; class by class, the first `rem` classes
    // have per + 1 tiles
    const int per = ntot / kBmhClasses, rem = ntot % kBmhClasses;
    for (int c0 = 0; c0 < ntot; c0 += 64) {
      const int u = c0 + lane, big = rem * (per + 1);
      const int cls = u < big ? u / (per + 1) : rem + (u - big) / per;
      const int c = cls + kBmhClasses * (u < big ? u % (per + 1) : (u - big) % per);
      int first = 0, count = 0;
      if (u < ntot) {
        int ax = tx + c / (W * W) - t.R, ay = ty + (c / W) % W - t.R, az = tz + c % W - t.R;
        ax = (ax < 0) ? ax + t.ntx : (ax >= t.ntx ? ax - t.ntx : ax);
        ay = (ay < 0) ? ay + t.ntx : (ay >= t.ntx ? ay - t.ntx : ay);
        az = (az < 0) ? az + t.ntx : (az >= t.ntx ? az - t.ntx : az);
        const int ct = (ax * t.ntx + ay) * t.ntx + az;
        first = t.tile_start[ct];
        count = t.tile_start[ct + 1] - first;
      }
      // where this tile's ions begin in the list of the 64 tiles
      int at = count;
#pragma unroll
      for (int m = 1; m < 64; m <<= 1) {
        const int v = __shfl_up(at, m, 64);
        if (lane >= m) at += v;
      }
      const int total = __shfl(at, 63, 64);
      at -= count;
      for (int l0 = 0; l0 < total; l0 += kBmhList) {
        const int k1 = min(count, l0 + kBmhList - at);
        for (int k = max(0, l0 - at); k < k1; ++k) {
          l[at + k - l0] = first + k;
          lc[at + k - l0] = (uint8_t)cls;
        }
        __threadfence_block();
        const int m = min(kBmhList, total - l0);
        for (int k = 0; k < m; k += 64) {
          const int h = min(k + lane, m - 1), j = t.sorted_idx[l[h]];
          b.test(k + lane < m, j, lc[h], pos[3 * j], pos[3 * j + 1], pos[3 * j + 2]);
        }
        __threadfence_block();
      }
    }
    e = b.finish(f_sr);
  }
  const double te = block_sum(e, red);
  if (threadIdx.x == 0) e_part[blockIdx.x] = te;
}

// First half kick and drift; remembers the positions and electrostatic
// forces before the drift for the work integral.
__global__ __launch_bounds__(kThreads) void k_md_kick_drift(MdParams p, double* pos, double* vel,
                                                            const double* __restrict__ mass,
                                                            const double* __restrict__ f_es,
                                                            const double* __restrict__ f_sr,
                                                            double* x_old, double* f_old) {
  const int i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= p.n) return;
  const double c = 0.5 * p.dt * p.accel / mass[i];
  double v0[3] = {vel[3 * i], vel[3 * i + 1], vel[3 * i + 2]};
  if (p.lgv) {
    // first Ornstein-Uhlenbeck half step (OVRVO)
    double z[3];
    langevin_normals(p.seed, p.step, 0, i, z);
    const double cs = sqrt(p.ou_b2 / mass[i]);
#pragma unroll
    for (int d = 0; d < 3; ++d) v0[d] = p.ou_a * v0[d] + cs * z[d];
  }
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const int k = 3 * i + d;
    const double v = v0[d] + c * (f_es[k] + f_sr[k]);
    vel[k] = v;
    x_old[k] = pos[k];
    f_old[k] = f_es[k];
    pos[k] = pos[k] + p.dt * v;
  }
}

// Second half kick, kinetic energy, momentum and the trapezoid work of the
// electrostatic force (equation "E_nostra").
__global__ __launch_bounds__(kThreads) void k_md_kick2(MdParams p, const double* pos, double* vel,
                                                       const double* __restrict__ mass,
                                                       const double* __restrict__ f_es,
                                                       const double* __restrict__ f_sr,
                                                       const double* x_old, const double* f_old,
                                                       int do_kick, double* part, int nb,
                                                       const Scalars* sc) {
  __shared__ double red[8];
  if (ctl_ld(&sc->err)) return;
  const int i = blockIdx.x * kThreads + threadIdx.x;
  double ke = 0, w = 0, px = 0, py = 0, pz = 0;
  if (i < p.n) {
    const double m = mass[i];
    const double c = 0.5 * p.dt * p.accel / m;
    double v[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const int k = 3 * i + d;
      v[d] = vel[k];
      if (do_kick) {
        v[d] += c * (f_es[k] + f_sr[k]);
        w += 0.5 * (f_old[k] + f_es[k]) * (pos[k] - x_old[k]);
      }
    }
    if (do_kick && p.lgv) {
      // second Ornstein-Uhlenbeck half step (OVRVO)
      double z[3];
      langevin_normals(p.seed, p.step, 1, i, z);
      const double cs = sqrt(p.ou_b2 / m);
#pragma unroll
      for (int d = 0; d < 3; ++d) v[d] = p.ou_a * v[d] + cs * z[d];
    }
    if (do_kick) {
#pragma unroll
      for (int d = 0; d < 3; ++d) vel[3 * i + d] = v[d];
    }
    ke = 0.5 * m * (v[0] * v[0] + v[1] * v[1] + v[2] * v[2]) / p.accel;
    px = m * v[0];
    py = m * v[1];
    pz = m * v[2];
  }
  const double t0 = block_sum(ke, red);
  const double t1 = block_sum(w, red);
  const double t2 = block_sum(px, red);
  const double t3 = block_sum(py, red);
  const double t4 = block_sum(pz, red);
  if (threadIdx.x == 0) {
    part[1 * nb + blockIdx.x] = t0;
    part[2 * nb + blockIdx.x] = t1;
    part[5 * nb + blockIdx.x] = t2;
    part[6 * nb + blockIdx.x] = t3;
    part[7 * nb + blockIdx.x] = t4;
  }
}

__global__ __launch_bounds__(kThreads) void k_md_finish(const double* part, int nb,
                                                        const double* e_part, int ne, int prime,
                                                        double* scalars, const Scalars* sc) {
  __shared__ double red[8];
  if (ctl_ld(&sc->err)) return;
  const double e_sr = sum_partials(e_part, ne, red);
  const double ke = sum_partials(part + 1 * nb, nb, red);
  const double w = sum_partials(part + 2 * nb, nb, red);
  const double px = sum_partials(part + 5 * nb, nb, red);
  const double py = sum_partials(part + 6 * nb, nb, red);
  const double pz = sum_partials(part + 7 * nb, nb, red);
  if (threadIdx.x == 0) {
    scalars[0] = prime ? 0.0 : scalars[0] - w;
    scalars[1] = e_sr;
    scalars[2] = ke;
    scalars[3] = px;
    scalars[4] = py;
    scalars[5] = pz;
  }
}

hipError_t launch_md_kick_drift(const maze_md_state& md, long long step, hipStream_t st) {
  MdParams p = md_params(md, 1.0, step);
  const int n = md.n_ions;
  hipLaunchKernelGGL(k_md_kick_drift, dim3(md_blocks(n)), dim3(kThreads), 0, st, p, md.pos_dev,
                     md.vel_dev, md.mass_dev, (const double*)md.f_es_dev,
                     (const double*)md.f_sr_dev, md.scratch_dev, md.scratch_dev + 3 * (size_t)n);
  return hipGetLastError();
}

// Tile search radius covering the cutoff (one more tile when the last tile
// of an axis is partial); 0 when the tile block would wrap onto itself, in
// which case the all-pairs kernel runs.
static int bmh_tile_radius(const DeviceState& d, double cutoff) {
  const double edge = kTile * d.h;
  int R = (int)std::ceil(cutoff / edge);
  if (d.N % kTile != 0) R += 1;
  return (2 * R + 1 <= d.ntx) ? R : 0;
}

int md_energy_partials(int n_ions) { return (n_ions + kBmhWaves - 1) / kBmhWaves; }

hipError_t launch_md_bmh(const maze_md_state& md, const DeviceState& d, hipStream_t st) {
  MdParams p = md_params(md, d.box);
  const int R = bmh_tile_radius(d, md.cutoff);
  const dim3 grid(md_energy_partials(md.n_ions));
  if (R > 0) {
    BmhTiles t{d.tile_start, d.sorted_idx, d.s_cell, d.ntx, R};
    hipLaunchKernelGGL(k_md_bmh_tiles, grid, dim3(kThreads), 0, st, p, t,
                       (const double*)md.pos_dev, md.species_dev, md.f_sr_dev, d.md_epart,
                       (const Scalars*)d.sc);
  } else {
    hipLaunchKernelGGL(k_md_bmh, grid, dim3(kThreads), 0, st, p, (const double*)md.pos_dev,
                       md.species_dev, md.f_sr_dev, d.md_epart,
                       (const Scalars*)d.sc);
  }
  return hipGetLastError();
}

static hipError_t md_finish(const maze_md_state& md, const DeviceState& d, int do_kick,
                            long long step, hipStream_t st) {
  MdParams p = md_params(md, 1.0, step);
  const int n = md.n_ions, nb = md_blocks(n);
  double* part = md.scratch_dev + 6 * (size_t)n;
  hipLaunchKernelGGL(k_md_kick2, dim3(nb), dim3(kThreads), 0, st, p, (const double*)md.pos_dev,
                     md.vel_dev, md.mass_dev, (const double*)md.f_es_dev,
                     (const double*)md.f_sr_dev, (const double*)md.scratch_dev,
                     (const double*)(md.scratch_dev + 3 * (size_t)n), do_kick, part, nb,
                     (const Scalars*)d.sc);
  hipLaunchKernelGGL(k_md_finish, dim3(1), dim3(kThreads), 0, st, (const double*)part, nb,
                     (const double*)d.md_epart, md_energy_partials(md.n_ions),
                     do_kick ? 0 : 1, md.scalars_dev, (const Scalars*)d.sc);
  return hipGetLastError();
}

hipError_t launch_md_finish(const maze_md_state& md, const DeviceState& d, long long step,
                            hipStream_t st) {
  return md_finish(md, d, 1, step, st);
}
hipError_t launch_md_prime(const maze_md_state& md, const DeviceState& d, hipStream_t st) {
  return md_finish(md, d, 0, 0, st);
}

}  // namespace maze
