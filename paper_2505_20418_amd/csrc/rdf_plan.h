// How a workgroup of the pair histogram divides its pairs and when its 32-bit
// counters go to the global ones. Plain arithmetic, for the kernel and for
// tests on the host.
#pragma once

#if defined(__HIPCC__)
#define RDF_FN __host__ __device__ inline
#else
#define RDF_FN inline
#endif

namespace maze {

// Bound on the pairs that a workgroup has counted since it last added its LDS
// counters to the histogram: no counter can hold more than that, whatever bin
// the pairs fell into.
struct RdfTaken {
  unsigned long long pairs = 0;
  // Takes up to ni * nj more. True: the counters have to be flushed first.
  RDF_FN bool flush_before(int ni, int nj) {
    const unsigned long long more = (unsigned long long)ni * (unsigned long long)nj;
    const bool full = pairs + more > 0xffffffffull;
    pairs = full ? more : pairs + more;
    return full;
  }
};

// Share of wavefront w in a block of ni by nj pairs: 64 j ions at a time,
// from j0 on in steps of 64 * waves, with the i ions [i0, i1) each. Where the
// j ions are fewer than 64 a wavefront, each takes a share of the i ions; a
// wavefront without a share, and every one of an empty block, has j0 = nj.
struct RdfShare {
  int j0, i0, i1;
};
RDF_FN RdfShare rdf_share(int ni, int nj, int w, int waves) {
  if (ni <= 0 || nj <= 0) return {nj, 0, 0};
  const int jw = (nj + 63) / 64, split = waves / jw > 1 ? waves / jw : 1;
  if (w >= jw * split) return {nj, 0, 0};
  return {(w % jw) * 64, ni * (w / jw) / split, ni * (w / jw + 1) / split};
}

// Whether a cell of `here` ions with `near` ions in it and around it makes the
// cell form slower than all pairs. A cell is one workgroup's; with all pairs
// a workgroup (of the 512 that are resident) has n^2 / 1024 to test. Cells of
// even density on the coarsest division, six a side, have 0.6 of that.
RDF_FN bool rdf_cell_heavy(long long here, long long near, int n) {
  return (unsigned long long)here * (unsigned long long)near >
         (unsigned long long)n * (unsigned long long)n / 1024;
}

}  // namespace maze
