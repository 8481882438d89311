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

}  // namespace maze
