"""Host arithmetic of the pair histogram kernel (csrc/rdf_plan.h), compiled
for the CPU: the flush rule of its 32-bit counters and the split of a block of pairs
over its wavefronts."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2505_20418_amd", "csrc")


def run_cpp(tmp_path, body):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text('#include <cstdio>\n#include <cstdlib>\n#include <vector>\n'
                   '#include "rdf_plan.h"\nusing namespace maze;\n'
                   '#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\\n", __LINE__, #x);'
                   ' std::exit(1); } } while (0)\nint main() {\n' + body + '\nreturn 0; }\n')
    subprocess.run([gxx, "-std=c++17", "-O1", "-fsanitize=undefined",
                    "-fno-sanitize-recover=all", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr


# (i ions, j ions) of the blocks: those of all pairs of few and of many ions, a
# dense cell's, ragged ones, and the largest that LDS holds
@pytest.mark.parametrize("ni,nj", [(64, 256), (64, 1024), (256, 2047), (63, 1023), (256, 2048)])
def test_no_counter_runs_over(tmp_path, ni, nj):
    """Every pair of every block in one bin: between flushes the bin's 32-bit
    counter never wraps, and a flush comes only where the next block could."""
    run_cpp(tmp_path, f"""
  const unsigned long long block = {ni}ull * {nj}ull;
  RdfTaken t;
  unsigned counter = 0;
  unsigned long long total = 0, flushed = 0, flushes = 0;
  for (long b = 0; b < 300000; ++b) {{
    if (t.flush_before({ni}, {nj})) {{
      CHECK(counter + block > 0xffffffffull);
      flushed += counter;
      counter = 0;
      ++flushes;
    }}
    counter += (unsigned)block;
    total += block;
  }}
  CHECK(flushed + counter == total);
  CHECK(flushes >= total / 0x100000000ull);
""")


def test_shares_cover_each_pair_once(tmp_path):
    """Empty blocks have no share (the last chunk of a cell's neighbours may
    add none), and every pair of the others is in exactly one."""
    run_cpp(tmp_path, """
  const int waves = 16;
  const int ns[] = {0, 1, 2, 15, 16, 17, 63, 64, 65, 100, 255, 256};
  const int js[] = {0, 1, 63, 64, 65, 127, 128, 300, 511, 512, 513, 1000, 1023, 1024, 1025,
                    2047, 2048};
  for (int ni : ns)
    for (int nj : js) {
      std::vector<int> hit((size_t)ni * nj + 1, 0);
      for (int w = 0; w < waves; ++w) {
        const RdfShare t = rdf_share(ni, nj, w, waves);
        CHECK(t.i0 >= 0 && t.i1 <= ni && t.j0 >= 0);
        for (int j0 = t.j0; j0 < nj; j0 += 64 * waves)
          for (int j = j0; j < j0 + 64 && j < nj; ++j)
            for (int i = t.i0; i < t.i1; ++i) ++hit[(size_t)i * nj + j];
      }
      for (size_t k = 0; k < (size_t)ni * nj; ++k) CHECK(hit[k] == 1);
    }
""")


def test_cells_for_even_frames_only(tmp_path):
    """Even density is never heavy, with room for a third more ions than the mean in a
    cell; all ions in one cell, or in the cells of a plane, are."""
    run_cpp(tmp_path, """
  for (int n : {16384, 17576, 32768, 100000, 3000000})
    for (int nc = 6; nc <= 16; ++nc) {
      const long long mean = n / (nc * nc * nc);
      CHECK(!rdf_cell_heavy(mean, 27 * mean, n));
      CHECK(!rdf_cell_heavy(4 * mean / 3, 27 * mean, n));
      CHECK(rdf_cell_heavy(n, n, n));
      const long long plane = n / (nc * nc);
      CHECK(rdf_cell_heavy(plane, 9 * plane, n) == (9 * 1024 > nc * nc * nc * nc));
    }
""")
