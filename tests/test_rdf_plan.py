"""Host arithmetic of the pair histogram kernel (csrc/rdf_plan.h), compiled
for the CPU: the flush rule of its 32-bit counters."""
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
