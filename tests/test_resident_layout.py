"""Shapes and workspaces of the resident recurrence, on the CPU: the header that
the launches and the buffers' sizes are computed from, compiled as it is and
walked over every chain that takes this path (L <= 20)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_10191_amd", "csrc")

PRELUDE = """
#include <cstdio>
#include <set>
#include "res_shape.hpp"
using namespace polfed;
static std::set<int64_t> sizes() {  // D of the chains up to L = 20
  std::set<int64_t> s;
  for (int L = 2; L <= kResMaxL; ++L) {
    int64_t d = 1;
    for (int n = 0; n <= L; ++n) {
      s.insert(d);
      d = d * (L - n) / (n + 1);
    }
  }
  return s;
}
"""


def run_host(tmp_path, main):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PRELUDE + main)
    cxx = shutil.which("g++") or "g++"
    subprocess.run([cxx, "-std=c++17", "-O1", f"-I{CSRC}", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    return r.stdout


@pytest.mark.parametrize("M", [4, 100, 2048])
def test_groups_of_kpm_vectors_fit_one_workspace(tmp_path, M):
    """A group of nb <= width vectors: its arrays lie one behind the other
    inside what the full width's group asked for, and it has the slabs (and so
    the tables) of that group."""
    out = run_host(tmp_path, """
int main() {
  const int M = %d;
  long n = 0;
  for (int64_t D : sizes())
    for (int width = 1; width <= 64; ++width) {
      const ResMomentsPlan full = res_moments_plan(D, M, width, width);
      for (int nb = 1; nb <= width; ++nb) {
        const ResMomentsPlan p = res_moments_plan(D, M, width, nb);
        ++n;
        bool ok = p.shape.nslab == full.shape.nslab;
        if (ok && p.shape.nslab) {
          const size_t sums = (size_t)M * nb * 8;  // and the error word
          ok = p.shape.ngrp + p.shape.pairs == nb && p.sc >= sizeof(ResState) &&
               p.sums >= p.sc + 16 * (size_t)nb && p.part >= p.sums + sums + 8 &&
               p.part + (size_t)std::min(M, kResMomentSteps) * nb * 8 * p.shape.nslab *
                            kResWaves <= full.bytes;
        }
        if (!ok) {
          std::printf("D = %%ld, %%d of %%d columns\\n", (long)D, nb, width);
          return 1;
        }
      }
    }
  std::printf("%%ld\\n", n);
}
""" % M)
    assert int(out) > 50000


def test_tail_behind_the_first_buffer_fits(tmp_path):
    """The team state, the scale and a full chunk's coefficients end inside the
    buffer wherever the D elements end (FP64 and FP32, D of every chain and of
    the quantum suns), and do not overlap."""
    run_host(tmp_path, """
int main() {
  std::set<int64_t> ds = sizes();
  for (int64_t d = 1; d <= 300; ++d) ds.insert(d);
  for (int b = 2; b <= 18; ++b) ds.insert(int64_t(1) << b);
  static_assert(ResTail::sc >= ResTail::st + sizeof(ResState), "state");
  static_assert(ResTail::A >= ResTail::sc + 2 * sizeof(double), "scale");
  for (int64_t D : ds)
    for (size_t elem : {size_t(4), size_t(8)}) {
      const size_t at = res_align((size_t)D * elem);
      const size_t end = at + ResTail::A + (size_t)(kResChunk + 1) * elem;
      if (end > (size_t)D * elem + ResTail::bytes) {
        std::printf("D = %ld, %zu bytes an element\\n", (long)D, elem);
        return 1;
      }
    }
}
""")


def test_a_given_up_barrier_is_not_cleared_between_launches(tmp_path):
    """Before a call's first launch the whole team state is cleared, before
    the ones that go on with its recurrence everything but err."""
    run_host(tmp_path, """
int main() {
  ResState st;
  int* p = reinterpret_cast<int*>(&st);
  for (bool first : {true, false}) {
    for (size_t i = 0; i < sizeof st / 4; ++i) p[i] = 7;
    for (size_t i = 0; i < sizeof st / 4; ++i)
      if (res_clears(i, first)) p[i] = 0;
    for (size_t i = 0; i < sizeof st / 4; ++i)
      if (p[i] != (&p[i] == &st.err && !first ? 7 : 0)) return 1;
  }
}
""")


def test_one_column_takes_one_workgroup_up_to_1024_rows(tmp_path):
    """Two rows a thread of one workgroup measured faster than two slabs with
    a barrier between them; above that, slabs of one row a thread."""
    run_host(tmp_path, """
int main() {
  for (int64_t D = 1; D <= 16384; ++D) {
    const ResShape x = res_shape(D, 1);
    if ((x.nslab == 1) != (D <= 1024) || x.pairs != 0 || x.ngrp != 1 ||
        (x.nslab > 1 && x.R != 1)) {
      std::printf("D = %ld: %d slabs, %d rows\\n", (long)D, x.nslab, x.R);
      return 1;
    }
  }
}
""")


def test_resident_launches_that_share_the_device(tmp_path):
    """Beside other streams: chains up to 8,192 rows for up to 8 columns (16 up to
    4,096 rows) leave half of every XCD free, longer ones do not go resident."""
    run_host(tmp_path, """
int main() {
  for (int64_t D = 1; D <= 98304; ++D)
    for (int nb : {1, 3, 8, 9, 16, 17, 64}) {
      const ResShape x = res_shape(D, nb);
      if (!x.nslab) continue;
      // the workgroups of all teams that the launch asks for on one XCD
      const int wgs = x.nslab == 1 ? (x.ngrp + 7) / 8 : ((x.ngrp + 7) / 8) * x.nslab;
      if (res_shares(x) && std::min(wgs, 32) > 16) return 1;
      if (!res_shares(x) && wgs <= 16) return 2;
      if (D <= 1024 && nb <= 64 && !res_shares(x)) return 3;
      if (D > 1024 && D <= 4096 && nb <= 16 && !res_shares(x)) return 4;
      if (D > 4096 && D <= 8192 && nb <= 8 && !res_shares(x)) return 5;
      if (D > 16384 && res_shares(x)) return 6;
    }
}
""")
