"""CPU test of the stop flag of the PCG kernels.  Block 0 sets the flag while other blocks of
the same launch read it, so the waves of a block may see it set or not, each for itself.
The kernels that move the solution vector run here, from their own source, as a workgroup
of host threads whose waves are shown different flags: the vector must not move in a launch
that ends the run, whatever each wave saw, and must move in one that does not."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1808_04669_amd", "csrc")

KERNELS = {"dfdg_kernels.hip": ["k_pcg_update", "k_pcg_jacobi", "k_pcg_upd_mg0_pre"],
           "dfdg_kernels3.hip": ["k_mf_update"]}
HELPERS = {"dfdg_kernels.hip": ["precond", "bsr_dinv"], "dfdg_kernels3.hip": ["mf_sp", "mf_sp2"]}

MAIN = r"""
static int G = 128;  // blocks of the launch: as many partials
template <typename K>
static bool run(const char* name, int threads, long n, K kernel) {
  // part: 1 a running iteration, 0 one whose sums end the run
  std::vector<double> x(n, 1.0);
  PcgScalars seen[2];
  auto moved = [&](double part, int first_done, int other_done) {
    std::fill(x.begin(), x.end(), 1.0);
    for (int w = 0; w < 2; ++w) {
      seen[w] = PcgScalars{};
      seen[w].tol2 = 1e-6;
      seen[w].maxit = 1000;
      seen[w].it = 5;
      seen[w].it2 = 6;
    }
    seen[0].done = first_done;
    seen[1].done = other_done;
    emu_block(1, G, threads, [&](int t) { kernel(part, x.data(), &seen[t < 64 ? 0 : 1]); });
    for (double v : x)
      if (v != 1.0) return true;
    return false;
  };
  bool ok = true;
  auto check = [&](bool want, double part, int a, int b, const char* what) {
    const bool got = moved(part, a, b);
    if (got != want) {
      std::printf("%s: x %s %s\n", name, got ? "moved" : "did not move", what);
      ok = false;
    }
  };
  check(true, 1, 0, 0, "in a running iteration");
  check(false, 0, 0, 0, "in the launch that ends the run, flag not seen");
  check(true, 1, 0, 0, "in a running iteration");  // (leaves large sums behind in LDS)
  check(false, 0, 0, 1, "in the launch that ends the run, flag seen by the later waves only");
  check(true, 1, 0, 0, "in a running iteration");
  check(false, 0, 1, 0, "in the launch that ends the run, flag seen by the first wave only");
  check(true, 1, 0, 0, "in a running iteration");
  check(false, 1, 1, 1, "after the run has ended");
  std::printf("%s %s\n", name, ok ? "ok" : "FAILED");
  return ok;
}

int main() {
  const int E = 128 * 256, NF = 2;  // a row a thread
  const long n = (long)E * 6;    // room for every NF below
  std::vector<double> a(n, 0.5), b(n, 0.25), c(n, 0.0), d(n, 0.0), e(n, 0.0), one(n, 1.0), q(2 * n, 0.5), zdef(E, 0.0);
  std::vector<double> vals(5L * NF * NF * E, 0.0), out(6 * G);
  std::vector<int> cols(5L * E);
  for (long i = 0; i < 5L * E; ++i) cols[i] = (int)(i % E);
  for (int F = 0; F < E; ++F) vals[F] = vals[3L * E + F] = 1.0;  // the identity in the first slot
  DevGeo g{};
  g.E = E;
  g.fgrid = G;
  g.zdef = zdef.data();
  DevBsr A{};
  A.ns = 5;
  A.cols = cols.data();
  A.vals = vals.data();
  A.dinv = A.binv = A.tdef = one.data();
  A.mfq = q.data();
  std::vector<double> rz(2 * G, 1.0), pq[2], pj[2];
  pq[1].assign(2 * G, 1.0);   // (p, S p) > 0
  pq[0].assign(2 * G, -1e-3); // breakdown
  pj[1].assign(6 * G, 1.0);
  pj[0].assign(6 * G, 1e-12); // converged
  bool ok = true;
  ok &= run("k_pcg_update", 256, n, [&](double part, double* x, PcgScalars* sc) {
    k_pcg_update<2, 0, double, double>(g, A, a.data(), b.data(), x, c.data(), d.data(), sc, rz.data(),
                                       pq[part > 0].data(), out.data());
  });
  ok &= run("k_pcg_update block Jacobi", 256, n, [&](double part, double* x, PcgScalars* sc) {
    k_pcg_update<1, 1, double, double>(g, A, a.data(), b.data(), x, c.data(), d.data(), sc, rz.data(),
                                       pq[part > 0].data(), out.data());
  });
  ok &= run("k_pcg_jacobi 128", 128, n, [&](double part, double* x, PcgScalars* sc) {
    k_pcg_jacobi<2, 5, 128>(g, A, a.data(), c.data(), b.data(), d.data(), one.data(), e.data(), x, sc, 1,
                            rz.data(), pj[part > 0].data(), out.data());
  });
  ok &= run("k_pcg_jacobi 256", 256, n, [&](double part, double* x, PcgScalars* sc) {
    k_pcg_jacobi<2, 5, 256>(g, A, a.data(), c.data(), b.data(), d.data(), one.data(), e.data(), x, sc, 1,
                            rz.data(), pj[part > 0].data(), out.data());
  });
  ok &= run("k_pcg_upd_mg0_pre", 256, n, [&](double part, double* x, PcgScalars* sc) {
    k_pcg_upd_mg0_pre<2, 5, double, double>(g, A, a.data(), b.data(), x, b.data(), c.data(), d.data(), CheB{1, 0, 0},
                                            sc, rz.data(), pq[part > 0].data(), out.data());
  });
  ok &= run("k_mf_update", 256, n, [&](double part, double* x, PcgScalars* sc) {
    k_mf_update<6, false>(g, A, a.data(), x, c.data(), d.data(), sc, rz.data(), pq[part > 0].data(), out.data());
  });
  ok &= run("k_mf_update block Jacobi", 256, n, [&](double part, double* x, PcgScalars* sc) {
    k_mf_update<1, true>(g, A, a.data(), x, c.data(), d.data(), sc, rz.data(), pq[part > 0].data(), out.data());
  });
  return ok ? 0 : 1;
}
"""


def _definition(src, name):
    """The text of the template function `name`, from its template line to the closing brace."""
    at = re.search(r"\b%s\(" % name, src).start()
    begin = src.rindex("\ntemplate <", 0, at) + 1
    i = src.index("{", src.index(")", at))
    depth = 0
    while True:
        depth += {"{": 1, "}": -1}.get(src[i], 0)
        i += 1
        if depth == 0:
            return src[begin:i] + "\n"


def test_stop_flag_seen_by_some_waves(tmp_path):
    cxx = shutil.which("g++")
    assert cxx, "the library's host sources need g++ as well"
    parts = ['#include "dfdg_device.h"\n#include "dfdg_internal.h"\n#include <cstdio>\n#include <type_traits>\n'
             "namespace dfdg {\nstruct CheB { double th, c1, c2; };\n"
             "template <int NF, int NS> constexpr int kSplit = facet_split(NF, NS);\n"
             # the launch's first loads and the smoothing's product: no part in the flag's logic
             "template <int SPL, int NS> inline void first_columns(const DevBsr&, int, int) {}\n"
             "template <int NF, int NS, int NA, typename V, typename GET>\n"
             "inline void spmv_part_mg2(const DevBsr&, int, int, int, GET, V (&a)[NA], V (&b)[NA]) {\n"
             "  for (int i = 0; i < NA; ++i) a[i] = b[i] = 0;\n}\n"]
    for names in (HELPERS, KERNELS):
        for f, fns in names.items():
            with open(os.path.join(CSRC, f)) as fh:
                src = fh.read()
            parts += [_definition(src, fn) for fn in fns]
    parts.append("}  // namespace dfdg\nusing namespace dfdg;\n" + MAIN)
    cpp = tmp_path / "flag.cpp"
    cpp.write_text("".join(parts))
    exe = tmp_path / "flag"
    subprocess.run([cxx, "-std=c++20", "-O1", "-w", "-pthread", "-I", os.path.join(ROOT, "tests", "host_hip"), "-I", CSRC,
                    str(cpp), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    print(r.stdout, r.stderr)
    assert r.returncode == 0, r.stdout
