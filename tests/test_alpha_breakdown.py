"""A CG column whose <p, A p> is not positive and finite, with alpha formed inside the D_eo launch.

Every block of that launch decides from the column state whether the column takes part (a
barrier depends on it), and blocks start at different times: the block that records the breakdown may
not change that decision for the blocks still to come.  The beta step that follows takes the column
out.  The state updates are compiled for the host here and run in the order of such a launch."""
import subprocess

from paper_1411_2223_amd import build

HARNESS = r"""
#include <stdio.h>
#include <string.h>
#include "asq_reduce.h"
using namespace asq;
#define CHECK(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)

int main() {
  const double bad[] = {0.0, -1.0, INFINITY, -INFINITY, NAN};
  for (double pAp : bad) {
    ColState S;
    memset(&S, 0, sizeof(S));
    S.tol = 1e-10;
    S.maxiter = 100;
    finalize_column(S, 4.0, OP_INIT);
    CHECK(state_on(S, MASK_ACTIVE));
    double alpha = 1;
    CHECK(!alpha_step(S, pAp, true, alpha) && alpha == 0);   // block 0
    CHECK(state_on(S, MASK_ACTIVE));                         // a block that starts now
    CHECK(!alpha_step(S, pAp, false, alpha) && alpha == 0);  // decides alike
    for (double s : {1.0, (double)NAN}) {                    // whatever the partials hold
      ColState E = S;
      finalize_column(E, s, OP_BETA);
      CHECK(!state_on(E, MASK_ACTIVE) && !state_on(E, MASK_RELIABLE) && !E.active && E.status == ASQ_ENAN);
      CHECK(E.iters == 0 && E.pbuf == 0 && E.rr == 4.0 && E.alpha == 0 && !E.converged);
    }
  }
  ColState S;
  memset(&S, 0, sizeof(S));
  S.tol = 1e-10;
  S.maxiter = 100;
  finalize_column(S, 4.0, OP_INIT);
  double alpha = 0;
  CHECK(alpha_step(S, 8.0, true, alpha) && alpha == 0.5 && S.alpha == 0.5 && S.pAp == 8.0);
  finalize_column(S, 1.0, OP_BETA);
  CHECK(state_on(S, MASK_ACTIVE) && S.iters == 1 && S.pbuf == 1 && S.beta == 0.25 && S.status == 0);
  printf("ok\n");
  return 0;
}
"""


def test_breakdown_keeps_the_column_on_until_beta(tmp_path):
    src, exe = tmp_path / "harness.hip", tmp_path / "harness"
    src.write_text(HARNESS)
    # host code only, as device code of this file would need a GPU to run
    r = subprocess.run([build.hipcc(), "--offload-host-only", "-O1", "-std=c++17", f"-I{build.INCLUDE}",
                        f"-I{build.CSRC}", str(src), "-o", str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout + r.stderr[-2000:]
