"""CPU test of the joint kernels' split plans (compiled from the library's host source): for
random shapes and several numbers of compute units, plans do not depend on the workspace from
the queried size on, the no-allocation forward's scratch array gives the forward's plan wherever
it accepts the problem, split workgroups fit the workspace, and chunks cover every tile once."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

from paper_2501_08453_amd import build as B  # noqa: E402

SOURCE = r"""
#include <cstdio>
#include <random>
#include "api.hip"

static int bad = 0;
static void check(bool ok, const char* what, const vc_jointattn_desc& d, int cus) {
  if (ok) return;
  if (bad++ < 10)
    printf("%s: B=%d H=%d D=%d T=%d F=%d %dx%d on %d compute units\n", what, d.batch, d.heads, d.head_dim, d.text_slot,
           d.frames, d.grid_h, d.grid_w, cus);
}
static bool same(const TailPlan& a, const TailPlan& b) {
  return a.items == b.items && a.chunks == b.chunks && a.span == b.span;
}
static bool covers(const TailPlan& p, int ntile) {
  return p.items == 0 || (p.chunks >= 2 && (p.chunks - 1) * p.span < ntile && p.chunks * p.span >= ntile);
}

int main() {
  std::mt19937 rng(7);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  auto in = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
  long split = 0, scratch_split = 0;
  for (int i = 0; i < 40000; ++i) {
    vc_jointattn_desc d{in(1, 4), in(1, 24), in(0, 1) ? 64 : 128, 0, 1, 1, (int)pow(10.0, 1.0 + 4.0 * u(rng)), 0.0f, 0};
    int64_t n = 0;
    if (check_desc(&d, &n) != VC_OK) return 2;
    const size_t f = vc_jointattn_fwd_workspace_bytes(&d), b = vc_jointattn_bwd_workspace_bytes(&d);
    const size_t s = vc_spatialattn_bwd_workspace_bytes(&d);
    for (int cus : {32, 64, 128, 256}) {
      const TailPlan fp = fwd_plan(&d, n, cus, f);
      split += fp.items > 0;
      check(covers(fp, ntiles(n)), "forward chunks", d, cus);
      check(tiles_bytes(&d, n) + (size_t)fp.items * fp.chunks * fwd_wg_bytes(d.head_dim) <= f, "forward partials", d, cus);
      check(same(fp, fwd_plan(&d, n, cus, 4 * f + 1)), "forward plan in a larger workspace", d, cus);
      if (fwd_ws_bytes(&d, n) <= VC_JOINTATTN_NOALLOC_SCRATCH_BYTES) {
        const TailPlan np = fwd_plan(&d, n, cus, VC_JOINTATTN_NOALLOC_SCRATCH_BYTES);
        scratch_split += np.items > 0;
        check(same(fp, np), "plan in the scratch array", d, cus);
        check(tiles_bytes(&d, n) + (size_t)np.items * np.chunks * fwd_wg_bytes(d.head_dim) <=
                  VC_JOINTATTN_NOALLOC_SCRATCH_BYTES, "partials in the scratch array", d, cus);
      }
      const TailPlan lp = fwd_plan(&d, n, cus, fwd_ws_bytes(&d, n));
      check(tiles_bytes(&d, n) + (size_t)lp.items * lp.chunks * fwd_wg_bytes(d.head_dim) <= fwd_ws_bytes(&d, n),
            "forward partials in the least workspace", d, cus);
      for (const SplitCost& c : {kSplitDkdv, kSplitDq})
        for (int skip : {0, fused_dq_blocks(&d, n) * 4}) {
          if (skip >= ntiles(n) || (skip && c.over == kSplitDkdv.over)) continue;
          const TailPlan bp = bwd_plan(&d, n, cus, c, skip, b);
          check(covers(bp, ntiles(n) - skip), "backward chunks", d, cus);
          check(same(bp, bwd_plan(&d, n, cus, c, skip, s)), "backward plan in the spatial workspace", d, cus);
          check(same(bp, bwd_plan(&d, n, cus, c, skip, 4 * b)), "backward plan in a larger workspace", d, cus);
          for (size_t have : {b, bwd_ws_bytes(&d, n)}) {
            const TailPlan hp = bwd_plan(&d, n, cus, c, skip, have);
            check(bwd_ws_bytes(&d, n) - tail_part_bytes(&d, n) + (size_t)hp.items * hp.chunks * tail_wg_bytes(d.head_dim) <=
                      have, "backward partials", d, cus);
          }
        }
    }
  }
  printf("%d wrong, %ld forward splits, %ld in the scratch array\n", bad, split, scratch_split);
  return bad ? 1 : split > 1000 && scratch_split > 1000 ? 0 : 3;
}
"""


def test_plans(tmp_path):
    try:
        cc = B.hipcc()
    except Exception as e:  # pragma: no cover - toolchain missing
        pytest.skip("hipcc not available: %s" % e)
    if not shutil.which(cc) and not os.path.exists(cc):
        pytest.skip("hipcc not available")
    src, exe = tmp_path / "plans.hip", tmp_path / "plans"
    src.write_text(SOURCE)
    flags = [f for f in B.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    r = subprocess.run([cc, *flags, "-I", os.path.join(ROOT, "include"), "-I", B.CSRC, str(src), "-o", str(exe),
                        "-L" + B.PKG, "-l:" + os.path.basename(B.LIB), "-Wl,-rpath," + B.PKG], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:]
