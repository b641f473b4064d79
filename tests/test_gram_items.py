"""Grid of the Gram products against the items the device forms, over the
states an element can be in when a launch runs (compiled for the host from the
kernels' own header)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include <cstdio>
#include "common.h"
using namespace dg;

static Opnd op(int n, const int* optP) {
  Opnd o{};
  o.nblk = n;
  for (int i = 0; i < n; ++i) o.optP[i] = optP[i];
  o.ncols = -1;
  return o;
}

int main() {
  const int xpw[3] = {0, 1, 0}, xp[2] = {0, 1}, one[1] = {0};
  const int edges[8] = {12, 15, 16, 20, 24, 30, 36, 48};
  long long launches = 0, shapes = 0;
  for (int a = 0; a < 8; ++a)
    for (int b = a; b < 8; b += 2)
      for (int J = 1; J <= 272; ++J)
        for (int split = 0; split <= 8; split += 4)
          for (int prod = 0; prod < 3; ++prod) {
            Elem e{};
            e.J = J;
            e.ng = edges[a] * edges[b] * edges[b];
            e.gram_split = split;
            e.gpart_cap = 16LL * (3 * J) * (3 * J);
            // S^T [S HS] with a block that may be carried, [X P]^T W, W^T W
            const Opnd A = prod == 0 ? op(3, xpw) : prod == 1 ? op(2, xp) : op(1, one);
            const Opnd B[2] = {prod == 0 ? A : op(1, one), A};
            const int njob = prod == 0 ? 2 : 1, tail = prod == 0;
            const int planned = gram_grid_items(e, e.ng, A, B, njob, tail, 1, true);
            for (int p = 0; p < 2; ++p)
              for (int carried = 0; carried <= tail; ++carried) {
                const int m = host_opnd_cols(A, p, J), skip = carried ? (p ? 2 : 1) * J : 0;
                const int n0 = host_opnd_cols(B[0], p, J) - skip;
                const int n1 = njob > 1 ? host_opnd_cols(B[1], p, J) - skip : 0;
                const int need = gram_items(e, e.ng, m, n0, n1);
                const int eager = gram_grid_items(e, e.ng, A, B, njob, tail, p, false);
                const long long part = (long long)gram_nchunk_e(e, e.ng, m, n0, n0 + n1) * m * (n0 + n1);
                ++shapes;
                if (planned < need || eager < need || part > e.gpart_cap)
                  std::printf("K %d J %d split %d product %d P %d carried %d: planned %d eager %d needed %d partials %lld of %lld\n",
                              e.ng, J, split, prod, p, carried, planned, eager, need, part, e.gpart_cap);
                launches += need;
              }
          }
  std::printf("%lld shapes, %lld items\n", shapes, launches);
}
"""


TUNED = r"""
#include <cstdio>
#include "common.h"
using namespace dg;

int main() {
  for (int K : {15, 100, 1728, 13824, 55296, 110592})
    for (int J = 1; J <= 272; ++J) {
      Elem e{};
      e.J = J;
      e.ng = K;
      e.gpart_cap = 16LL * (3 * J) * (3 * J);
      const int dflt = gram_nchunk_e(e, K, 3 * J, J, 2 * J);
      for (int split = 1; split <= 8; ++split) {
        e.gram_split = split;
        const int c = gram_nchunk_e(e, K, 3 * J, J, 2 * J), most = cdiv(K, 16);
        const int want = split < most ? split : most;
        if (c != (split < 8 || want > dflt ? want : dflt)) std::printf("K %d J %d split %d: %d\n", K, J, split, c);
        if ((long long)c * 3 * J * 2 * J > e.gpart_cap) std::printf("K %d J %d split %d: partials\n", K, J, split);
      }
    }
  std::printf("done\n");
}
"""


def _run(text, tmp_path):
    src, exe = tmp_path / "items.hip", tmp_path / "items"
    src.write_text(text)
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-std=c++17", "-O1", "--offload-host-only",
                    "-I" + os.path.join(ROOT, "paper_1506_08147_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.strip().split("\n")


def test_grid_covers_every_state(tmp_path):
    lines = _run(SRC, tmp_path)
    assert len(lines) == 1 and lines[0].endswith("items"), lines[:5]


def test_tuned_chunk_counts(tmp_path):
    """Exactly the tuned count, of which the largest is never below the default."""
    assert _run(TUNED, tmp_path) == ["done"]
