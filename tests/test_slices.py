"""The room a bf16 backward workspace has for partial weight gradients against the slice rule of csrc/common.h, which is
compiled here for the host: no token count up to the one the workspace was sized for may have more slices (no GPU needed)."""
import os
import subprocess

import pytest

import paper_2501_14183_amd as vd

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <cstdio>
#include "%s/paper_2501_14183_amd/csrc/common.h"
// d, rows of the bound, most slices of any row count up to it with the tiles chosen for the bound
int main() {
  for (int d = 64; d <= 1024; d += 64)
    for (long long bound = 1; bound <= 80000; bound += bound < 2000 ? 97 : 509) {
      const bool many = vd_attn_bf16_many_tokens(d, bound);
      int most = 1;
      for (long long M = 1; M <= bound; M += M < 600 ? 1 : 37) {
        const int s = vd_attn_bf16_splitk(d, M, many, nullptr);
        if (s > most) most = s;
      }
      const int s = vd_attn_bf16_splitk(d, bound, many, nullptr);
      std::printf("%%d %%lld %%d\n", d, bound, s > most ? s : most);
    }
}
"""


@pytest.fixture(scope="module")
def slices(tmp_path_factory):
    path = tmp_path_factory.mktemp("slices")
    (path / "rule.cpp").write_text(PROGRAM % ROOT)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-Wno-unused-command-line-argument",
                    str(path / "rule.cpp"), "-o", str(path / "rule")], check=True, capture_output=True, text=True)
    out = subprocess.run([str(path / "rule")], check=True, capture_output=True, text=True).stdout
    return [tuple(int(v) for v in line.split()) for line in out.splitlines()]


def test_workspace_has_room_for_every_slice(slices):
    lib = vd.load_library()
    assert max(s for _, _, s in slices) > 8                       # (the widths of one column of tiles reach 15)
    short, last = [], {}
    for d, rows, most in slices:
        H = d // 64
        total = lib.vardrop_attn_workspace_bytes(1, rows, d, H, vd.BF16)
        before = 4 * rows * d * 2 + 2 * H * rows * 4              # dO, dQ, dK, dV and two row sums, to 256 bytes
        room = total - (before + 255) // 256 * 256
        if room < 4 * most * d * d * 4:
            short.append((d, rows, most, room // (16 * d * d)))
        assert total >= last.get(d, 0), (d, rows)                 # a larger workspace serves every smaller selection
        last[d] = total
    assert not short, "d, rows, slices, room for: %s ..." % short[:5]
