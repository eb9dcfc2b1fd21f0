"""The buffer window of a right-hand-side tile in the Dslash's gather-ahead form, on the host: whichever
way the range check of a raw buffer load treats the scalar offset, a load that it lets through lies
inside the caller's vector, for waves with a whole tile, a partial one and none at all."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "dslash_kernel.hpp"
#include <cstdio>
using u64 = unsigned long long;
int main() {
  int bad = 0;
  // sites of one parity: 4^4 up to the largest lattice whose tile spans less than 2^32 bytes
  const unsigned sites[] = {128u, 4096u, 131072u, 663552u, 2097152u, 11184808u, 44739240u};
  const struct { int width, rt, elem; } forms[] = {{2, 1, 8}, {4, 2, 8}, {1, 1, 16}, {2, 2, 16}};
  for (const auto &f : forms)
    for (unsigned vh : sites) {
      const unsigned plane = vh * unsigned(f.elem);
      if (u64(vh) * f.elem * 3 * f.width >= (1ull << 32)) continue;
      for (int n = 1; n <= 64; ++n) {
        const u64 total = u64(n) * 3 * plane;
        for (int tile = 0; tile < (n + f.width - 1) / f.width + 16; ++tile) {  // up to 16 waves past the last
          const dslash::TileWindow w = dslash::tile_window(tile, f.width, n, plane);
          for (int k = 0; k < f.width; ++k)  // rhs of the tile: group h, rhs r of it
            for (unsigned off : {0u, plane / 2, plane - 16})
              for (int b = 0; b < 3; ++b) {
                const unsigned voff = off + unsigned(k * 3) * plane, soff = unsigned(b) * w.step;
                const bool in[] = {voff < w.bytes,                  // scalar offset left out of the check
                                   voff < w.bytes - soff,           // taken from the size, 32 bits
                                   u64(voff) + soff < w.bytes};     // added to the offset
                const bool exists = tile * f.width + k < n;
                const u64 at = u64(w.rhs) * 3 * plane + voff + soff;
                const u64 want = (u64(tile) * f.width + k) * 3 * plane + u64(b) * plane + off;
                for (int c = 0; c < 3; ++c) {
                  if (in[c] && at + 16 > total) bad |= 1 << c;                      // past the vector
                  if (exists && (!in[c] || at != want)) bad |= 8 << c;              // not its own rhs
                  if (!exists && in[c]) bad |= 64 << c;                             // a rhs that does not exist
                }
              }
        }
      }
    }
  std::printf("%d\n", bad);
  return bad != 0;
}
"""


def test_every_load_that_passes_the_range_check_is_inside_the_vector(tmp_path):
    src = tmp_path / "window.hip"
    src.write_text(PROGRAM)
    exe = tmp_path / "window"
    cmd = ["/opt/rocm/bin/hipcc", "-x", "hip", "--offload-host-only", "-O1", "-std=c++17",
           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_1409_1510_amd", "csrc"),
           str(src), "-o", str(exe)]
    res = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and res.stdout.strip() == "0", res.stdout
