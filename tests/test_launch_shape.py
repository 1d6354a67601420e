"""The rule that chooses one or two lanes per orbit, compiled for the host: a
launch shape the caller asks for is the one that runs."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_two_lanes_by_default_do_not_override_a_shape(tmp_path):
    src = tmp_path / "lanes.hip"
    src.write_text(r"""
#include <cstdio>
#include "aw_launch.hpp"
using namespace aw;
int main() {
  int bad = 0;
  auto want = [&](const char *what, bool got, bool exp) { if (got != exp) { printf("%s\n", what); ++bad; } };
  for (int64_t n : {int64_t(1), int64_t(2150), int64_t(32768), int64_t(32769), int64_t(1) << 31}) {
    const bool few = n <= 32768;
    for (bool part : {false, true}) {
      want("default", fwd_two_lanes(Tuning{}, n, part, 256), few);
      for (int block : {0, 64, 128, 256, 512})
        for (int opl : {1, 2})
          for (int unroll : {1, 2})
            for (int renorm : {1, 8, 16}) {
              Tuning t;
              t.block = block; t.opl = opl; t.unroll = unroll; t.renorm = renorm;
              const bool shaped = block || opl == 2 || unroll == 2;
              want("shape", fwd_two_lanes(t, n, part, 256), few && (part || !shaped));
              t.lpo = 1;
              want("one lane asked for", fwd_two_lanes(t, n, part, 256), false);
              t.lpo = 2;
              want("two lanes asked for", fwd_two_lanes(t, n, part, 256), true);
            }
    }
  }
  want("empty", fwd_two_lanes(Tuning{}, 0, false, 256), false);
  if (!bad) printf("ok\n");
  return bad;
}
""")
    exe = tmp_path / "lanes"
    hipcc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    csrc = os.path.join(ROOT, "paper_1107_4107_amd", "csrc")
    subprocess.run([hipcc, "-std=c++17", "-O1", "--offload-arch=gfx950", "-I", csrc, str(src), "-o", str(exe)],
                   check=True, capture_output=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout


def test_the_autotuner_can_choose_the_default():
    """The default shape is among the candidates: the automatic block for a
    single ensemble, the block it stands for (512) for a batch."""
    from paper_1107_4107_amd import Tuning, autotune
    t = Tuning()
    assert (t.block, t.orbits_per_lane, t.unroll) in autotune.CANDIDATES
    assert (512, t.orbits_per_lane, 1) in autotune.BATCH_CANDIDATES
