"""The partial tiles that a chunk's workgroup leaves for the workgroup that
adds them up: in the gfx950 code of k_segment_accum every wave has to wait for
its own stores before the barrier that one wave's release and count follow.
The barrier itself waits for LDS operations only, and the release's wait covers
the releasing wave's stores only."""
import os
import re
import subprocess

from paper_1107_4107_amd import build


def _assembly(tmp_path, source):
    out = tmp_path / "dev.s"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-Wall")]
    subprocess.run([build.hipcc(), *flags, "-w", "-I", build.INCLUDE, "-I", build.CSRC, "-S", "--cuda-device-only",
                    os.path.join(build.CSRC, source), "-o", str(out)], check=True, timeout=600)
    return out.read_text()


def test_every_wave_waits_for_its_partial_tile_before_the_release(tmp_path):
    text = _assembly(tmp_path, "aw_hist.hip")
    name = re.search(r"^(_ZN2aw\d+k_segment_accum\S*):", text, re.M).group(1)
    body = text[text.index(f"\n{name}:"):]
    body = [s.strip() for s in body[:body.index(".Lfunc_end")].splitlines()]
    release = [i for i, s in enumerate(body) if s.startswith("buffer_wbl2")]
    assert len(release) == 1, "one release per workgroup"
    barrier = max(i for i in range(release[0]) if body[i].startswith("s_barrier"))
    stores = [i for i in range(barrier) if body[i].startswith("global_store")]
    assert stores, "the partial tile is stored before the barrier"
    waits = [s for s in body[stores[-1]:barrier] if re.match(r"s_waitcnt\b.*\bvmcnt\(0\)", s)]
    assert waits, f"no wait for outstanding stores before the barrier: {body[stores[-1]:barrier + 1]}"
