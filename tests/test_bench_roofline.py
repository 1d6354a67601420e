"""The operations the bench's roofline counts are those the kernel executes:
the hardware's counts per map step, recorded with the profile, and no more FP64
instructions than VALU instructions in all."""
import json
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


def _record():
    with open(os.path.join(ROOT, "profiles", "valu_c2.json")) as f:
        return json.load(f)


class _Aw:
    """What the roofline asks of the package: the credited counts."""
    @staticmethod
    def step_op_counts(form, tangent):
        return 387, 171, 40


class _Ens:
    map_form, tangent, size, n_steps = "s6", True, 1 << 20, 100_000


def test_roofline_counts_what_the_kernel_executes():
    rec = _record()
    r = bench.roofline(_Aw, _Ens, 1000.0, "c2")
    ops, hw = r["fp64_ops_per_map_step"], rec["fp64_insts_per_map_step"]
    for k in ("fma", "mul", "add"):
        # the counters also see the prologue, the rescales and the outputs, spread over 1e5 steps
        assert hw[k] - 1 < ops[k] <= hw[k], (k, ops[k], hw[k])
    assert r["flop_per_map_step"] == 2 * ops["fma"] + ops["mul"] + ops["add"]
    assert sum(ops.values()) <= rec["valu_insts_per_map_step"]
    assert r["achieved"] == r["flop_per_map_step"] * _Ens.size * _Ens.n_steps / 1e12
    assert r["frac"] == r["achieved"] / bench.FP64_PEAK_TFLOPS


def test_forms_and_tangent_scale_with_the_stages():
    f, m, a = bench.executed_ops("s6", True)
    assert (f, m, a) == (9 * 27 + 10 * 6 + 3, 9 * 15, 9 * 10 + 3) and f + m + a == 534
    f, m, a = bench.executed_ops("s6", False)
    assert (f, m, a) == (9 * 19 + 10 * 3 + 3, 9 * 10, 9 * 10 + 3)
    assert bench.executed_ops("stdmap", True) == (27 + 6 + 3, 15, 13)
