"""bench.py's bytes and FLOP per kernel group follow the kernels that the layer runs."""
import pytest

import bench
import paper_2602_05711_amd as P
import synth
from paper_2602_05711_amd import binding as B

# (workload, changes, groups that launch nothing)
CASES = [("train_bf16", {}, set()), ("decode64_bf16", {}, {"schedule", "expert_dot"}),
         ("decode1_bf16", {}, {"schedule"}), ("tiny_f32", {}, {"schedule", "expert_dot"}),
         ("paper_k512_bf16", {}, set()), ("paper_k512_bf16", {"T": 511}, {"schedule", "expert_dot"}),
         ("paper_k512_bf16", {"group_size": 64}, set()), ("paper_k4096_bf16", {}, set())]


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]} {c[1]}" for c in CASES])
def test_groups_that_launch_nothing_are_absent(case):
    name, kw, absent = case
    w = synth.WORKLOADS[name].with_(**kw)
    path = B.omnimoe_layer_kernels(P.make_desc(w))
    work, gone = bench.kernel_work(w, 1000, path)
    assert set(gone) == absent and set(work) == set(P.KERNEL_NAMES)
    assert all(amount > 0 for _, amount in work.values())


def test_bytes_of_the_stage_in_one_kernel_and_of_the_sweeps():
    w = synth.WORKLOADS["paper_k512_bf16"]
    n, row = 5000, w.d * 2
    sep, _ = bench.kernel_work(w, n, B.PATH_SCHEDULE)
    one, _ = bench.kernel_work(w, n, B.PATH_TOKEN_STAGE)
    # u and v rows, x, y, idx and gates
    assert one["accumulate"] == ("hbm", 2 * n * row + w.T * row + w.T * w.d * 4 + 8 * w.M)
    swept, _ = bench.kernel_work(w, n, B.PATH_SWEEP_STAGE)
    assert swept["schedule"] == ("hbm", 12 * w.M) and swept["expert_dot"] == sep["expert_dot"]
    summed, _ = bench.kernel_work(w, n, B.PATH_SCHEDULE | B.PATH_GROUPED | B.PATH_SWEEP_SUM)
    assert summed["accumulate"][1] == sep["accumulate"][1] + 16 * w.M and summed["schedule"] == sep["schedule"]
