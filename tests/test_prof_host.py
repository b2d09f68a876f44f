"""The counter summaries follow the kernel that a run was mostly made of, and become stale with
every source that the step kernels are built from."""
import os
import re

from paper_1211_6932_amd import prof

CSRC = os.path.join(prof.ROOT, "paper_1211_6932_amd", "csrc")


def counters(d, counter, kernels):
    d.mkdir()
    rows = ["Kernel_Name,Counter_Name,Counter_Value"]
    rows += [f'"{name}",{counter},{v}' for name, vals in kernels for v in vals]
    (d / "x_counter_collection.csv").write_text("\n".join(rows) + "\n")
    return str(d)


def test_traffic_is_that_of_the_kernel_with_the_most_launches(tmp_path):
    left_over = "void lbmp::d2q9_strip<0, true, 0, 0>(float const*, float*, lbmp::StepConst, int*)"
    two = "void lbmp::d2q9_two<true, 0, 8>(float const*, float*, lbmp::StepConst, int*)"
    copy = "lbmp::copy_probe(HIP_vector_type<float, 4u> const*)"
    dirs = [counters(tmp_path / c, c, [(left_over, [9e6]), (two, [1e6, 2e6, 3e6]), (copy, [1048576.0])])
            for c in ("FETCH_SIZE", "WRITE_SIZE")]
    r = prof.traffic(*dirs, "f32", 1000)
    assert r["bytes_per_launch"] == 2 * 2e6 * 1024


def test_step_kernels():
    for name in ("void lbmp::d2q9_region<3, true, 0, 0>(...)", "void lbmp::d2q9_two<false, 1, 4>(...)",
                 "_ZN4lbmp11d2q9_regionILi5ELb1ELi0ELi0EEEvPKDF16_PDF16_NS_9StepConstEiPi",
                 "void lbmp::d2q9_mr<true, 0, 1>(...)"):
        assert prof._is_step_kernel(name), name
    for name in ("void lbmp::d2q9_mr<true, 2, 0>(...)", "void lbmp::d2q9_mr<true, 1, 0>(...)",
                 "void lbmp::d2q9_batch_two<true, 0, 8>(...)", "void lbmp::d2q9_init<0, true, 1>(...)"):
        assert not prof._is_step_kernel(name), name


def test_the_hash_covers_what_the_step_kernels_include():
    seen, todo = set(), ["d2q9_kernels.hip"]
    while todo:
        f = todo.pop()
        if f in seen:
            continue
        seen.add(f)
        todo += re.findall(r'#include "([\w.]+)"', open(os.path.join(CSRC, f)).read())
    assert {os.path.join("paper_1211_6932_amd", "csrc", f) for f in seen} <= set(prof.KERNEL_SOURCES)
