"""Host-side pieces of the benchmark driver (no GPU)."""
import json
import os
import subprocess
import sys

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_recorded_workloads_skips_cut_lines(tmp_path):
    p = tmp_path / "all.jsonl"
    assert bench.recorded_workloads(str(p)) == set()
    assert bench.recorded_workloads(None) == set()
    lines = [json.dumps({"config": {"workload": w}}) for w in bench.WORKLOADS[:2]]
    p.write_text("\n".join(lines) + "\n" + lines[0][: len(lines[0]) // 2])  # last line cut short
    assert bench.recorded_workloads(str(p)) == set(bench.WORKLOADS[:2])


def test_more_than_one_gpu_is_refused():
    r = subprocess.run([sys.executable, "bench.py", "--gpus", "2"], cwd=ROOT, capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 2
    assert "one GPU" in r.stderr


class _Events:
    """Stands in for the library's timers: which events each kernel id holds."""
    SP_KERNEL_ATTN_DQ, SP_KERNEL_ATTN_DKDV = 2, 3

    def __init__(self):
        self.armed = {}

    def sp_profile_events(self, kid, start, stop):
        assert 1 <= kid <= 9
        self.armed.pop(kid, None)
        if start is not None:
            self.armed[kid] = (start, stop)


def test_backward_in_one_launch_is_one_row():
    ev = _Events()
    t = bench.KernelTimers(ev, None)
    t.on, t.pool = True, [(f"a{i}", f"b{i}") for i in range(8)]
    t.arm_backward(True, 6.0, 8.0)
    assert [u[:2] for u in t.used] == [(bench.ONE_LAUNCH, 14.0)]
    assert ev.armed == {3: ("a0", "b0")}
    # followed by one in two launches: the first one's events are let go
    t.arm_backward(False, 6.0, 8.0, mixed=True)
    assert [u[:2] for u in t.used[1:]] == [(2, 6.0), (3, 8.0)]
    assert ev.armed == {2: ("a1", "b1"), 3: ("a2", "b2")}
    t.only = {bench.ONE_LAUNCH}
    t.arm_backward(False, 6.0, 8.0, mixed=True)
    assert ev.armed == {} and len(t.used) == 3
    t.disarm()
