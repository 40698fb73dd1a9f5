"""bench.py argument handling that needs no GPU."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused_with_a_message():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 2
    assert "ONE GPU" in r.stderr


def test_backward_is_priced_as_it_runs():
    sys.path.insert(0, ROOT)
    try:
        import bench
    finally:
        sys.path.remove(ROOT)
    one_launch, stream = 2, 1
    assert bench.forms_operator(4, 1, 1, 1, one_launch) and bench.forms_operator(4, 1, 0, 500, stream)
    assert bench.forms_operator(7, 1, 1, 3, one_launch) and not bench.forms_operator(7, 1, 1, 3, stream)      # padded: passes on the stream path
    assert not bench.forms_operator(8, 1, 1, 2, one_launch) and not bench.forms_operator(4, 2, 1, 2, stream)  # so few steps are cheaper as passes
    assert bench.forms_operator(4, 4, 1, 10, one_launch) and not bench.forms_operator(4, 4, 0, 10, one_launch)
    assert not bench.forms_operator(16, 1, 1, 100, one_launch)
