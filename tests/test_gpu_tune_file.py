"""Lines of the autotuner's cache file that another program or another version
wrote."""
import pytest

import lbm_workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lbm(require_gpu):
    import torch
    torch.cuda.set_device(0)
    from paper_1701_00702_amd import lbm as mod
    return mod


def _key(lbm, p, prec, path):
    """The handle's key in the file, without the mark of the launches that won."""
    s = lbm.Solver(p, prec)
    s.step(7)
    lbm.lbm_autotune(s.h, 3, str(path))
    s.close()
    line = path.read_text().splitlines()[-1].split()[0]
    for mark in (":own", ":shape"):
        line = line.removesuffix(mark)
    path.unlink()
    return line


def _square(n):
    return W.scaled_cavity(W.case_c2()[0], n, n)


def test_a_line_of_the_own_launches_takes_no_shape_from_the_file(lbm, tmp_path):
    # three FP64 steps per launch have no persistent grid: the line names the
    # launches, and the shape beside them is the library's
    path = tmp_path / "tune.txt"
    key = _key(lbm, _square(640), "f64", path)
    path.write_text(f"{key}:own 256 2 0 4 2 0\n")
    s = lbm.Solver(_square(640), "f64")
    lbm.lbm_autotune(s.h, 3, str(path))
    assert len(path.read_text().splitlines()) == 1 and lbm.lbm_launch_steps(s.h) == (3, 32, 8)
    s.step(20)
    assert s.diagnostics()["nonfinite"] == 0
    assert lbm.lbm_get_launch(s.h)["persistent"] == 0
    s.close()
