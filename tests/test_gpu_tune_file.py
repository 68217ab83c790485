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


@pytest.mark.parametrize("n,prec", [(64, "f64"), (64, "f32h64"), (640, "f64")])
def test_a_line_timed_without_the_own_launches_is_passed_over(lbm, tmp_path, n, prec):
    # an unmarked line of a handle that has launches of its own: whoever wrote it
    # did not time them; the choice is made anew, once
    path = tmp_path / "tune.txt"
    key = _key(lbm, _square(n), prec, path)
    path.write_text(f"{key} 512 1 1 0 1 0\n")
    seen = []
    for _ in range(2):
        s = lbm.Solver(_square(n), prec)
        s.step(7)
        lbm.lbm_autotune(s.h, 10, str(path))
        seen.append(lbm.lbm_launch_steps(s.h))
        s.close()
    lines = path.read_text().splitlines()
    assert len(lines) == 2 and lines[1].split()[0] in (key + ":own", key + ":shape")
    assert seen[0][0] > 1 and seen[0] == seen[1]


@pytest.mark.parametrize("n,prec", [(64, "f16split"), (300, "f32h64")])
def test_a_line_of_a_handle_without_own_launches_is_taken(lbm, tmp_path, n, prec):
    path = tmp_path / "tune.txt"
    key = _key(lbm, _square(n), prec, path)
    path.write_text(f"{key} 512 1 1 0 1 0\n")
    s = lbm.Solver(_square(n), prec)
    lbm.lbm_autotune(s.h, 10, str(path))
    assert lbm.lbm_launch_steps(s.h)[0] == 1 and len(path.read_text().splitlines()) == 1
    s.close()
