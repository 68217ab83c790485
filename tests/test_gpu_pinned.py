"""Pinned memory of the read-backs: what a read takes depends on what is read."""
import os
import subprocess
import sys

import numpy as np
import pytest

import lbm_workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lbm(require_gpu):
    import torch
    torch.cuda.set_device(0)
    from paper_1701_00702_amd import lbm as mod
    return mod


def _mapped_mib():
    return int(open("/proc/self/statm").read().split()[0]) * 4096 / 2**20


def test_a_few_rows_of_a_large_cavity_pin_no_slots(lbm):
    # the slots' 24 MiB of pinned memory cost more at their first use than a small
    # read is worth: the first two of fewer than 2^19 nodes go without
    p = W.scaled_cavity(W.case_c2()[0], 1024, 1024)
    first = lbm.Solver(p, "f32h64")          # what the runtime allocates once
    first.fields_rows(3, 1), first.fields_rows(3, 1), first.fields()
    s = lbm.Solver(p, "f32h64")
    s.set_initial(0, *W.initial_temperatures(p, 30, amplitude=1e-2))
    s.step(3)
    before = _mapped_mib()
    reads = [s.fields_rows(500, 2), s.fields_rows(500, 2)]
    grown = _mapped_mib() - before
    reads += [s.fields_rows(500, 2), s.fields_rows(500, 2)]
    pinned = _mapped_mib() - before
    whole = s.fields()
    reads.append(s.fields_rows(500, 2))
    for r in reads:
        for k in whole:
            assert np.array_equal(r[k], whole[k][500:502]), k
    assert grown < 12 and pinned >= 24, (grown, pinned)
    s.close()
    first.close()


CHILD = """
import sys
sys.path.insert(0, {root!r})
import torch
import lbm_workloads as W
from paper_1701_00702_amd import lbm
from test_gpu_pinned import _mapped_mib
p = W.scaled_cavity(W.case_c2()[0], 1024, 1024)
need = lbm.lbm_workspace_bytes(p, "f32h64")
ws = torch.empty(need + 256, dtype=torch.uint8, device="cuda")
own, other = torch.cuda.Stream(), torch.cuda.Stream()
s = lbm.Solver(p, "f32h64", workspace=((ws.data_ptr() + 255) // 256 * 256, need), stream=own.cuda_stream)
s.step(3)
s.fields()
x, y = torch.zeros(64, device="cuda"), torch.zeros(64, device="cuda")
g = torch.cuda.CUDAGraph()
torch.cuda.synchronize()
with torch.cuda.graph(g, stream=other, capture_error_mode={mode!r}):
    torch.add(x, 1, out=y)
    before = _mapped_mib()
    s.close()
    print("freed", before - _mapped_mib(), flush=True)
for k in range(3):
    x.fill_(k)
    torch.cuda.synchronize()
    g.replay()
    torch.cuda.synchronize()
    assert bool((y == k + 1).all())
print("replayed")
"""


@pytest.mark.parametrize("mode", ["thread_local", "global"])
def test_a_handle_destroyed_during_a_capture_gives_its_memory_back(require_gpu, mode):
    # a capture of another stream goes on beside lbm_destroy, and the handle's
    # pinned memory is freed (a process of its own, which an error would stay with)
    here = os.path.dirname(os.path.abspath(__file__))
    r = subprocess.run([sys.executable, "-c", CHILD.format(root=os.path.dirname(here), mode=mode)], capture_output=True,
                       text=True, timeout=100, env=dict(os.environ, PYTHONPATH=here))
    freed = [float(l.split()[1]) for l in r.stdout.splitlines() if l.startswith("freed")]
    assert freed and freed[0] >= 24 and "replayed" in r.stdout, (r.stdout, r.stderr[-2000:])
