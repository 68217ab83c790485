"""Pinned memory of the read-backs: what a read takes depends on what is read."""
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
