"""Kernels at the sizes where their work splits change: window and tile edges,
remainders, smallest and largest cases, against the oracle or the general
statement of what they compute."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests.gpu_util import device, log

pytestmark = pytest.mark.gpu


def _ctx(**kw):
    from paper_2103_16141_amd.api import Context
    return Context(0, **kw)


def _status(fn):
    from paper_2103_16141_amd._native import SivfError
    try:
        fn()
    except SivfError as e:
        return e.name, str(e)
    return "SIVF_OK", ""


# ---------------------------------------------------------------- validation
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("shift", [0, 1])
def test_validation_of_long_and_short_rows_at_window_edges(dtype, shift):
    # nonzeros are read 4 per thread and 256 per wave whatever their rows; rows
    # of 1, 255 .. 257, 1,023 .. 1,025 and 5,000 nonzeros put faults on both
    # sides of those edges, and shift = 1 takes arrays off 16-byte alignment
    from paper_2103_16141_amd.api import DeviceCsr
    log("validation windows %s shift %d" % (np.dtype(dtype), shift))
    lens = [1, 255, 256, 257, 0, 1023, 1024, 1025, 0, 0, 5000, 3]
    d = 6000
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    col = np.concatenate([np.arange(m) for m in lens]).astype(np.int32)   # every row starts below its predecessor's end
    val = np.ones(rp[-1], dtype)
    ctx = _ctx()

    def check(c, v):
        cc = torch.from_numpy(np.concatenate([np.zeros(shift, np.int32), c])).to(device())[shift:]
        vv = torch.from_numpy(np.concatenate([np.zeros(shift, dtype), v])).to(device())[shift:]
        return _status(lambda: ctx.validate(DeviceCsr(torch.from_numpy(rp).to(device()), cc, vv, d)))

    assert check(col, val)[0] == "SIVF_OK"
    rows = np.repeat(np.arange(len(lens)), lens)
    edges = sorted({p for e in (256, 512, 768, 1024, 2048, 4096, len(col)) for p in (e - 1, e, e + 1) if 0 < p < len(col)})
    for p in edges:
        if rows[p] == rows[p - 1]:
            c = col.copy()
            c[p] = c[p - 1]
            name, msg = check(c, val)
            assert name == "SIVF_E_UNSORTED" and "row %d " % rows[p] in msg, p
        if p + 1 == len(col) or rows[p] != rows[p + 1]:
            c = col.copy()
            c[p] = d
            name, msg = check(c, val)
            assert name == "SIVF_E_RANGE" and "row %d " % rows[p] in msg, p
        v = val.copy()
        v[p] = -np.inf if p % 2 else np.nan
        name, msg = check(col, v)
        assert name == "SIVF_E_NONFINITE" and "row %d " % rows[p] in msg, p
