"""The lookup-only code's batch-1 product where a block row is split over workgroups: row counts that take every split, a last
group of eight block rows that is not full, rows of one block, and of less than a step, with the oracle's dequantizer."""
import numpy as np
import pytest

import oracle
import qtip_synth as synth
from qtip_synth import CODE_LUT

pytestmark = pytest.mark.gpu


# (the last five: rows over whole rounds of workgroups, one or several for each, with one and with several steps of a row)
@pytest.mark.parametrize("k", [2, 3, 4])
@pytest.mark.parametrize("m,n", [(32, 8), (32, 1032), (288, 136), (4096, 520), (4128, 264), (8224, 72), (8192, 4104),
                                 (8224, 8), (8704, 40), (2080, 14464), (4160, 20480), (8288, 8200)])
def test_every_split(k, m, n):
    import torch
    import paper_2406_11235_amd as q
    w = synth.Workload("lut_split", 31, 7 * k + m % 97, m, n, CODE_LUT, k, 1, 8, 8, row_scale=True)
    inp = synth.make_inputs(w)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    x = torch.randn(1, n, device="cuda").half()
    y = torch.full((m + 64,), float("nan"), device="cuda")
    q.qtip_decode_matmat(d(inp.codes), 14, k, 1, CODE_LUT, d(inp.lut), m, n, x, 1, d(inp.row_scale), y)
    torch.cuda.synchronize()
    W = oracle.dequantize(inp.codes, 14, k, 1, CODE_LUT, m, n, inp.lut, tile=(32, 8))
    ref = W.view(np.float16).astype(np.float64) @ x[0].double().cpu().numpy() * inp.row_scale.astype(np.float64)
    got = y.cpu().numpy()
    assert np.all(np.isnan(got[m:]))
    assert np.abs(got[:m] - ref).max() <= 1e-5 * np.abs(ref).max()
