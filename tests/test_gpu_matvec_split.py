"""The batch-1 product where a tile row is split over workgroups: sizes that take one, two and four, a last group of eight tile
rows that is not full, rows that end inside a step, all codes, against the oracle's dequantizer; the call that transforms
its own input gives the bits of the two calls."""
import numpy as np
import pytest

import oracle
import qtip_synth as synth
from qtip_synth import CODE_1MAD, CODE_3INST, CODE_HYB, CODE_HYB1, CODE_HYB2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("code,V", [(CODE_1MAD, 1), (CODE_3INST, 1), (CODE_HYB, 2), (CODE_HYB2, 2), (CODE_HYB1, 1)])
@pytest.mark.parametrize("k", [2, 3, 4])
@pytest.mark.parametrize("m,n,block", [(16, 16, 16), (144, 1024, 512), (784, 1040, 16), (1040, 2064, 16), (2064, 4096, 2048),
                                       (48, 8192, 8192), (1040, 8448, 256), (4112, 1088, 64)])
def test_every_split(code, V, k, m, n, block):
    import torch
    import paper_2406_11235_amd as q
    w = synth.Workload("mv_split", 33, 5 * k + code + m % 89, m, n, code, k, V, block, 16, row_scale=True)
    inp = synth.make_inputs(w)
    d = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()
    codes, lut, sc, x, sg = d(inp.codes), d(inp.lut), d(inp.row_scale), d(inp.X[:1]), d(inp.signs_n)
    xt = torch.empty((1, n), dtype=torch.float16, device="cuda")
    q.qtip_rht(x, sg, n, block, 1, 0, xt)
    y = torch.full((m + 64,), float("nan"), device="cuda")
    q.qtip_decode_matmat(codes, 16, k, V, code, lut, m, n, xt, 1, sc, y)
    y2, xt2 = torch.full((m + 64,), float("nan"), device="cuda"), torch.empty_like(xt)
    q.qtip_rht_decode_matvec(codes, 16, k, V, code, lut, m, n, x, sg, block, sc, y2, xt2)
    torch.cuda.synchronize()
    W = oracle.dequantize(inp.codes, 16, k, V, code, m, n, inp.lut)
    ref = W.view(np.float16).astype(np.float64) @ xt[0].double().cpu().numpy() * inp.row_scale.astype(np.float64)
    got = y.cpu().numpy()
    assert np.all(np.isnan(got[m:])) and np.array_equal(got[:m], y2.cpu().numpy()[:m])
    # (the 1MAD loop contracts the unrounded quotient: 2^-12 of a weight)
    assert np.abs(got[:m] - ref).max() <= (5e-4 if code == CODE_1MAD else 1e-5) * np.abs(ref).max()


@pytest.mark.parametrize("code,V", [(CODE_1MAD, 1), (CODE_3INST, 1), (CODE_HYB, 2), (CODE_HYB2, 2), (CODE_HYB1, 1)])
@pytest.mark.parametrize("k", [2, 3, 4])
@pytest.mark.parametrize("m,n", [(4112, 4096), (5392, 4112), (6144, 4096), (8336, 8208), (7936, 4096), (7680, 2048)])
def test_rows_behind_whole_rounds(code, V, k, m, n):
    """More tile rows than CUs: one behind the last round, a last group of eight that is not full, as many parts as CUs, two
    rounds before, and too many to split; all of them against the product of the dequantized weights in binary64, and the
    first, the last whole and the last ones against the oracle's dequantizer as well."""
    import torch
    import paper_2406_11235_amd as q
    w = synth.Workload("mv_tail", 34, 5 * k + code + m % 89, m, n, code, k, V, 16, 16, row_scale=True)
    inp = synth.make_inputs(w)
    d = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()
    codes, lut, sc, x, sg = d(inp.codes), d(inp.lut), d(inp.row_scale), d(inp.X[:1]), d(inp.signs_n)
    xt = torch.empty((1, n), dtype=torch.float16, device="cuda")
    q.qtip_rht(x, sg, n, 16, 1, 0, xt)
    y = torch.full((m + 64,), float("nan"), device="cuda")
    q.qtip_decode_matmat(codes, 16, k, V, code, lut, m, n, xt, 1, sc, y)
    y2, xt2 = torch.full((m + 64,), float("nan"), device="cuda"), torch.empty_like(xt)
    q.qtip_rht_decode_matvec(codes, 16, k, V, code, lut, m, n, x, sg, 16, sc, y2, xt2)
    torch.cuda.synchronize()
    got = y.cpu().numpy()
    assert np.all(np.isnan(got[m:])) and np.array_equal(got[:m], y2.cpu().numpy()[:m])
    Wg = torch.empty((m, n), dtype=torch.float16, device="cuda")
    q.qtip_dequantize(codes, 16, k, V, code, lut, m, n, Wg)
    all_rows = (Wg.double() @ xt[0].double()) * sc.double()
    # (the 1MAD loop contracts the unrounded quotient: 2^-12 of a weight)
    bound = 5e-4 if code == CODE_1MAD else 1e-5
    assert (y[:m].double() - all_rows).abs().max() <= bound * all_rows.abs().max()
    tm = m // 16
    for I0, I1 in ((0, 2), (tm // 256 * 256 - 1, min(tm, tm // 256 * 256 + 3)), (tm - 3, tm)):
        part = np.ascontiguousarray(inp.codes.reshape(tm, -1)[I0:I1]).reshape(-1, inp.codes.shape[-1])
        W = oracle.dequantize(part, 16, k, V, code, 16 * (I1 - I0), n, inp.lut)
        ref = W.view(np.float16).astype(np.float64) @ xt[0].double().cpu().numpy()
        ref *= inp.row_scale[16 * I0:16 * I1].astype(np.float64)
        # (the scale is that of all rows)
        assert np.abs(got[16 * I0:16 * I1] - ref).max() <= bound * np.abs(got[:m]).max()
