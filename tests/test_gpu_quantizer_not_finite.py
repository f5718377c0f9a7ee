"""Blocks with samples that are infinite, undefined or so large that their squares overflow, and tables with an infinite
entry: ties between infinities decide there, and all of the second pass is a search.  The binary32 search of the oracle
says which stream comes out, and that the error is +inf, not NaN; the blocks between are none the wiser."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import oracle
from qtip_synth import CODE_1MAD, CODE_3INST, CODE_HYB, CODE_HYB1, CODE_HYB2, CODE_LUT

pytestmark = pytest.mark.gpu

INF, NAN = float("inf"), float("nan")
TABLE = {CODE_HYB: 1024, CODE_HYB2: 1024, CODE_HYB1: 64, CODE_LUT: 1 << 14}
# sample of the sequence, value: the first steps, whose states are forced; the middle, where the first pass ends; the last step
ODD = [(0, INF), (0, NAN), (1, 1e20), (3, -INF), (5, NAN), (11, 3e38), (127, NAN), (128, INF), (129, -2e19), (200, NAN),
       (254, 1e20), (255, NAN), (255, INF)]


@pytest.mark.parametrize("code_id,k,infinite_entry", [
    (CODE_3INST, 2, False), (CODE_3INST, 3, False), (CODE_1MAD, 4, False), (CODE_HYB1, 2, False), (CODE_HYB1, 3, True),
    (CODE_HYB, 2, False), (CODE_HYB2, 2, True), (CODE_HYB, 4, False), (CODE_LUT, 2, False)])
@pytest.mark.parametrize("how", ["one launch", "several", "in parts"])
def test_streams_of_odd_samples(code_id, k, infinite_entry, how):
    import torch

    import paper_2406_11235_amd as q
    L, V = (14, 1) if code_id == CODE_LUT else (16, 2 if code_id in (CODE_HYB, CODE_HYB2) else 1)
    ty, tx, kv = (8, 32, k) if code_id == CODE_LUT else (16, 16, k * V)
    rng = np.random.default_rng(100 * code_id + k)
    lut = rng.standard_normal(TABLE[code_id]).astype(np.float16) if code_id in TABLE else None
    odd = ODD
    if infinite_entry:
        lut[[5, 40]] = np.float16(INF), np.float16(-INF)
        odd = [(u, v) for u, v in ODD if np.isfinite(v)]  # (an infinite sample less an infinite entry is undefined)
    elif kv > 4:
        odd = [(u, v) for u, v in ODD if v == v]  # (minima there begin with +inf)
    # (in parts: a workspace for one sequence at a time, among more than one launch takes, and one copy fewer than a walk
    # needs, or as many as are still cheaper than several sequences at a time)
    tiles = {"one launch": 20, "several": 900, "in parts": 769 if kv == 3 else 257}[how]
    size = q.qtip_quantize_gpu_workspace(k, V, 1 if how == "in parts" else tiles)
    if how == "in parts" and L == 16 and kv <= 4:
        copies = {(2, 1): 49, (3, 1): 63, (4, 1): 126, (4, 2): 62}[kv, V]
        size = 256 + copies * (4 << (16 - kv))
    W = rng.standard_normal((tiles, 256)).astype(np.float32)
    for i, (u, v) in enumerate(odd):
        W[2 + i, u] = v
    W[2 + len(odd)] = 1e20
    check = [0, 1, *range(2, 3 + len(odd)), tiles - 1]
    Wd = torch.from_numpy(np.ascontiguousarray(W.reshape(tiles, tx, ty).transpose(1, 0, 2).reshape(tx, -1))).cuda()
    lut_d = None if lut is None else torch.from_numpy(lut).cuda()
    codes = torch.zeros(tiles, 8 * k, dtype=torch.int32, device="cuda")
    err = torch.zeros(tiles, device="cuda")
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    q.qtip_quantize_gpu(Wd, tx, ty * tiles, L, k, V, code_id, lut_d, codes, err, ws, size)
    codes, err = codes.cpu().numpy().view(np.uint32), err.cpu().numpy()
    C = oracle.codebook(L, V, code_id, lut)
    with ThreadPoolExecutor(8) as pool:
        want = list(pool.map(lambda t: oracle.tailbiting_quantize_f32(W[t], L, k, V, C), check))
    for t, (d, words) in zip(check, want):
        assert err[t] == d and np.array_equal(codes[t], words), (t, err[t], d)
    assert np.isinf(err[2:3 + len(odd)]).all() and np.isfinite(err[[0, 1, tiles - 1]]).all()
