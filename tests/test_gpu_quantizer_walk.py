"""A walk back has one wave where there are many sequences and four where there are few: the same
sequences quantized in one call and in two halves, on either side of that line, give the same streams."""
import pytest

from qtip_synth import CODE_1MAD, CODE_3INST, CODE_HYB, CODE_HYB1, CODE_LUT

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("code_id,k,tiles", [(CODE_3INST, 2, 1040), (CODE_1MAD, 3, 1026), (CODE_HYB1, 2, 2048),
                                             (CODE_LUT, 2, 514), (CODE_LUT, 3, 514)])
def test_one_call_equals_two_halves(code_id, k, tiles):
    import torch

    import paper_2406_11235_amd as q
    g = torch.Generator(device="cuda").manual_seed(240611235 + 10 * k + code_id)
    L, tx, ty = (14, 32, 8) if code_id == CODE_LUT else (16, 16, 16)
    table = {CODE_HYB1: 64, CODE_LUT: 1 << 14}.get(code_id)
    lut = None if table is None else torch.randn(table, device="cuda", generator=g).half()
    W = torch.randn(tx, ty * tiles, device="cuda", generator=g)

    def quantize(W):
        count = W.shape[1] // ty
        codes = torch.zeros(count, 8 * k, dtype=torch.int32, device="cuda")
        err = torch.zeros(count, device="cuda")
        # (room for every copy that the walks of all of them need, so that they are in flight together)
        size = q.qtip_quantize_gpu_workspace(k, 1, 2 * count)
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        q.qtip_quantize_gpu(W, tx, ty * count, L, k, 1, code_id, lut, codes, err, ws, size)
        return codes, err

    codes, err = quantize(W)
    halves = [quantize(h.contiguous()) for h in W.split(ty * tiles // 2, dim=1)]
    assert torch.equal(codes, torch.cat([c for c, _ in halves]))
    assert torch.equal(err, torch.cat([e for _, e in halves]))


@pytest.mark.parametrize("code_id,k", [(CODE_3INST, 2), (CODE_3INST, 3), (CODE_1MAD, 4), (CODE_HYB1, 2), (CODE_HYB, 2)])
def test_forward_passes_in_parts(code_id, k):
    """A forward pass that is repeated for a few copies at a time, down to one and to a last one that only has the copy of
    its first step, gives what one pass gives, and what the oracle gives."""
    import numpy as np
    import torch

    import oracle
    import paper_2406_11235_amd as q
    V = 2 if code_id == CODE_HYB else 1
    kv, steps, tiles = k * V, 256 // V, 800
    table = {CODE_HYB1: 64, CODE_HYB: 1024}.get(code_id)
    g = torch.Generator(device="cuda").manual_seed(11 * k + code_id)
    lut = None if table is None else torch.randn(table, device="cuda", generator=g).half()
    W = torch.randn(16, 16 * tiles, device="cuda", generator=g)
    copy = (1 << (16 - kv)) * 4
    head = q.qtip_quantize_gpu_workspace(k, V, tiles) - tiles * steps * (2048 if kv == 2 else 1024) * 4
    every = -(-(steps - 1) // {2: 5, 3: 3, 4: 2}[kv]) - 1
    got = []
    for copies in (every + 1, every, every - 1, every // 2, 1):
        size = head + tiles * copies * copy
        codes = torch.zeros(tiles, 8 * k, dtype=torch.int32, device="cuda")
        err = torch.zeros(tiles, device="cuda")
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        q.qtip_quantize_gpu(W, 16, 16 * tiles, 16, k, V, code_id, lut, codes, err, ws, size)
        got.append((codes.cpu().numpy().view(np.uint32), err.cpu().numpy()))
    for codes, err in got[1:]:
        assert np.array_equal(codes, got[0][0]) and np.array_equal(err, got[0][1])
    C = oracle.codebook(16, V, code_id, None if lut is None else lut.cpu().numpy())
    for J in (0, tiles - 1):
        want, words = oracle.tailbiting_quantize_f32(W[:, 16 * J:16 * J + 16].cpu().numpy().reshape(-1), 16, k, V, C)
        assert np.array_equal(got[0][0][J], words) and got[0][1][J] == want
