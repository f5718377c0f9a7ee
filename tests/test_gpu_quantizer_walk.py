"""A walk back has one wave where there are many sequences and four where there are few: the same
sequences quantized in one call and in two halves, on either side of that line, give the same streams."""
import pytest

from qtip_synth import CODE_1MAD, CODE_3INST, CODE_HYB1, CODE_LUT

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
