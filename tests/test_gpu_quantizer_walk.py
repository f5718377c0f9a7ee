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


# (sequences in flight, copies of each) for sequences that are not one launch's.  A sequence that callers bring room for has 32
# copies, of 50, 84 and 63 that a walk takes at kV = 2, 3 and 4 (V = 2), and 64 of 127 at kV = 4 (V = 1): the fewest of
# which a plan is made; up to twice as many less one are a single sequence's, and one fewer than all of them leaves a part with
# nothing but the copy of the second pass's first step.  kV = 3: two parts and three, the last one of two copies.
PARTS = {(2, 1): [(200, 32), (2, 45), (1, 49)], (3, 1): [(200, 32), (2, 41), (1, 63)],
         (4, 1): [(200, 64), (2, 95), (1, 126)], (4, 2): [(200, 32), (2, 47), (1, 62)]}


@pytest.mark.parametrize("code_id,k", [(CODE_3INST, 2), (CODE_3INST, 3), (CODE_1MAD, 4), (CODE_HYB1, 2), (CODE_HYB, 2)])
def test_forward_passes_in_parts(code_id, k):
    """A forward pass that is repeated for some of the copies at a time gives what one pass gives, and what the oracle gives."""
    import numpy as np
    import torch

    import oracle
    import paper_2406_11235_amd as q
    V = 2 if code_id == CODE_HYB else 1
    kv, tiles = k * V, 800
    table = {CODE_HYB1: 64, CODE_HYB: 1024}.get(code_id)
    g = torch.Generator(device="cuda").manual_seed(11 * k + code_id)
    lut = None if table is None else torch.randn(table, device="cuda", generator=g).half()
    W = torch.randn(16, 16 * tiles, device="cuda", generator=g)
    copy = 1 << (16 - kv)  # words
    unused = 0x7FC0ABCD    # (no number that a copy or a final value holds)

    def head(count):  # words: final state, overlap and final value of every sequence in flight, in whole 256 bytes
        return (3 * count + 63) // 64 * 64

    def quantize(in_flight, copies):
        words = head(in_flight) + in_flight * copies * copy
        codes = torch.zeros(tiles, 8 * k, dtype=torch.int32, device="cuda")
        err = torch.zeros(tiles, device="cuda")
        ws = torch.full((words,), unused, dtype=torch.int32, device="cuda")
        q.qtip_quantize_gpu(W, 16, 16 * tiles, 16, k, V, code_id, lut, codes, err, ws, 4 * words)
        # the plan that was made has this many sequences in flight, and with them this many copies: what the head has
        # no use for, ahead of the copies, is as it was
        free = ws[:head(in_flight)] == unused
        assert not free[:3 * in_flight].any() and free[3 * in_flight:].all() and head(in_flight) > 3 * in_flight
        return codes.cpu().numpy().view(np.uint32), err.cpu().numpy()

    whole, err = quantize(tiles, 130)
    for in_flight, copies in PARTS[kv, V]:
        c, e = quantize(in_flight, copies)
        assert np.array_equal(c, whole) and np.array_equal(e, err), (in_flight, copies)
    C = oracle.codebook(16, V, code_id, None if lut is None else lut.cpu().numpy())
    for J in (0, tiles - 1):
        want, words = oracle.tailbiting_quantize_f32(W[:, 16 * J:16 * J + 16].cpu().numpy().reshape(-1), 16, k, V, C)
        assert np.array_equal(whole[J], words) and err[J] == want
