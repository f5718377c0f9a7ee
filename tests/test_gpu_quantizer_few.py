"""Up to 256 sequences (768 at kV = 3) go through Algorithm 4 in one launch where the workspace asks for it: the same streams
and errors, bit for bit, as from several launches, for every number of copies that the workspace can hold."""
import pytest

from qtip_synth import CODE_1MAD, CODE_3INST, CODE_HYB, CODE_HYB1, CODE_HYB2

pytestmark = pytest.mark.gpu

# steps between two copies and levels of a tree in one launch
TREE = {2: 6, 3: 4, 4: 3}


@pytest.mark.parametrize("code_id,k", [(CODE_3INST, 2), (CODE_3INST, 3), (CODE_3INST, 4), (CODE_1MAD, 2), (CODE_1MAD, 3),
                                       (CODE_1MAD, 4), (CODE_HYB1, 2), (CODE_HYB1, 3), (CODE_HYB1, 4), (CODE_HYB, 2),
                                       (CODE_HYB2, 2)])
@pytest.mark.parametrize("m,n", [(16, 16), (48, 80), (16, 4096), (32, 2064), (16, 12288)])
def test_one_launch_equals_several(code_id, k, m, n):
    import torch

    import paper_2406_11235_amd as q
    V = 2 if code_id in (CODE_HYB, CODE_HYB2) else 1
    tiles, kv, steps = m // 16 * (n // 16), k * V, 256 // V
    g = torch.Generator(device="cuda").manual_seed(240611235 + 10 * k + code_id + n)
    table = {CODE_HYB1: 64, CODE_HYB: 1024, CODE_HYB2: 1024}.get(code_id)
    lut = None if table is None else torch.randn(table, device="cuda", generator=g).half()
    W = torch.randn(m, n, device="cuda", generator=g)
    # values that tie, and one that is far from every code value
    W[:, 3:5] = 0
    W[1, 2] = 3e4
    copy = (1 << (16 - kv)) * 4
    head = q.qtip_quantize_gpu_workspace(k, V, tiles) - tiles * steps * (2048 if kv == 2 else 1024) * 4
    smallest = q.qtip_quantize_gpu_workspace(k, V, 1)

    def quantize(W, size):
        count = W.numel() // 256
        ws = torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")
        codes = torch.zeros(count, 8 * k, dtype=torch.int32, device="cuda")
        err = torch.zeros(count, device="cuda")
        q.qtip_quantize_gpu(W, m, W.shape[1], 16, k, V, code_id, lut, codes, err, ws, size)
        # (only several launches keep the sequences' final states, below 2^16, at the workspace's head)
        return codes, err, bool((ws[:4 * count].view(torch.int32) == -1).all())

    # several launches: among more sequences than one launch takes
    many = torch.cat([W, torch.randn(m, 16 * -(-769 // (m // 16)), device="cuda", generator=g)], dim=1)
    want = [x.view(m // 16, many.shape[1] // 16, -1)[:, :n // 16].reshape(tiles, -1)
            for x in quantize(many, q.qtip_quantize_gpu_workspace(k, V, many.numel() // 256))[:2]]
    longest = {2: 8, 3: 8, 4: 5}[kv]
    least = -(-(steps - 1) // longest) - 1  # copies of the longest segments; the one fewer is several launches too
    every = -(-(steps - 1) // {2: 5, 3: 3, 4: 2}[kv]) - 1
    for copies in [least - 1, least, least + 1, (steps - 1) // TREE[kv] - 1, every - 1, every, every + 7]:
        size = max(smallest, head + tiles * copies * copy)
        codes, err, one = quantize(W, size)
        room = (size - head) // (tiles * copy)
        assert one == (tiles <= (768 if kv == 3 else 256) and room >= least and
                       (tiles <= {2: 128, 3: 512, 4: 256}[kv] or room < every)), copies
        assert torch.equal(codes, want[0]) and torch.equal(err, want[1][:, 0]), copies
