"""The block LDL decomposition at the sizes where its panels and its triangle of updates can go wrong: one block, less than
a panel, panels and one block more, both forms of the update, both group sizes.  L D L^T gives the matrix back, A is
zero where it has no block, D symmetric."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("g", [8, 16])
@pytest.mark.parametrize("n", [16, 32, 112, 128, 144, 256, 272, 416, 1152, 1184])
def test_reconstructs(n, g):
    import torch
    import paper_2406_11235_amd as q
    gen = torch.Generator(device="cuda").manual_seed(n + g)
    X = torch.randn(3 * n, n, dtype=torch.float64, device="cuda", generator=gen)
    X = 0.8 * X[:, :1] + 0.2 * X
    H = X.T.contiguous() @ X / (3 * n) + 1e-3 * torch.eye(n, dtype=torch.float64, device="cuda")
    Hin = torch.tril(H)
    for i in range(0, n, g):  # only blocks on and below the diagonal are read
        Hin[i:i + g, i:i + g] = H[i:i + g, i:i + g]
        Hin[i:i + g, (i // 16 + 1) * 16:] = float("nan")
    if g == 8:
        for i in range(0, n, 16):
            Hin[i:i + 16, i:i + 16] = H[i:i + 16, i:i + 16]
    A = torch.full((n, n), float("nan"), device="cuda")
    D = torch.full((n // g, g, g), float("nan"), dtype=torch.float64, device="cuda")
    size = q.qtip_block_ldl_workspace(n)
    ws = torch.full((size // 8,), float("nan"), dtype=torch.float64, device="cuda")
    q.qtip_block_ldl(Hin, n, g, A, D, ws, size)
    L = A.double() + torch.eye(n, dtype=torch.float64, device="cuda")
    back = L @ torch.block_diag(*D) @ L.T.contiguous()
    torch.cuda.synchronize()
    assert float((back - H).norm() / H.norm()) < 1e-7  # A is rounded to binary32
    blk = torch.arange(n, device="cuda") // g
    assert bool((A[blk[:, None] <= blk[None, :]] == 0).all())
    assert float((D - D.transpose(1, 2)).abs().max()) < 1e-12 * float(D.abs().max())
    # without D, the same A
    A2 = torch.empty_like(A)
    q.qtip_block_ldl(Hin, n, g, A2, None, ws, size)
    torch.cuda.synchronize()
    assert torch.equal(A, A2)
