"""The block LDL decomposition at the sizes where its panels and its triangle of updates can go wrong: one block, less than
a panel, panels and one block more, both forms of the update, both group sizes.  H has nothing above its diagonal;
L D L^T gives the matrix back, A is zero where it has no block, D symmetric."""
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
    # only the lower triangle is read
    Hin = torch.where(torch.ones_like(H, dtype=torch.bool).tril(), H, float("nan"))
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


@pytest.mark.parametrize("g", [8, 16])
@pytest.mark.parametrize("n", [2048, 3200, 3216, 4240, 8336])
def test_reconstructs_large(n, g):
    """More work beside a panel's chain than idle CUs, T made beside the first panel or ahead of it, one, two and four block
    rows per workgroup."""
    import torch
    import paper_2406_11235_amd as q
    gen = torch.Generator(device="cuda").manual_seed(n + g)
    X = torch.randn(n, n, dtype=torch.float64, device="cuda", generator=gen)
    H = X.T.contiguous() @ X / n + torch.eye(n, dtype=torch.float64, device="cuda")
    A = torch.full((n, n), float("nan"), device="cuda")
    D = torch.full((n // g, g, g), float("nan"), dtype=torch.float64, device="cuda")
    size = q.qtip_block_ldl_workspace(n)
    ws = torch.full((size // 8,), float("nan"), dtype=torch.float64, device="cuda")
    q.qtip_block_ldl(torch.tril(H), n, g, A, D, ws, size)
    blk = torch.arange(n, device="cuda") // g
    assert bool((A[blk[:, None] <= blk[None, :]] == 0).all())
    L = A.double().view(n, n // g, g)  # block columns
    L = L + torch.eye(n, dtype=torch.float64, device="cuda").view(n, n // g, g)
    LD = torch.matmul(L.transpose(0, 1).contiguous(), D).transpose(0, 1).reshape(n, n)
    back = LD @ L.reshape(n, n).T.contiguous()
    assert float((back - H).norm() / H.norm()) < 1e-7  # A is rounded to binary32


@pytest.mark.parametrize("g", [8, 16])
@pytest.mark.parametrize("filled", ["lower triangle", "g x g blocks", "everything"])
def test_what_stands_above_the_diagonal_does_not_matter(g, filled):
    """H filled in with zeros above its diagonal, above its diagonal blocks of g, and whole: the same A and D."""
    import torch
    import paper_2406_11235_amd as q
    n = 176
    gen = torch.Generator(device="cuda").manual_seed(g)
    X = torch.randn(3 * n, n, dtype=torch.float64, device="cuda", generator=gen)
    H = X.T.contiguous() @ X / (3 * n)
    H = torch.tril(H) + torch.tril(H, -1).T
    Hin = torch.tril(H) if filled != "everything" else H.clone()
    if filled == "g x g blocks":
        for i in range(0, n, g):
            Hin[i:i + g, i:i + g] = H[i:i + g, i:i + g]
    size = q.qtip_block_ldl_workspace(n)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    A, D = torch.empty(n, n, device="cuda"), torch.empty(n // g, g, g, dtype=torch.float64, device="cuda")
    q.qtip_block_ldl(Hin, n, g, A, D, ws, size)
    torch.cuda.synchronize()
    # the definition, in binary64 on the host: L_ij D_j = S_ij, S_ik -= L_ij S_kj^T
    S, L = H.cpu(), torch.eye(n, dtype=torch.float64)
    for j in range(0, n, g):
        Dj = S[j:j + g, j:j + g].clone()
        assert float((D[j // g].cpu() - Dj).norm() / Dj.norm()) < 1e-11, j
        L[j + g:, j:j + g] = torch.linalg.solve(Dj, S[j + g:, j:j + g].T).T
        S[j + g:, j + g:] -= L[j + g:, j:j + g] @ S[j + g:, j:j + g].T
    ref = L - torch.eye(n, dtype=torch.float64)
    assert float((A.cpu().double() - ref).norm() / ref.norm()) < 1e-7  # (half a unit of binary32: 6e-8)


@pytest.mark.parametrize("n,g", [(4256, 16), (4240, 8), (8352, 16)])
def test_two_and_four_rows_per_workgroup(n, g):
    """More block rows below a panel than CUs: two and four of them per workgroup, the last ones not full."""
    test_reconstructs(n, g)
