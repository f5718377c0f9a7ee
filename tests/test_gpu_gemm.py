"""The batched product at the sizes where its splits can go wrong: every split of outputs, batch rows
and inputs (by sizes that the launcher's rule gives to it), edges of tiles, odd numbers of steps, the smallest of
everything, for every code, against the decoded matrix times the activations in binary64."""
import pytest

from qtip_synth import CODE_1MAD, CODE_3INST, CODE_HYB, CODE_HYB1, CODE_HYB2, CODE_LUT

pytestmark = pytest.mark.gpu

CODES = {CODE_1MAD: (16, 1, 0), CODE_3INST: (16, 1, 0), CODE_HYB: (16, 2, 1024), CODE_HYB2: (16, 2, 1024),
         CODE_LUT: (14, 1, 1 << 14), CODE_HYB1: (16, 1, 64)}
# m, n, B: 32 x 32, 32 x 64, 64 x 64, 64 x 128, 128 x 128 and 128 x 256 outputs x batch rows of a workgroup (32 x 32, the first three,
# for the lookup-only code alone: the others' few outputs are another kernel's, and the end of MORE_THAN_16 has theirs)
SHAPES = [(32, 16, 17), (96, 208, 33), (544, 1056, 40), (8192, 80, 49), (8224, 48, 64), (16384, 144, 100),
          (8224, 112, 200), (16416, 80, 1000), (16384, 272, 769)]


@pytest.fixture(scope="module")
def q():
    import paper_2406_11235_amd as q
    q.lib()
    return q


def check(q, code, k, m, n, B, scaled, seed=0):
    import torch
    L, V, entries = CODES[code]
    g = torch.Generator(device="cuda").manual_seed(seed)
    codes = torch.randint(-2**31, 2**31, (m * n // 256, 8 * k), dtype=torch.int32, device="cuda", generator=g)
    lut = torch.randn(entries, device="cuda", generator=g).half() if entries else None
    X = torch.randn(B, n, device="cuda", generator=g).half()
    sc = (torch.rand(m, device="cuda", generator=g) + 0.5).half() if scaled else None
    # a guard behind Y, and nothing left from before in it
    buf = torch.full((B * m + 4096,), float("nan"), device="cuda")
    q.qtip_decode_matmat(codes, L, k, V, code, lut, m, n, X, B, sc, buf)
    W = torch.empty(m, n, dtype=torch.float16, device="cuda")
    q.qtip_dequantize(codes, L, k, V, code, lut, m, n, W)
    ref = X.double() @ W.double().T.contiguous()
    if scaled:
        ref = ref * sc.double()
    Y = buf[:B * m].view(B, m).double()
    torch.cuda.synchronize()
    assert torch.isfinite(Y).all() and torch.isnan(buf[B * m:]).all()
    err = float((Y - ref).abs().max() / ref.abs().max())
    assert err <= 1e-5, (code, k, m, n, B, err)


@pytest.mark.parametrize("code", list(CODES))
@pytest.mark.parametrize("k", [2, 3, 4])
def test_splits(q, code, k):
    for i, (m, n, B) in enumerate(SHAPES):
        check(q, code, k, m, n, B, scaled=i % 2 == 0, seed=i)


# up to 16 batch rows: halves of tile rows, with 8 and 16 waves and steps that do not fill; one and two tile rows per
# workgroup, with 8 and 16 waves, the last pair half empty; one and 16 copies of the hash code's table; slices with nothing; pairs
# between the rounds where rows are not whole cache lines
UP_TO_16 = [(16, 16), (1024, 1040), (2048, 4112), (1008, 4128), (2064, 4144), (4112, 272), (4112, 4128), (4112, 8208),
            (10256, 144), (14352, 80), (14352, 4112), (14352, 8208), (16400, 272), (10256, 2064), (10256, 4112)]


@pytest.mark.parametrize("code", [c for c in CODES if c != CODE_LUT])
@pytest.mark.parametrize("k", [2, 3, 4])
def test_up_to_16_rows(q, code, k):
    for i, (m, n) in enumerate(UP_TO_16):
        for B in ((2, 9) if i % 2 else (8, 16)):
            check(q, code, k, m, n, B, scaled=B < 9, seed=i)


# above that: 16 and 32 rows at a time, halves of tile rows, the last group nearly empty; up to 32 rows of many outputs; and the
# 32 x 32 and 32 x 64 splits where outputs are too many for these
MORE_THAN_16 = [(16, 1040, 17), (240, 4112, 100), (1024, 1056, 64), (1040, 144, 49), (2032, 4128, 50), (48, 80, 1000),
                (4096, 272, 17), (8208, 144, 32), (14352, 4112, 18), (4112, 208, 17), (2080, 1056, 40), (2080, 272, 100)]


@pytest.mark.parametrize("code", [c for c in CODES if c != CODE_LUT])
@pytest.mark.parametrize("k", [2, 3, 4])
def test_more_than_16_rows_at_a_time(q, code, k):
    for i, (m, n, B) in enumerate(MORE_THAN_16):
        check(q, code, k, m, n, B, scaled=i % 2 == 0, seed=i)


@pytest.mark.parametrize("k", [2, 3, 4])
def test_up_to_16_rows_of_the_lookup_only_code(q, k):
    for m, n, B in ((32, 8, 2), (96, 1032, 9), (4128, 2056, 16), (8224, 264, 3), (32, 14464, 8), (32, 16392, 8)):
        check(q, CODE_LUT, k, m, n, B, scaled=B > 8)


@pytest.mark.parametrize("k", [2, 3, 4])
def test_few_outputs_of_the_lookup_only_code(q, k):
    """Up to eight workgroups; an odd number of blocks, slices that do not fill."""
    for m, n in ((32, 2056), (96, 4104), (224, 8192), (256, 16384)):
        for B in (2, 3, 9, 16):
            check(q, CODE_LUT, k, m, n, B, scaled=B > 8, seed=n)


@pytest.mark.parametrize("code", [c for c in CODES if c != CODE_LUT])
@pytest.mark.parametrize("B, m", [(20, 4128), (50, 2080), (70, 1408), (130, 864)])
def test_slices_that_are_not_whole_stages_of_many_outputs(q, code, B, m):
    """The next test for the codes of 16 x 16 tiles, whose few outputs are another kernel's."""
    for n in [*range(16, 160, 16), 16 * 31, 16 * 32, 16 * 33, 16 * 61, 16 * 97]:
        check(q, code, 2 + n // 16 % 3, m, n, B, scaled=False, seed=n)


@pytest.mark.parametrize("code", list(CODES))
@pytest.mark.parametrize("B", [20, 50, 70, 130])
def test_slices_that_are_not_whole_stages(q, code, B):
    """One to nine steps, and around whole stages of eight, four and two slices of the inputs: a slice's first stage begins
    ahead of the slice, and of the row, with zeros for inputs."""
    for n in [*range(16, 160, 16), 16 * 31, 16 * 32, 16 * 33, 16 * 61, 16 * 97]:
        check(q, code, 2 + n // 16 % 3, 96, n, B, scaled=False, seed=n)


def test_half_a_step_of_the_lookup_only_code(q):
    for n in (8, 24, 8 * 65, 8 * 129):
        for m, B in ((32, 18), (64, 70), (4128, 300), (16416, 700)):
            check(q, CODE_LUT, 2 + n % 3, m, n, B, scaled=False)


# few outputs, 16 batch rows at a time (32 x 32 for the lookup-only code); and 32 x 64, 32 x 32 and 64 x 128 outputs x batch rows,
# whose copies of a slice's last stage run into the next row and whose first stage begins ahead of the row: whole stages of all
# slices, one step more, half and less
@pytest.mark.parametrize("code", [CODE_3INST, CODE_HYB, CODE_LUT])
@pytest.mark.parametrize("m,B", [(64, 37), (4128, 37), (4128, 70), (8192, 200)])
@pytest.mark.parametrize("n", [16, 80, 528, 1024, 1040])
def test_a_batch_row_meets_nothing_but_itself(q, code, m, B, n):
    """An infinity among a batch row's first, last or other inputs leaves the others finite, and as they are without it; rows
    of a last, partly filled tile included."""
    import torch
    L, V, entries = CODES[code]
    codes = torch.randint(-2**31, 2**31, (m * n // 256, 16), dtype=torch.int32, device="cuda")
    lut = torch.randn(entries, device="cuda").half() if entries else None
    X = torch.randn(B, n, device="cuda").half()
    Y, without = torch.empty(B, m, device="cuda"), torch.empty(B, m, device="cuda")
    q.qtip_decode_matmat(codes, L, 2, V, code, lut, m, n, X, B, None, without)
    for row, place in ((5, 3), (0, n - 1), (B - 2, 0), (B - 2, n - 1), (B - 1, 0)):
        Z = X.clone()
        Z[row, place] = float("inf")
        q.qtip_decode_matmat(codes, L, 2, V, code, lut, m, n, Z, B, None, Y)
        ok = torch.arange(B, device="cuda") != row
        assert torch.equal(Y[ok], without[ok]) and not torch.isfinite(Y[row]).any(), (row, place)


@pytest.mark.parametrize("code", [c for c in CODES if c != CODE_LUT])
@pytest.mark.parametrize("B", [2, 8, 9, 16])
def test_splits_of_small_batches(q, code, B):
    """At most 16 batch rows: one and two tile rows per workgroup, a last pair that is not full, both wave counts."""
    for k in (2, 3, 4):
        for m, n in ((16, 16), (4080, 48), (4112, 80), (8208, 1040), (10240, 16)):
            check(q, code, k, m, n, B, scaled=True, seed=B)


@pytest.mark.parametrize("m,n,B", [(14304, 4112, 997), (4096, 4112, 500), (8192, 8208, 100)])
def test_long_rows_are_not_one_chain_of_sums(q, m, n, B):
    """Chains of 16 matrix instructions whose sums are added up: 1.2e-7 to 1.3e-7 of the result's 2-norm is rounding
    (binary32's half unit is 6e-8, and an error of a random sign per addition grows with the root of the chain);
    one chain over 4096 inputs has 2.1e-7 or more with four slices of the inputs, and 4.1e-7 with one."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(m)
    codes = torch.randint(-2**31, 2**31, (m * n // 256, 16), dtype=torch.int32, device="cuda", generator=g)
    X = torch.randn(B, n, device="cuda", generator=g).half()
    Y = torch.empty(B, m, device="cuda")
    W = torch.empty(m, n, dtype=torch.float16, device="cuda")
    q.qtip_decode_matmat(codes, 16, 2, 1, CODE_3INST, None, m, n, X, B, None, Y)
    q.qtip_dequantize(codes, 16, 2, 1, CODE_3INST, None, m, n, W)
    ref = X.double() @ W.double().T.contiguous()
    assert (Y.double() - ref).norm() <= 1.8e-7 * ref.norm()


@pytest.mark.parametrize("k", [2, 3, 4])
@pytest.mark.parametrize("m,n", [(1024, 4096), (2048, 14464)])
def test_slices_of_the_lookup_only_code_are_not_one_chain_of_sums(q, k, m, n):
    """17 to 32 batch rows, whose waves split the inputs: a wave's sums go to totals after 16 matrix instructions as well.
    A chain of c instructions of 16 products has an error that grows with the root of c: 1.2e-7 to 1.3e-7 of the result's
    2-norm for 16 and the few sums over chains and waves (binary32's half unit is 6e-8); without totals it is 1.56e-7 for
    chains of 32 (n = 4096) and 2.76e-7 for 113 (n = 14464), with twice as many slices 1.30e-7 and 2.1e-7."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(n)
    codes = torch.randint(-2**31, 2**31, (m * n // 256, 8 * k), dtype=torch.int32, device="cuda", generator=g)
    lut = torch.randn(1 << 14, device="cuda", generator=g).half()
    W = torch.empty(m, n, dtype=torch.float16, device="cuda")
    q.qtip_dequantize(codes, 14, k, 1, CODE_LUT, lut, m, n, W)
    Wt = W.double().T.contiguous()
    for B in (17, 24, 32):
        X = torch.randn(B, n, device="cuda", generator=g).half()
        Y = torch.empty(B, m, device="cuda")
        q.qtip_decode_matmat(codes, 14, k, 1, CODE_LUT, lut, m, n, X, B, None, Y)
        ref = X.double() @ Wt
        assert (Y.double() - ref).norm() <= 1.4e-7 * ref.norm(), B


@pytest.mark.parametrize("k", [2, 3, 4])
@pytest.mark.parametrize("m,n,B", [(4128, 8, 33), (8192, 24, 64), (4160, 264, 50), (4096, 4104, 47)])
def test_stages_of_two_tiles(q, k, m, n, B):
    """33 to 64 batch rows of the lookup-only code in tiles of 32 x 64, whose stages are two tiles: half a tile, one and a
    half, one more half than whole stages; the long rows' sums within the bound of the test above."""
    import torch
    check(q, CODE_LUT, k, m, n, B, scaled=k == 3, seed=n)
    if n < 4096:
        return
    g = torch.Generator(device="cuda").manual_seed(n)
    codes = torch.randint(-2**31, 2**31, (m * n // 256, 8 * k), dtype=torch.int32, device="cuda", generator=g)
    lut = torch.randn(1 << 14, device="cuda", generator=g).half()
    X = torch.randn(B, n, device="cuda", generator=g).half()
    Y = torch.empty(B, m, device="cuda")
    W = torch.empty(m, n, dtype=torch.float16, device="cuda")
    q.qtip_decode_matmat(codes, 14, k, 1, CODE_LUT, lut, m, n, X, B, None, Y)
    q.qtip_dequantize(codes, 14, k, 1, CODE_LUT, lut, m, n, W)
    ref = X.double() @ W.double().T.contiguous()
    assert (Y.double() - ref).norm() <= 1.4e-7 * ref.norm()


def check_sparse(q, code, m, n, rows, k=None):
    """All but about 1200 inputs, the first, the last and some everywhere, are zeros, so that a single wrong tile shows: a
    wave's running sum changes in at most 400 of its additions, each of which is off by at most a unit of the sum, 2^-23."""
    import torch
    L, V, entries = CODES[code]
    k = k or 2 + code % 3
    g = torch.Generator(device="cuda").manual_seed(code)
    codes = torch.randint(-2**31, 2**31, (m * n // 256, 8 * k), dtype=torch.int32, device="cuda", generator=g)
    lut = torch.randn(entries, device="cuda", generator=g).half() if entries else None
    sc = (torch.rand(m, device="cuda", generator=g) + 0.5).half()
    some = torch.randint(0, n, (1000,), device="cuda", generator=g)
    some = torch.cat([torch.arange(40, device="cuda"), some, torch.arange(n - 120, n, device="cuda")]).unique()
    X = torch.zeros(max(rows), n, dtype=torch.float16, device="cuda")
    X[:, some] = torch.randn(max(rows), len(some), device="cuda", generator=g).half()
    W = torch.empty(m, n, dtype=torch.float16, device="cuda")
    q.qtip_dequantize(codes, L, k, V, code, lut, m, n, W)
    ref = (X[:, some].double() @ W[:, some].double().T.contiguous()) * sc.double()
    for B in rows:
        buf = torch.full((B * m + 4096,), float("nan"), device="cuda")
        q.qtip_decode_matmat(codes, L, k, V, code, lut, m, n, X, B, sc, buf)
        Y = buf[:B * m].view(B, m).double()
        torch.cuda.synchronize()
        assert torch.isnan(buf[B * m:]).all()
        assert (Y - ref[:B]).norm() <= 400 * 2.0**-23 * ref[:B].norm(), (code, B)


@pytest.mark.parametrize("code", list(CODES))
@pytest.mark.parametrize("n", [2**22 + 80, 2**25, 2**25 + 80])
def test_very_long_rows(q, code, n):
    """Lengths at which the larger splits' 32-bit offsets, and then every split's, do not reach."""
    check_sparse(q, code, 32 if code == CODE_LUT else 48, n, (17, 32, 33, 65))


@pytest.mark.parametrize("k", [2, 3, 4])
@pytest.mark.parametrize("n", [2**22, 2**22 + 80, 2**25 + 80])
def test_very_long_rows_of_few_batch_rows(q, k, n):
    """The lookup-only code where its own kernel gets what the other one's offsets do not reach, and before."""
    check_sparse(q, CODE_LUT, 32, n, (2, 9, 16), k)


@pytest.mark.parametrize("code", [c for c in CODES if c != CODE_LUT])
def test_very_long_rows_decoded_for_more_than_16_rows_at_once(q, code):
    """More than 512 tile rows times groups of 16 rows: weights decoded for 32 rows and for 64, a last pair of tile rows
    that is not full."""
    check_sparse(q, code, 16 * 171, 2**22 + 16, (48, 50, 64, 65, 97))
    check_sparse(q, code, 16 * 257, 2**22 + 16, (17, 32))
