"""The rules that split products over workgroups do not make a matrix or a batch slower than one with more rows."""
import pytest

from qtip_synth import CODE_1MAD, CODE_3INST, CODE_HYB, CODE_HYB1, CODE_HYB2, CODE_LUT

pytestmark = pytest.mark.gpu

TABLE = {CODE_HYB: 1024, CODE_HYB2: 1024, CODE_HYB1: 64, CODE_LUT: 1 << 14}


class Product:
    def __init__(self, code, k, m, n, B=1):
        import torch
        g = torch.Generator(device="cuda").manual_seed(24061123 + k)
        self.L, self.V = (14, 1) if code == CODE_LUT else (16, 2 if code in (CODE_HYB, CODE_HYB2) else 1)
        self.code, self.k, self.m, self.n = code, k, m, n
        self.codes = torch.randint(-2**31, 2**31, (m * n // 256, 8 * k), dtype=torch.int32, device="cuda", generator=g)
        self.lut = torch.randn(TABLE[code], device="cuda", generator=g).half() if code in TABLE else None
        self.x = torch.randn(B, n, device="cuda", generator=g).half()

    def __call__(self, m, B=1):
        """The first m rows, the first B of the batch."""
        import torch
        import paper_2406_11235_amd as q
        if B > 1:
            Y = torch.empty(B, m, device="cuda")
            q.qtip_decode_matmat(self.codes, self.L, self.k, self.V, self.code, self.lut, m, self.n, self.x, B, None, Y)
            return Y
        y = torch.empty(m, device="cuda")
        q.qtip_decode_matvec(self.codes, self.L, self.k, self.V, self.code, self.lut, m, self.n, self.x, y)
        return y

    def us(self, m, B=1):
        import torch
        self(m, B)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            kept = [self(m, B) for _ in range(20)]
        times = []
        for _ in range(6):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            graph.replay()
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b) * 1e3 / len(kept))
        return min(times[1:])


# (times of the fewer rows over those of the more with the parts of the rows behind whole rounds in more than one round of
# their own: 1.3 to 1.75; the lookup-only code's with rows round the workgroups or quarters at too low a price: 1.25 to 1.47)
@pytest.mark.parametrize("code,k,fewer,more,n", [
    (CODE_HYB, 4, 7168, 8192, 14336), (CODE_HYB, 3, 11264, 12288, 14336), (CODE_HYB2, 4, 11264, 12288, 14336),
    (CODE_3INST, 4, 7168, 8192, 14336), (CODE_HYB1, 4, 7168, 8192, 28672),
    (CODE_LUT, 4, 3200, 4096, 28672), (CODE_LUT, 4, 6912, 8192, 14464), (CODE_LUT, 4, 6912, 8192, 28672),
    (CODE_LUT, 4, 22528, 24576, 28672)])
def test_fewer_rows_take_no_longer(code, k, fewer, more, n):
    product = Product(code, k, more, n)
    a, b = product.us(fewer), product.us(more)
    assert a <= 1.15 * b, (a, b)


# (a row's sum is taken in one order by whole rows and in another by halves: 128 tile rows, which are always halves, give the
# same bits as the same rows of a larger matrix only if that is in halves too)
@pytest.mark.parametrize("code,k,m,n,halves", [
    (CODE_HYB1, 2, 4112, 4608, True), (CODE_HYB1, 2, 6144, 4096, True), (CODE_HYB1, 2, 10240, 7168, True),
    (CODE_HYB1, 2, 4112, 6144, False), (CODE_HYB1, 2, 6144, 8192, False), (CODE_HYB1, 3, 5632, 5120, True),
    (CODE_HYB1, 3, 5632, 6144, False), (CODE_HYB1, 4, 5632, 4608, True), (CODE_1MAD, 2, 6144, 4096, True),
    (CODE_1MAD, 2, 6144, 5120, False), (CODE_3INST, 2, 5632, 6144, False), (CODE_3INST, 2, 5632, 14336, True),
    (CODE_3INST, 2, 4112, 4096, False), (CODE_3INST, 3, 6144, 4096, False)])
def test_rows_in_halves(code, k, m, n, halves):
    import torch
    product = Product(code, k, m, n)
    assert torch.equal(product(2048), product(m)[:2048]) == halves


# (with one time per round for all codes: 1.16 to 1.41; with one workgroup of 32 x 32 on a CU, where there is room for two, 1.15)
@pytest.mark.parametrize("code,k,m,n,fewer,more", [
    (CODE_3INST, 2, 4128, 768, 96, 128),
    (CODE_HYB, 2, 9216, 4096, 96, 128), (CODE_HYB1, 2, 6400, 2048, 160, 192), (CODE_3INST, 3, 4128, 14464, 224, 256),
    (CODE_LUT, 2, 8192, 1024, 160, 192), (CODE_LUT, 4, 6144, 4096, 192, 224)])
def test_fewer_batch_rows_take_no_longer(code, k, m, n, fewer, more):
    product = Product(code, k, m, n, more)
    a, b = product.us(m, fewer), product.us(m, more)
    assert a <= 1.1 * b, (a, b)


# (two and more batch rows, up to 16: a row's sum is over 16 waves' slices of the inputs or over eight's, whatever rows share a
# workgroup; 4096 rows have 16 waves.  Before the rule looked at the code: V = 1 hash code, 14336 x 4096, 3 bits, 8 rows 16.6 us with
# eight waves, 19.0 with 16; HYB2 3 bits 10240 x 8192, 16 rows, single rows 22.8, pairs 25.8)
@pytest.mark.parametrize("code,k,m,n,B,waves", [
    (CODE_HYB1, 3, 14336, 4096, 8, 8), (CODE_HYB1, 3, 10240, 4096, 8, 8), (CODE_HYB1, 3, 10240, 8192, 8, 16),
    (CODE_HYB1, 2, 14336, 4096, 8, 16), (CODE_HYB1, 2, 14336, 8192, 16, 8), (CODE_HYB1, 3, 16400, 4096, 2, 8),
    (CODE_3INST, 3, 10240, 4096, 2, 16), (CODE_3INST, 2, 14336, 8192, 8, 16), (CODE_3INST, 2, 14336, 8192, 9, 8),
    (CODE_3INST, 4, 14336, 8192, 8, 8), (CODE_1MAD, 4, 14336, 8192, 8, 16), (CODE_1MAD, 3, 8192, 4096, 16, 16),
    (CODE_HYB2, 3, 10240, 8192, 16, 8), (CODE_HYB2, 4, 10240, 8192, 16, 16), (CODE_HYB, 4, 14336, 2048, 8, 8)])
def test_waves_of_up_to_16_batch_rows(code, k, m, n, B, waves):
    import torch
    product = Product(code, k, m, n, B)
    assert torch.equal(product(4096, B), product(m, B)[:, :4096]) == (waves == 16)


# (the kernel for 16 batch rows at a time gives each of 17 and more the bits that it gives to one of 16; the other kernel
# sums in another order.  us, that kernel before the rule ended at 256 rows, and the other: 16 x 4096, 2-bit 3INST, 2000 rows 28.7 and
# 9.5; before it looked for a table: 3-bit 1MAD 14336 x 14336, 32 rows, 53.9 and 50.2; before it looked where rows begin: 3-bit HYB
# 480 x 28400, 140 rows, 54.5 and 38.6)
@pytest.mark.parametrize("code,k,m,n,B,same", [
    (CODE_3INST, 2, 16, 4096, 256, True), (CODE_3INST, 2, 16, 4096, 257, False), (CODE_HYB, 4, 16, 4096, 2000, False),
    (CODE_1MAD, 3, 2064, 4096, 32, True), (CODE_1MAD, 3, 2064, 4096, 33, False), (CODE_HYB2, 2, 4096, 4096, 32, True),
    (CODE_HYB, 4, 8208, 4096, 32, True), (CODE_HYB, 4, 8208, 4112, 32, False), (CODE_HYB1, 2, 8208, 8192, 17, True),
    (CODE_HYB1, 2, 8208, 8208, 17, False), (CODE_3INST, 2, 8208, 4096, 32, False), (CODE_1MAD, 3, 14336, 1024, 17, False),
    (CODE_HYB, 3, 2064, 2048, 32, True), (CODE_HYB, 3, 2064, 2112, 32, False), (CODE_HYB2, 2, 2064, 8208, 32, False),
    (CODE_HYB2, 2, 2064, 8256, 32, True), (CODE_3INST, 2, 2064, 4112, 32, False), (CODE_3INST, 2, 2064, 4160, 32, True),
    (CODE_HYB1, 4, 2064, 8176, 32, True), (CODE_HYB1, 4, 2064, 8208, 32, False), (CODE_HYB1, 4, 2064, 8256, 32, True),
    (CODE_3INST, 2, 1280, 1008, 64, True), (CODE_3INST, 2, 1280, 1008, 80, False), (CODE_3INST, 2, 1280, 960, 80, True)])
def test_which_kernel_takes_more_than_16_batch_rows(code, k, m, n, B, same):
    import torch
    product = Product(code, k, m, n, B)
    assert torch.equal(product(m, 16), product(m, B)[:16]) == same
