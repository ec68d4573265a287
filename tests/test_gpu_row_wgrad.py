"""GPU unit tests of the row-tile path's float32 weight-gradient product through its test hook:
split operands (three bfloat16 parts each) against 64 bits and against the float32 matrix
instructions, which the library takes for the smallest batches and wherever a sum is not finite."""
import ctypes

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def wgrad():
    from paper_2312_06126_amd import spz
    f = spz.load().spzt_row_wgrad
    i32, ptr = ctypes.c_int32, ctypes.c_void_p
    f.argtypes = [i32] * 6 + [ptr] * 3
    f.restype = ctypes.c_int

    def pack(x):   # [rows, columns] -> fragments [row group, column block, half, column, 4]
        rows, cols = x.shape
        return x.reshape(rows // 8, 2, 4, cols // 32, 32).permute(0, 3, 1, 4, 2).contiguous()

    def run(a, b, split, slices):
        m, n = a.shape[1] // 32, b.shape[1] // 32
        pa, pb = pack(a), pack(b)
        part = torch.empty(slices * m * n * 1024, device="cuda")
        torch.cuda.synchronize()
        assert f(0, int(split), a.shape[0], m, n, slices, pa.data_ptr(), pb.data_ptr(), part.data_ptr()) == 0
        blocks = part.reshape(slices, m, n, 4, 2, 32, 4)   # row 8 g + 4 h + e, column r
        return blocks.permute(0, 1, 3, 4, 6, 2, 5).reshape(slices, m * 32, n * 32)
    return run


def operands(rows, m, n, kind, seed, scale=1.0):
    """Output gradients of `rows` rows (a magnitude a row, over the batch) and what they meet: ReLU
    outputs with masked gradients, or observations. Rows of padding are zero."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    live = rows
    rows = (rows + 31) // 32 * 32
    a = torch.randn(rows, 32 * m, device="cuda", generator=g) * torch.randn(rows, 1, device="cuda", generator=g) / live
    b = torch.randn(rows, 32 * n, device="cuda", generator=g)
    if kind == "relu":
        a = a * (torch.rand(rows, 32 * m, device="cuda", generator=g) < 0.5)
        b = torch.relu(b + 0.3)
    a[live:] = 0
    return a * scale, b


def errors(out, a, b):
    ref = a.double().t() @ b.double()
    return (out.double().sum(0) - ref).abs(), ref, a.double().abs().t() @ b.double().abs()


@pytest.mark.parametrize("kind", ["relu", "obs"])
@pytest.mark.parametrize("rows,m,n,slices", [(32, 4, 4, 1), (33, 1, 3, 2), (96, 3, 2, 1), (256, 2, 2, 8), (1000, 7, 4, 20),
                                             (8192, 4, 5, 64), (32768, 2, 2, 64), (131072, 1, 2, 64)])
def test_split_is_nearer_to_64_bits(wgrad, kind, rows, m, n, slices):
    """From the library's smallest split batch on. Bound of an element: the running sum is rounded
    once for 16 rows and at the end (2^-23 each, as the instruction's own rounding is not known
    to be to nearest), the products' lost parts are below 2^-25."""
    e2 = {0: 0.0, 1: 0.0}
    for seed in range(4):
        a, b = operands(rows, m, n, kind, seed)
        for split in (0, 1):
            err, ref, mag = errors(wgrad(a, b, split, slices), a, b)
            e2[split] += float((err ** 2).sum() / (ref ** 2).sum())
            if split:
                per_slice = a.shape[0] / slices / 16 + 3
                assert float((err - per_slice * 2.0 ** -23 * mag).max()) <= 0.0
    assert e2[1] <= e2[0], (e2[1] / e2[0]) ** 0.5


@pytest.mark.parametrize("scale", [1e-30, 1e-34, 1e-36, 1e20])
def test_split_keeps_24_bits_over_the_exponent_range(wgrad, scale):
    a, b = operands(256, 2, 2, "obs", 3, scale * 256)
    err, ref, _ = errors(wgrad(a, b, 1, 4), a, b)
    assert float(((err ** 2).sum() / (ref ** 2).sum()) ** 0.5) <= 1.5e-7   # float32 instructions: 1.45e-7


@pytest.mark.parametrize("what", ["inf", "ninf", "nan", "inf_and_zero", "overflow", "huge"])
def test_not_finite_as_float32(wgrad, what):
    """Infinities, NaN, overflowing sums and values past the scaled range give what the float32
    instructions give, bit for bit but for a NaN's payload, in the tiles that hold them; the
    other tiles are not touched by it."""
    a, b = operands(512, 5, 5, "obs", 4)
    if what == "inf_and_zero":
        b[100, ::3] = 0.0
    clean = wgrad(a, b, 1, 4)
    if what in ("inf", "ninf", "nan"):
        a[100, 40] = float(what.replace("ninf", "-inf"))
    elif what == "inf_and_zero":
        a[100, 40] = float("inf")
    elif what == "overflow":
        a[:, 40] = 1e30
        b[:, 70] = 1e30
    else:
        a[100, 40] = 1e35
    got, want = wgrad(a, b, 1, 4), wgrad(a, b, 0, 4)
    same = (got == want) | (got.isnan() & want.isnan())
    hit = torch.zeros_like(same)   # slice 0 of rows 0 .. 127, the tile pair of column 40 (and 70)
    if what == "overflow":
        hit[:, :64] = True
        hit[:, :, 64:128] = True
        assert same[:, :64, 64:128].all() and want[:, 40, 70].isinf().all()
    else:
        hit[0, :64] = True
        assert same[0, :64].all()
        if what != "huge":
            assert not want[0, 40].isfinite().any()
    assert torch.equal(got[~hit], clean[~hit])
