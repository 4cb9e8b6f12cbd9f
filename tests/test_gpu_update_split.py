"""Update with fp32 weights on the bf16 matrix instruction: every kernel form at its tile edges, ragged and unaligned
operands, its accuracy on dense and sparse rows, and magnitudes out to infinities and denormals."""
import numpy as np
import pytest
import torch

from paper_2209_06800_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda"


def place(x, ld, shift):
    """A copy of x with leading dimension ld whose first element lies `shift` elements past a 16-byte boundary."""
    n, d = x.shape
    buf = torch.full((n * ld + shift,), float("nan"), device=DEV)
    v = buf[shift:].as_strided((n, d), (ld, 1))
    v.copy_(x)
    return v


def reference(a, w, b):
    """float64 result, and a forward-error bound: d_in products and additions, each within 2^-24 of its partial sum, the
    sums bounded by |a| @ |w| -- the bound of a plain fp32 dot product, with a factor 2 for the bias and the last rounding."""
    a, w = a.double().cpu(), w.double().cpu()
    b = b.double().cpu()
    return a @ w + b, 2.0 * (a.shape[1] + 2) * 2.0 ** -24 * (a.abs() @ w.abs() + b.abs())


@pytest.mark.parametrize("n,d_in,d_out,ld,shift", [
    (1, 1, 1, 1, 0), (1000, 3, 40, 3, 1), (1, 4, 1, 4, 0), (31, 5, 3, 5, 1), (33, 16, 16, 16, 0), (64, 31, 33, 31, 3), (257, 33, 32, 33, 1), (1000, 75, 47, 75, 2),
    (4097, 100, 256, 100, 0), (300, 256, 65, 256, 0), (2049, 602, 256, 608, 0), (513, 602, 255, 602, 1), (70000, 64, 64, 64, 0),
    (70001, 100, 200, 103, 1), (70003, 257, 129, 257, 0), (9000, 320, 64, 320, 0), (9000, 321, 64, 321, 0), (66000, 161, 128, 161, 0),
    (200, 1000, 300, 1000, 0), (70000, 40, 256, 40, 0)])
def test_update_split_shapes(n, d_in, d_out, ld, shift):
    g = torch.Generator(device=DEV).manual_seed(n + 7 * d_in + d_out)
    a = place(torch.randn(n, d_in, device=DEV, generator=g), ld, shift)
    w = place(torch.randn(d_in, d_out, device=DEV, generator=g) * 0.1, d_out, shift)
    b = torch.randn(d_out, device=DEV, generator=g)
    ref, bound = reference(a, w, b)
    for out_dtype in (torch.float32, torch.bfloat16):
        buf = torch.full((n + 1, d_out + 3), float("nan"), dtype=out_dtype, device=DEV)
        binding.mgg_update(a, w, b, "none", out=buf[:n, :d_out])
        assert torch.isnan(buf[:, d_out:]).all() and torch.isnan(buf[n:]).all()       # nothing past the edges
        err = (buf[:n, :d_out].double().cpu() - ref).abs()
        extra = 0 if out_dtype == torch.float32 else 2.0 ** -8 * ref.abs()             # half a unit in the last place of bf16
        assert (err <= bound + extra).all(), (err - bound).max()


@pytest.mark.parametrize("d_in,d_out", [(64, 64), (602, 256)])
@pytest.mark.parametrize("where", ["a", "w"])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan"), 3.4e38, 1e-30, 1e-37, 0.0])
def test_update_split_magnitudes(d_in, d_out, where, value):
    """One row of A, or one column of W, of extreme magnitude: infinities stay infinities of the right sign, NaN stays in
    its row or column, tiny and huge operands keep fp32 accuracy."""
    n = 333
    g = torch.Generator(device=DEV).manual_seed(d_in)
    a = torch.rand(n, d_in, device=DEV, generator=g) + 0.5
    w = torch.rand(d_in, d_out, device=DEV, generator=g) + 0.5
    if where == "a":
        if abs(value) < 1:
            a[40] *= value
        else:
            a[40, 3] = value
    elif abs(value) < 1:
        w[:, 5] *= value
    else:
        w[3, 5] = value
    if value == 3.4e38:                        # keeps the products inside fp32
        a, w = (a, w * 0.25) if where == "a" else (a * 0.25, w)
    out = binding.mgg_update(a, w, None, "none").double().cpu()
    ref, bound = reference(a, w, torch.zeros(d_out, device=DEV))
    fin = torch.isfinite(ref)
    assert torch.equal(torch.isnan(ref), torch.isnan(out))
    assert torch.equal(ref[torch.isinf(ref)], out[torch.isinf(ref)])
    assert ((out - ref).abs()[fin] <= bound[fin] + d_in * 2.0 ** -126).all()          # (results below the normal range may be flushed)


@pytest.mark.parametrize("n,d_in,d_out,tiny", [(1, 4, 1, False), (9001, 16, 7, False), (9001, 100, 32, True), (20011, 64, 33, False),
                                               (20011, 64, 64, True), (20011, 64, 65, False), (20011, 352, 64, False)])
def test_update_split_softmax(n, d_in, d_out, tiny):
    """Softmax on the accumulators (up to 64 columns, W resident), in the tiles that are computed again too, and around the
    sizes where it stays a second pass.  A softmax moves by at most half the change of its logits; 1e-6 for expf, the sum
    and the division."""
    g = torch.Generator(device=DEV).manual_seed(d_out)
    a = torch.randn(n, d_in, device=DEV, generator=g)
    w = torch.randn(d_in, d_out, device=DEV, generator=g) * 0.3
    b = torch.randn(d_out, device=DEV, generator=g)
    if tiny:
        a[n // 2] *= 1e-30
    logits, bound = reference(a, w, b)
    ref = torch.softmax(logits, 1)
    buf = torch.full((n + 1, d_out + 3), float("nan"), device=DEV)
    binding.mgg_update(a, w, b, "softmax", out=buf[:n, :d_out])
    assert torch.isnan(buf[:, d_out:]).all() and torch.isnan(buf[n:]).all()
    err = (buf[:n, :d_out].double().cpu() - ref).abs()
    assert (err <= 1e-6 + bound.amax(1, keepdim=True) * ref).all(), err.max()


# One shape for each kernel form of the dispatch (and both for a single block of columns and for several side by side).
FORMS = {
    "narrow1": [(1000, 100, 16), (333, 64, 7)],
    "narrow2": [(5000, 64, 24), (9001, 640, 32)],
    "resident1": [(2000, 602, 256), (301, 64, 40)],
    "resident2": [(70001, 64, 64), (9001, 64, 47)],
    "resident4": [(70003, 100, 200), (9003, 64, 128)],
    "slab4": [(70003, 257, 129), (66001, 161, 128)],
    "slab2": [(20001, 602, 256), (66001, 330, 64)],
    "slab1": [(301, 1000, 300), (300, 1400, 9)],
}
SHAPES = [s for v in FORMS.values() for s in v]


def form(n, d_in, d_out):
    """The dispatch rule of the fp32 Update without softmax, as its comment states it."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    slabs = -(-d_in // 32)

    def resident(cols):
        return slabs * 192 * cols + 8 * 4608 <= 159 * 1024

    if d_out <= 16 and resident(16):
        return "narrow1"
    if d_out <= 32 and resident(32):
        return "narrow2"
    nt = 4 if d_out > 64 else 2 if d_out > 32 else 1
    while nt > 1 and -(-n // (32 if resident(32 * nt) else 256)) * -(-d_out // (32 * nt)) < cus:
        nt //= 2
    return ("resident" if resident(32 * nt) else "slab") + str(nt)


def test_every_form_of_the_split_kernel_has_its_shapes():
    for name, shapes in FORMS.items():
        assert [form(*s) for s in shapes] == [name] * len(shapes)


def one_product_per_element(n, d_in, d_out, pairs):
    """Row r holds a single non-zero, at k = r % d_in, and W repeats a few values: every sum is one product.  The pairs (a, w)
    sit in tiles of their own from both ends, in the first, the middle and the last column; all else is 1 * 1."""
    a = torch.zeros(n, d_in, device=DEV)
    w = torch.ones(d_in, d_out, device=DEV)
    a[torch.arange(n, device=DEV), torch.arange(n, device=DEV) % d_in] = 1.0
    rows = [(33 * i, n - 1 - 33 * i) for i in range(len(pairs))]             # a tile each
    for (av, wv), rr in zip(pairs, rows):
        for r in rr:
            a[r, r % d_in] = av
    k_of = torch.arange(n, device=DEV) % d_in
    for (av, wv), rr in zip(pairs, rows):
        for r in rr:
            w[r % d_in, [0, d_out // 2, d_out - 1]] = wv
    return a, w, a.gather(1, k_of[:, None]).double() * w[k_of].double()


@pytest.mark.parametrize("act", ["none", "relu"])
@pytest.mark.parametrize("n,d_in,d_out", SHAPES)
def test_update_split_overflow(n, d_in, d_out, act):
    """Products around the largest fp32 number: finite where fp32 is finite, an infinity of the right sign where it is not,
    and never a NaN (which ReLU would turn into 0)."""
    pairs = [(1.2345e25, 7.77e20), (-1.2345e25, 7.77e20), (1.844e19, 1.844e19), (1.9e19, -1.9e19), (3.4e38, 0.999), (1e20, 1e15), (-2.5e30, 1e8)]
    a, w, ref = one_product_per_element(n, d_in, d_out, pairs)
    out = binding.mgg_update(a, w, None, act)
    ref = torch.relu(ref.float()) if act == "relu" else ref.float()           # (each element one product: rounded once)
    assert torch.equal(torch.isinf(ref), torch.isinf(out)) and not torch.isnan(out).any()
    assert torch.equal(ref[torch.isinf(ref)], out[torch.isinf(ref)])
    fin = torch.isfinite(ref)
    assert ((out - ref).abs()[fin] <= 2.0 ** -23 * ref.abs()[fin]).all()


@pytest.mark.parametrize("n,d_in,d_out", SHAPES)
def test_update_split_small_beside_ordinary(n, d_in, d_out):
    """Elements down to the denormal range beside ordinary ones, where the ordinary ones meet zero weights (and the same with
    the roles of A and W exchanged): what is left is one product, right to fp32."""
    g = torch.Generator(device=DEV).manual_seed(d_in)
    v = torch.rand(n, device=DEV, generator=g) + 1.0
    v.view(torch.int32)[::2] |= 1                                             # an odd last bit: all 24 are needed
    for exp_a, exp_w in ((-115, 100), (-122, 100), (-130, 110), (-140, 120), (100, -122), (110, -135)):
        a = torch.zeros(n, d_in, device=DEV)
        w = torch.zeros(d_in, d_out, device=DEV)
        a[:, 0] = 1.0                                                         # ordinary, meets zeros
        w[2, :] = 1.0
        a[:, 1] = v * 2.0 ** (exp_a // 2) * 2.0 ** (exp_a - exp_a // 2)       # (in two factors: 2^-140 itself is a denormal)
        w[1, :] = 1.5 * 2.0 ** (exp_w // 2) * 2.0 ** (exp_w - exp_w // 2)
        ref = a[:, 1:2].double() * w[1:2].double()
        out = binding.mgg_update(a, w, None, "none").double()
        assert ((out - ref).abs() <= 2.0 ** -23 * ref.abs() + 2.0 ** -149).all(), (exp_a, exp_w)


@pytest.mark.parametrize("n,d_in,d_out", SHAPES)
def test_update_split_sparse_rows_keep_fp32_accuracy(n, d_in, d_out):
    """Rows with one non-zero, two, and one in sixteen: the 2-norm error is no larger than that of a plain fp32 sum (each
    product exact, one rounding per addition), and a single product is rounded once."""
    g = torch.Generator(device=DEV).manual_seed(n)
    w = torch.randn(d_in, d_out, device=DEV, generator=g) * 0.1
    x = torch.randn(n, d_in, device=DEV, generator=g)
    first = torch.randint(0, d_in, (n, 1), device=DEV, generator=g)
    cols = torch.arange(d_in, device=DEV)
    masks = {"one": cols == first, "two": (cols == first) | (cols == (first + d_in // 2) % d_in), "one in 16": (cols % 16 == 5).expand(n, -1)}
    for name, keep in masks.items():
        a = torch.where(keep, x, torch.zeros((), device=DEV))
        out, ref = binding.mgg_update(a, w, None, "none").double(), a.double() @ w.double()
        plain = torch.zeros(n, d_out, device=DEV)
        for k in keep.any(0).nonzero().flatten().tolist():
            plain = (plain.double() + a[:, k:k + 1].double() * w[k].double()).float()
        # (2 % for the chance in a finite sample)
        assert (out - ref).norm() <= 1.02 * (plain.double() - ref).norm(), name
        if name == "one":
            assert ((out - ref).abs() <= (1 + 2.0 ** -6) * 2.0 ** -24 * ref.abs()).all()


@pytest.mark.parametrize("act", ["none", "relu", "softmax"])
@pytest.mark.parametrize("n,d_in,d_out", SHAPES)
def test_update_split_rows_and_columns_stand_alone(n, d_in, d_out, act):
    """A row of the result is a function of that row of A and of W, bit for bit, whatever the scale of its neighbours in
    the tile; without softmax, so is a column of that column of W."""
    g = torch.Generator(device=DEV).manual_seed(n + d_out)
    a = torch.randn(n, d_in, device=DEV, generator=g)
    w = torch.randn(d_in, d_out, device=DEV, generator=g) * 0.2
    b = torch.randn(d_out, device=DEV, generator=g)
    plain = binding.mgg_update(a, w, b, act).clone()
    odd = a.clone()
    rows = [40, 41, 42, 43, n - 1]
    odd[40] *= 1e-30
    odd[41] *= 1e33
    odd[42, 3] = float("inf")
    odd[43, 0] = float("nan")
    odd[n - 1, d_in - 1] = -3e38
    keep = torch.ones(n, dtype=torch.bool, device=DEV)
    keep[rows] = False
    out = binding.mgg_update(odd, w, b, act)
    assert torch.equal(out[keep], plain[keep])
    if act == "softmax":
        return
    for value in (1e-30, 1e33, float("inf")):
        w2 = w.clone()
        w2[:, d_out - 1] *= value
        out = binding.mgg_update(a, w2, b, act)
        assert torch.equal(out[:, :d_out - 1], plain[:, :d_out - 1])


@pytest.mark.parametrize("n,d_in,d_out", SHAPES)
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan"), 1e30, 1e-30, 1e-37])
def test_update_split_magnitudes_in_every_form(n, d_in, d_out, value):
    """Rows of A in the first and the last tile, or the last column of W, of extreme magnitude."""
    g = torch.Generator(device=DEV).manual_seed(d_in)
    for where in ("a", "w"):
        a = torch.rand(n, d_in, device=DEV, generator=g) + 0.5
        w = torch.rand(d_in, d_out, device=DEV, generator=g) + 0.5
        rows = [3, n - 1]
        if where == "a":
            if abs(value) < 1:
                a[rows] *= value
            else:
                a[rows, d_in - 1] = value
        elif abs(value) < 1:
            w[:, d_out - 1] *= value
        else:
            w[3, d_out - 1] = value
        out = binding.mgg_update(a, w, None, "none").double()
        a, w = a.double(), w.double()
        # (float64 products of 0 and what is not there do not arise: all operands are positive or the value itself)
        ref, bound = a @ w, 2.0 * (d_in + 2) * 2.0 ** -24 * (a.abs() @ w.abs())
        fin = torch.isfinite(ref)
        assert torch.equal(torch.isnan(ref), torch.isnan(out))
        assert torch.equal(ref[torch.isinf(ref)], out[torch.isinf(ref)])
        assert ((out - ref).abs()[fin] <= bound[fin] + d_in * 2.0 ** -149).all()


@pytest.mark.parametrize("n", [1, 15, 17, 32, 33, 8193])
@pytest.mark.parametrize("d_in,d_out", [(4, 1), (5, 3), (31, 4), (32, 15), (33, 16), (100, 17), (64, 20), (65, 31), (600, 32)])
def test_update_split_narrow_edges(n, d_in, d_out):
    """Up to 32 columns: every remainder of rows, k and columns, rows of A and out at any element, each activation and
    output type; nothing past the edges."""
    g = torch.Generator(device=DEV).manual_seed(100 * d_in + d_out + n)
    a = place(torch.randn(n, d_in, device=DEV, generator=g), d_in + 1, 1)
    w = place(torch.randn(d_in, d_out, device=DEV, generator=g) * 0.3, d_out, 3)
    b = torch.randn(d_out, device=DEV, generator=g)
    ref, bound = reference(a, w, b)
    for act in ("none", "relu", "softmax"):
        want = torch.relu(ref) if act == "relu" else torch.softmax(ref, 1) if act == "softmax" else ref
        # (a softmax moves by at most half the change of its logits; 1e-6 for expf, the sum and the division)
        tol = 1e-6 + bound.amax(1, keepdim=True) * want if act == "softmax" else bound
        for out_dtype in (torch.float32, torch.bfloat16):
            buf = torch.full((n + 1, d_out + 3), float("nan"), dtype=out_dtype, device=DEV)
            binding.mgg_update(a, w, b, act, out=buf[:n, :d_out])
            assert torch.isnan(buf[:, d_out:]).all() and torch.isnan(buf[n:]).all()
            extra = 0 if out_dtype == torch.float32 else 2.0 ** -8 * want.abs()        # half a unit in the last place of bf16
            assert ((buf[:n, :d_out].double().cpu() - want).abs() <= tol + extra).all(), (act, out_dtype)


@pytest.mark.parametrize("act", ["none", "softmax"])
@pytest.mark.parametrize("d_in,d_out", [(64, 7), (100, 24), (64, 33), (100, 47), (100, 64), (320, 64), (602, 64), (602, 128), (64, 200), (602, 256)])
def test_update_split_rows_do_not_depend_on_how_many_there_are(d_in, d_out, act):
    """A row has the same bits in a call of any number of rows, whichever kernel form that number selects."""
    g = torch.Generator(device=DEV).manual_seed(d_in + d_out)
    a = torch.randn(70001, d_in, device=DEV, generator=g)
    w = torch.randn(d_in, d_out, device=DEV, generator=g) * 0.2
    b = torch.randn(d_out, device=DEV, generator=g)
    whole = binding.mgg_update(a, w, b, act)
    for n in (1, 33, 2000, 9001, 20001):
        assert torch.equal(binding.mgg_update(a[:n], w, b, act), whole[:n]), n


@pytest.mark.parametrize("n", [1, 129, 1000])
@pytest.mark.parametrize("d_in,d_out", [(1, 1), (2, 32), (3, 33), (3, 64), (1, 65), (2, 128), (3, 129), (2, 256), (3, 300)])
def test_update_of_rows_shorter_than_a_vector(n, d_in, d_out):
    """d_in below 4 stays with the fp32 instruction: all its column widths, operands at any element."""
    g = torch.Generator(device=DEV).manual_seed(d_in + d_out)
    a = place(torch.randn(n, d_in, device=DEV, generator=g), d_in + 1, 1)
    w = place(torch.randn(d_in, d_out, device=DEV, generator=g), d_out, 2)
    b = torch.randn(d_out, device=DEV, generator=g)
    ref, bound = reference(a, w, b)
    buf = torch.full((n + 1, d_out + 3), float("nan"), device=DEV)
    binding.mgg_update(a, w, b, "relu", out=buf[:n, :d_out])
    assert torch.isnan(buf[:, d_out:]).all() and torch.isnan(buf[n:]).all()
    assert ((buf[:n, :d_out].double().cpu() - torch.relu(ref)).abs() <= bound).all()
