"""GPU parity: vq_layernorm_quantize against the CPU oracle -- levels and packed bytes bit-exact
(both sides run Eq. 5 in fp32 in element order and decide with the same comparator arithmetic),
the residual sum identical."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from oracle import vqo
from paper_2504_18547_amd import vitq
from tests.gpu_util import dev, from_qmat, storage_of


def _case(rng, rows, cols, scale=1.0):
    x = (rng.standard_normal((rows, cols)) * rng.uniform(0.2, 4.0, (rows, 1)) * scale
         + rng.uniform(-2, 2, (rows, 1))).astype(np.float32)
    gamma = rng.uniform(0.5, 1.5, cols).astype(np.float32)
    beta = (rng.standard_normal(cols) * 0.3).astype(np.float32)
    return x, gamma, beta


def _check(x, gamma, beta, eps, step, bits, res=None, ld=None):
    rows, cols = x.shape
    out = vitq.QMat.empty(rows, cols, bits)
    out.data.fill_(0xFF)                      # the whole 16-byte padded row must be overwritten
    if ld is None:
        xd, rd = dev(x), dev(res)
    else:                                     # rows embedded in a wider buffer
        big = torch.zeros((rows, ld), dtype=torch.float32, device="cuda")
        big[:, :cols] = dev(x)
        xd = big[:, :cols]
        rd = None
        if res is not None:
            bigr = torch.zeros((rows, ld), dtype=torch.float32, device="cuda")
            bigr[:, :cols] = dev(res)
            rd = bigr[:, :cols]
    sd = torch.full((rows, ld or cols), -7.0, dtype=torch.float32, device="cuda")[:, :cols] if res is not None else None
    vitq.vq_layernorm_quantize(xd, rd, sd, dev(gamma), dev(beta), eps, step, out)
    torch.cuda.synchronize()
    ref = vqo.layernorm_quantize(x, gamma, beta, eps, step, bits, res=res, want_sum=res is not None)
    got = from_qmat(out)
    assert np.array_equal(got, ref["q"]), "levels differ: %d of %d" % ((got != ref["q"]).sum(), got.size)
    assert np.array_equal(out.data.cpu().numpy(), vqo.pack(ref["q"], storage_of(bits)))
    if res is not None:
        assert np.array_equal(sd.cpu().numpy(), ref["sum"])
    return ref


@pytest.mark.parametrize("bits", [2, 3, 4, 8])
@pytest.mark.parametrize("rows,cols", [(197, 384), (130, 768), (3, 1024), (70, 37), (1, 1), (65, 5), (64, 130)])
def test_shapes_and_bit_widths(bits, rows, cols):
    rng = np.random.default_rng(rows * 31 + cols + bits)
    x, gamma, beta = _case(rng, rows, cols)
    lo, hi = vqo.qrange(bits)
    ref = _check(x, gamma, beta, 1e-5, np.float32(2.5 / hi), bits)
    if rows * cols > 5000:
        assert len(np.unique(ref["q"])) >= min(hi - lo + 1, 100)


def test_residual_strided_rows_and_no_eps():
    rng = np.random.default_rng(9)
    x, gamma, beta = _case(rng, 100, 384)
    res = rng.standard_normal((100, 384)).astype(np.float32)
    _check(x, gamma, beta, 0.0, np.float32(0.35), 4, res=res)
    _check(x, gamma, beta, 1e-6, np.float32(0.35), 4, res=res, ld=400)
    _check(x[:, :383], gamma[:383], beta[:383], 1e-6, np.float32(0.35), 4, res=res[:, :383], ld=400)   # unaligned


def test_gamma_of_any_sign_constant_rows_and_extreme_values():
    rng = np.random.default_rng(10)
    x, gamma, beta = _case(rng, 80, 256)
    gamma[::3] *= -1
    gamma[7] = 0.0
    x[3, :] = 1.75                            # constant row
    x[4, :] = 0.0
    x[5, :] *= 1e18                           # squares overflow to inf on both sides alike
    x[6, :] *= 1e-20                          # squares underflow
    x[8, 17] = np.inf
    x[9, 0] = np.nan                          # every comparison false from there on
    # deviations outside the range in which the kernel replaces the division of Eq. 5 by a corrected
    # reciprocal multiply (it must notice and divide), and one row that mixes both regimes
    x[10, :] *= 1e37
    x[11, :] *= 1e-33
    x[12, :] *= 1e-41                         # subnormal inputs
    x[13, 40:] *= 1e-36
    x[14, :] = 3.0e-38
    x[14, 100] = 3.0000004e-38                # a subnormal deviation from an ordinary mean
    for eps in (0.0, 1e-5):
        _check(x, gamma, beta, eps, np.float32(0.3), 4)
    _check(x, gamma, beta, 1e-5, np.float32(0.02), 8)


def test_block_sized_input_sampled():
    """The benchmark's size (50,432 x 768): the whole matrix on the GPU, sampled rows by the oracle."""
    rng = np.random.default_rng(11)
    rows, cols = 256 * 197, 768
    x = torch.randn((rows, cols), generator=torch.Generator().manual_seed(5)).numpy()
    gamma = rng.uniform(0.5, 1.5, cols).astype(np.float32)
    beta = (rng.standard_normal(cols) * 0.3).astype(np.float32)
    out = vitq.QMat.empty(rows, cols, 4)
    vitq.vq_layernorm_quantize(dev(x), None, None, dev(gamma), dev(beta), 1e-5, 0.4, out)
    torch.cuda.synchronize()
    sample = np.r_[0:64, 25000:25064, rows - 64:rows]
    ref = vqo.layernorm_quantize(x[sample], gamma, beta, 1e-5, 0.4, 4)
    got = vqo.unpack(out.data.cpu().numpy()[sample], cols, 4)
    assert np.array_equal(got, ref["q"])


def test_bad_arguments_leave_output_untouched():
    out = vitq.QMat.empty(4, 8, 4)
    out.data.fill_(0x5A)
    x = torch.zeros((4, 8), device="cuda")
    g = torch.ones(8, device="cuda")
    for eps, step in ((-1.0, 0.5), (0.0, 0.0), (float("nan"), 0.5)):
        with pytest.raises(vitq.VitqError) as e:
            vitq.vq_layernorm_quantize(x, None, None, g, g, eps, step, out)
        assert e.value.status == vitq.STATUS_NAMES.index("VQ_ERR_STEP")
    torch.cuda.synchronize()
    assert torch.all(out.data == 0x5A)


def test_every_binary_exponent_of_the_input_scale():
    # one row per power of two from 2^-140 to 2^126: the kernel's division-free mean update is only
    # used while the deviations are ordinary numbers, and must hand over to the division outside
    # that range without a visible seam (both sides overflow and underflow alike)
    rng = np.random.default_rng(77)
    exps = np.arange(-140, 127)
    cols = 200
    base = rng.standard_normal((len(exps), cols)).astype(np.float32)
    with np.errstate(over="ignore", under="ignore"):
        x = (base.astype(np.float64) * np.exp2(exps.astype(np.float64))[:, None]).astype(np.float32)
    x[5, 10:60] = 0.0                          # exact zero deviations inside a tiny row
    x[200, 3] = x[200, 4]                      # a repeated value
    gamma = rng.uniform(0.5, 1.5, cols).astype(np.float32)
    beta = rng.normal(0, 0.3, cols).astype(np.float32)
    for eps in (0.0, 1e-6):
        _check(x, gamma, beta, eps, np.float32(0.4), 4)


@pytest.mark.parametrize("bits,gsign", [(4, 1.0), (4, -1.0), (8, 1.0), (3, 1.0)])
def test_values_planted_on_both_sides_of_every_guard_band(bits, gsign):
    """A guessed level stands without the comparator when it is provably far from a boundary.  beta is chosen
    per column so that one element of that column sits a chosen distance (2^-27 .. 2^-12 levels, either
    side) from a comparator boundary; every level must still be the oracle's."""
    rows, cols, eps = 64, 768, np.float32(1e-6)
    rng = np.random.default_rng(900 + bits)
    x, gamma, _ = _case(rng, rows, cols)
    gamma = (gamma * gsign).astype(np.float32)
    lo, hi = vqo.qrange(bits)
    step = np.float32(4.0 / hi)
    # Eq. 5 in fp32, element order, all rows at once (the statistics do not depend on beta)
    mu = np.zeros(rows, np.float32)
    m2 = np.zeros(rows, np.float32)
    for i in range(cols):
        d1 = x[:, i] - mu
        mu = mu + d1 / np.float32(i + 1)
        m2 = m2 + d1 * (x[:, i] - mu)
    V = (m2 + np.float32(cols) * eps).astype(np.float64)
    sigma = np.sqrt(V / cols)
    beta = np.zeros(cols, np.float32)
    for j in range(cols):
        r = j % rows
        g = np.float32(np.float32(x[r, j] - mu[r]) * gamma[j])
        k = int(rng.integers(lo + 1, hi + 1))
        delta = float(rng.choice([-1.0, 1.0])) * 2.0 ** float(rng.uniform(-27, -12))
        beta[j] = np.float32(float(step) * (k - 0.5 + delta) - float(g) / sigma[r])
    _check(x, gamma, beta, eps, step, bits)


@pytest.mark.parametrize("rows,cols", [(12288, 36), (12289, 36), (24576, 33), (24577, 32), (20, 4096), (20, 4128), (17, 4131),
                                       (16, 31), (33, 96)])
def test_rows_per_workgroup_chunk_edges_and_table_end(rows, cols):
    """The sizes at which the rows per workgroup change, rows that end on, before and after a 32-column
    chunk, and rows longer than the 4096-entry table of reciprocals (those steps divide)."""
    rng = np.random.default_rng(rows + 7 * cols)
    x, gamma, beta = _case(rng, rows, cols)
    _check(x, gamma, beta, 1e-6, np.float32(0.4), 4)


@pytest.mark.parametrize("cols", [64, 66])
def test_sum_in_place_and_sum_without_residual(cols):
    """sum_out may be x itself (the stream updated in place); without a residual it receives x."""
    rng = np.random.default_rng(cols)
    x, gamma, beta = _case(rng, 50, cols)
    beta[:8] = np.float32(0.4) * np.float32(0.5)          # elements on and near boundaries: the comparator path
    x[:, :8] = x[:, :1]
    res = rng.standard_normal((50, cols)).astype(np.float32)
    for r in (res, None):
        ref = vqo.layernorm_quantize(x, gamma, beta, 1e-6, np.float32(0.4), 4, res=r, want_sum=True)
        xd = dev(x)
        out = vitq.QMat.empty(50, cols, 4)
        vitq.vq_layernorm_quantize(xd, dev(r), xd, dev(gamma), dev(beta), 1e-6, 0.4, out)
        torch.cuda.synchronize()
        assert np.array_equal(from_qmat(out), ref["q"])
        assert np.array_equal(xd.cpu().numpy(), ref["sum"] if r is not None else x)


@pytest.mark.parametrize("stride", [1 << 32, (1 << 32) + 48])
def test_output_rows_more_than_four_gib_apart(stride):
    """The output stride is a 64-bit number of bytes: two rows 2^32 bytes apart and further."""
    rng = np.random.default_rng(32)
    x, gamma, beta = _case(rng, 2, 96)
    out = vitq.QMat.empty(2, 96, 4, row_stride=stride)
    out.data[:, :64].fill_(0xFF)
    vitq.vq_layernorm_quantize(dev(x), None, None, dev(gamma), dev(beta), 1e-6, 0.4, out)
    torch.cuda.synchronize()
    want = vqo.pack(vqo.layernorm_quantize(x, gamma, beta, 1e-6, np.float32(0.4), 4)["q"], 4)
    got = out.data[:, :64].cpu().numpy()
    assert np.array_equal(got[:, :48], want[:, :48])
    assert (got[:, 48:] == 0xFF).all()                    # nothing beyond the padded row


def test_more_rows_than_one_grid_holds():
    """A grid holds at most 2^32 - 1 work-items, i.e. 613,566,720 rows in workgroups of 448 for 64 rows: a
    longer matrix is dealt to several launches.  Rows at the start, around that edge and at the end by
    the oracle; every row's padding shows that it was written."""
    edge = (2 ** 32 - 1) // 448 * 64
    rows, cols = edge + 1000, 4
    gen = torch.Generator(device="cuda")
    gen.manual_seed(6)
    x = torch.randn((rows, cols), generator=gen, device="cuda")
    rng = np.random.default_rng(6)
    _, gamma, beta = _case(rng, 1, cols)
    out = vitq.QMat(torch.full((rows, 16), 0xFF, dtype=torch.uint8, device="cuda"), cols, 4, 4)
    vitq.vq_layernorm_quantize(x, None, None, dev(gamma), dev(beta), 1e-6, 0.4, out)
    torch.cuda.synchronize()
    for lo, hi in ((0, 100), (edge - 100, edge + 100), (rows - 100, rows)):
        ref = vqo.layernorm_quantize(x[lo:hi].cpu().numpy(), gamma, beta, 1e-6, np.float32(0.4), 4)
        assert np.array_equal(out.data[lo:hi].cpu().numpy(), vqo.pack(ref["q"], 4))
    assert int(out.data[:, 2:].view(torch.int16).count_nonzero()) == 0


@pytest.mark.parametrize("rows,cols", [(20, 768), (12289, 64), (24577, 260)])
@pytest.mark.parametrize("off", [1, 2, 3])
def test_gamma_and_beta_at_any_float_address(rows, cols, off):
    """Parameters that are slices of a flat buffer: 4, 8 and 12 bytes past a 16-byte boundary, with aligned rows."""
    rng = np.random.default_rng(rows + off)
    x, gamma, beta = _case(rng, rows, cols)
    flat = torch.zeros(2 * cols + 8, device="cuda")
    gd, bd = flat[off:off + cols], flat[off + cols + 1:off + 2 * cols + 1]
    gd.copy_(dev(gamma))
    bd.copy_(dev(beta))
    out = vitq.QMat.empty(rows, cols, 4)
    vitq.vq_layernorm_quantize(dev(x), None, None, gd, bd, 1e-6, 0.4, out)
    torch.cuda.synchronize()
    assert np.array_equal(from_qmat(out), vqo.layernorm_quantize(x, gamma, beta, 1e-6, np.float32(0.4), 4)["q"])


@pytest.mark.parametrize("bits", [2, 4, 8])
@pytest.mark.parametrize("rows", [1, 57, 12300, 24600])           # one per rows-per-workgroup, whole and cut short
@pytest.mark.parametrize("cols", [1, 16, 33, 65, 100, 128, 129])
def test_short_rows_side_by_side(rows, cols, bits):
    """Rows of up to 128 columns stay in LDS and a wave decides 2 to 16 of them at once: every number of lanes
    per row (16, 32, 64 and 128 padded columns), the first longer rows, columns on a boundary (gamma 0)
    that go through the comparator, residual and sum in place."""
    rng = np.random.default_rng(rows + 1000 * cols + bits)
    x, gamma, beta = _case(rng, rows, cols)
    step = np.float32(2.5 / vqo.qrange(bits)[1])
    gamma[::5], beta[::5] = 0.0, step * np.float32(0.5)
    _check(x, gamma, beta, 1e-6, step, bits)
    res = rng.standard_normal((rows, cols)).astype(np.float32)
    ref = vqo.layernorm_quantize(x, gamma, beta, 1e-6, step, bits, res=res, want_sum=True)
    xd = dev(x)
    out = vitq.QMat.empty(rows, cols, bits)
    out.data.fill_(0xFF)
    vitq.vq_layernorm_quantize(xd, dev(res), xd, dev(gamma), dev(beta), 1e-6, step, out)
    torch.cuda.synchronize()
    assert np.array_equal(out.data.cpu().numpy(), vqo.pack(ref["q"], storage_of(bits)))
    assert np.array_equal(xd.cpu().numpy(), ref["sum"])


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("cols", [132, 384, 388, 500, 768, 772, 1152, 1156])      # pieces per lane, chunk ends, the longest row
@pytest.mark.parametrize("rows", [3, 197, 1025])
def test_rows_that_stay_in_registers(rows, cols, bits):
    """Rows of up to 1152 columns held by the loading waves: whole and partial chunks, workgroups cut short, a row of every
    kind that leaves the fast paths (tiny, huge, constant, not finite), columns on a boundary (the comparator)."""
    rng = np.random.default_rng(rows + 1000 * cols + bits)
    x, gamma, beta = _case(rng, rows, cols)
    step = np.float32(2.5 / vqo.qrange(bits)[1])
    gamma[::7], beta[::7] = 0.0, step * np.float32(0.5)
    x[0, cols - 1] = 1e4
    x[1] *= 1e-36
    x[2] = 0.75
    if rows > 100:
        x[60], x[77, 33], x[90, 1:] = x[60] * 1e37, np.nan, 0.0
    _check(x, gamma, beta, 1e-6, step, bits)


@pytest.mark.parametrize("rows,cols", [(4096, 132), (4097, 260), (8192, 196), (8193, 132), (16384, 132), (16385, 132)])
def test_rows_per_workgroup_of_the_one_round_form(rows, cols):
    """The sizes at which its lanes per walking wave change (16, 32, 64 rows per CU) and where it ends, rows at any distance."""
    rng = np.random.default_rng(rows + cols)
    x, gamma, beta = _case(rng, rows, cols)
    _check(x, gamma, beta, 1e-6, np.float32(0.4), 4)
    _check(x, gamma, beta, 0.0, np.float32(0.02), 8)
    big = torch.zeros((rows, cols + 12), device="cuda")
    big[:, :cols] = dev(x)
    out = vitq.QMat.empty(rows, cols, 4, row_stride=(cols // 2 + 15) // 16 * 16 + 32)
    out.data.fill_(0x5A)
    vitq.vq_layernorm_quantize(big[:, :cols], None, None, dev(gamma), dev(beta), 1e-6, 0.4, out)
    torch.cuda.synchronize()
    row_bytes = (cols // 2 + 15) // 16 * 16
    got = out.data.cpu().numpy()
    want = vqo.pack(vqo.layernorm_quantize(x, gamma, beta, 1e-6, np.float32(0.4), 4)["q"], 4)
    assert np.array_equal(got[:, :row_bytes], want[:, :row_bytes]) and (got[:, row_bytes:] == 0x5A).all()


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("rows,cols", [
    (4200, 388), (8192, 768), (5000, 772), (8192, 1152),          # up to 32 rows per workgroup, each number of pieces per lane
    (8200, 260), (16384, 384), (12608, 768), (16384, 500), (9000, 1000), (16384, 1152),       # up to 64
])
def test_rows_that_stay_in_registers_many_per_workgroup(rows, cols, bits):
    """The forms whose walking wave holds more than 16 rows: workgroups from the first to the last by the oracle, with rows of every
    kind that leaves the fast paths in lanes past 16 and 32, columns on a boundary, bytes past the row untouched."""
    rng = np.random.default_rng(rows + 1000 * cols + bits)
    x, gamma, beta = _case(rng, rows, cols)
    hi, sa = vqo.qrange(bits)[1], storage_of(bits)
    step = np.float32(2.5 / hi)
    gamma[::7], beta[::7] = 0.0, step * np.float32(0.5)
    per = -(-rows // 256)                                          # rows of a workgroup
    for first in (0, 100 * per):
        x[first + per - 1] *= 1e-36
        x[first + per - 2, cols - 1] = 1e4
        x[first + per - 3] = 0.75
        x[first + per // 2], x[first + per // 2 + 1, 33], x[first + per // 2 + 2, 1:] = x[first + per // 2] * 1e37, np.nan, 0.0
    row_bytes = (cols * sa // 8 + 15) // 16 * 16
    out = vitq.QMat.empty(rows, cols, bits, row_stride=row_bytes + 16)
    out.data.fill_(0x5A)
    xd, gd, bd = dev(x), dev(gamma), dev(beta)
    vitq.vq_layernorm_quantize(xd, None, None, gd, bd, 1e-6, step, out)
    torch.cuda.synchronize()
    got = out.data.cpu().numpy()
    last = (rows - 1) // per * per
    at = np.unique(np.r_[0:2 * per, 100 * per:101 * per, last - per:rows, rng.integers(0, rows, 150)])
    want = vqo.pack(vqo.layernorm_quantize(x[at], gamma, beta, 1e-6, step, bits)["q"], sa)
    assert np.array_equal(got[at, :row_bytes], want[:, :row_bytes]) and (got[:, row_bytes:] == 0x5A).all()
