"""GPU parity: vq_linear_absorbed (integer-only linear + quantizer: equivalent bias in the integer
domain, scales absorbed into the comparator references) against the CPU oracle, bit-exact."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from oracle import vqo
from paper_2504_18547_amd import vitq
from tests.gpu_util import dev, from_qmat, to_qmat


def _operands(seed, M, K, Nout, bits_w, bits_a):
    rng = np.random.default_rng(seed)
    lo_a, hi_a = vqo.qrange(bits_a)
    lo_w, hi_w = vqo.qrange(bits_w)
    xq = rng.integers(lo_a, hi_a + 1, size=(M, K)).astype(np.int8)
    wq = rng.integers(lo_w, hi_w + 1, size=(Nout, K)).astype(np.int8)
    s_w = rng.uniform(0.002, 0.02, Nout).astype(np.float32)
    bias = rng.normal(0, 0.05, Nout).astype(np.float32)
    return xq, wq, s_w, bias


def _run(xq, wq, b_int, thr, bits_w, bits_a, bits_y, want_acc=True, sum_may_leave_int32=False):
    M, Nout = xq.shape[0], wq.shape[0]
    xd, wd = to_qmat(xq, bits_a), to_qmat(wq, bits_w)
    out = vitq.QMat.empty(M, Nout, bits_y, storage_bits=4 if bits_y <= 4 else 8)   # 2-bit levels in 4-bit fields
    out.data.fill_(0xFF)
    acc = torch.full((M, Nout), -7, dtype=torch.int32, device="cuda") if want_acc else None
    bd = None if b_int is None else torch.from_numpy(np.ascontiguousarray(b_int)).cuda()
    td = torch.from_numpy(np.ascontiguousarray(thr)).cuda()
    vitq.vq_linear_absorbed(xd, wd, bd, td, acc, out)
    torch.cuda.synchronize()
    ref = vqo.linear_absorbed(xq, wq, b_int, thr, bits_y)
    assert sum_may_leave_int32 or ref["overflow"] == 0
    got = from_qmat(out)
    assert np.array_equal(got, ref["yq"]), "levels differ at %d of %d" % ((got != ref["yq"]).sum(), got.size)
    assert np.array_equal(out.data.cpu().numpy(), vqo.pack(ref["yq"], out.storage_bits))
    if want_acc:
        assert np.array_equal(acc.cpu().numpy(), ref["acc"])
    return ref


@pytest.mark.parametrize("bits_w,bits_a,bits_y,M,K,Nout", [
    (4, 4, 4, 300, 200, 48),        # ragged token tile, K tail, one partial channel tile
    (4, 4, 4, 591, 768, 768),       # the projection of three ViT-B images
    (4, 4, 3, 130, 384, 144),
    (4, 4, 2, 64, 96, 16),
    (3, 3, 3, 197, 384, 384),
    (2, 4, 4, 77, 160, 32),
    (8, 8, 8, 150, 320, 64),        # 255 references per channel: read from global memory
    (8, 8, 4, 129, 64, 160),
    (4, 4, 8, 40, 128, 32),
    (8, 8, 6, 70, 128, 32),         # 63 references: both levels of the two-level table end early
    (4, 4, 5, 33, 256, 48),         # 31 references
    (8, 8, 7, 20, 64, 16),          # 127 references
    (4, 4, 4, 2177, 600, 2048),     # 288 small tiles, 144 large: an even deal, 128x256, five k-stages and a tail
    (4, 4, 8, 2177, 600, 2048),     # the same with 255 references
    (4, 4, 8, 4249, 72, 2064),      # 255 references, 578 small tiles, 289 large: three units against four, 128x128
    (4, 4, 6, 4249, 72, 2064),      # the same with 63 references
    (4, 4, 8, 200, 400, 48),        # one small tile per CU, 128x128
    (4, 4, 8, 513, 96, 4096),       # 160 of them
])
def test_against_oracle(bits_w, bits_a, bits_y, M, K, Nout):
    xq, wq, s_w, bias = _operands(1000 + M + bits_y, M, K, Nout, bits_w, bits_a)
    s_x = np.float32(0.05)
    acc_std = float(np.std(xq.astype(np.int64) @ wq.astype(np.int64).T * (s_x * s_w)[None, :]))
    lo, hi = vqo.qrange(bits_y)
    s_y = np.float32(2.5 * acc_std / hi)                           # levels spread over the whole range
    b_int, thr = vitq.vq_absorb_thresholds(s_x, s_w, bias, [s_y], bits_y)
    b_ref, thr_ref = vqo.absorb(s_x, s_w, bias, s_y, bits_y)
    assert np.array_equal(b_int, b_ref) and np.array_equal(thr, thr_ref)
    ref = _run(xq, wq, b_int, thr, bits_w, bits_a, bits_y)
    assert len(np.unique(ref["yq"])) >= min(hi - lo + 1, 12) - 2


def test_no_bias_and_per_channel_output_steps():
    xq, wq, s_w, _ = _operands(5, 100, 256, 96, 4, 4)
    s_y = np.random.default_rng(6).uniform(0.02, 0.4, 96).astype(np.float32)
    b_int, thr = vitq.vq_absorb_thresholds(0.05, s_w, None, s_y, 4)
    assert not b_int.any()
    _run(xq, wq, None, thr, 4, 4, 4, want_acc=False)


def test_irregular_reference_tables():
    # references that are far from equally spaced, repeated, or saturated: the count must still be exact
    xq, wq, _, _ = _operands(9, 200, 128, 32, 4, 4)
    rng = np.random.default_rng(10)
    thr = np.sort(rng.integers(-900, 900, size=(32, 15)), axis=1).astype(np.int32)
    thr[0, :] = 17                                   # all equal
    thr[1, :5] = -2 ** 31
    thr[1, 5:] = 2 ** 31 - 1                         # five always exceeded (but by INT32_MIN), ten never
    thr[2, :] = np.sort(np.r_[rng.integers(-5, 5, 14), 100000]).astype(np.int32)   # one far outlier
    thr[3, :] = np.arange(15) - 7                    # unit spacing around zero
    thr[4, 7:] = thr[4, 7]                           # upper half collapsed
    b_int = rng.integers(-50, 50, 32).astype(np.int32)
    ref = _run(xq, wq, b_int, thr, 4, 4, 4)
    assert set(np.unique(ref["yq"][:, 0])) <= {-8, 7}
    assert np.all(ref["yq"][:, 1] == -3)


@pytest.mark.parametrize("bits_w,bits_a,bits_y,M,Nout", [
    (4, 4, 4, 300, 272), (4, 4, 3, 130, 144), (2, 4, 4, 130, 144), (8, 8, 4, 130, 144), (4, 4, 2, 40, 16)])
def test_evenly_spaced_references_and_where_that_ends(bits_w, bits_a, bits_y, M, Nout):
    """Tables with a constant spacing, sums on and next to the references; then one channel of the first tile at every bound
    of what counts as even: the spacing, a reference off its place, the distance from the bias, the first one far away."""
    xq, wq, _, _ = _operands(31 + Nout, M, 160, Nout, bits_w, bits_a)
    rng = np.random.default_rng(32)
    n = (1 << bits_y) - 1
    wide = 8 if bits_a == 8 else 1
    gaps = rng.choice([4, 5, 16, 37, 60], Nout) * wide
    b_int = rng.integers(-50, 50, Nout).astype(np.int32)
    thr = ((np.arange(n)[None, :] - n // 2) * gaps[:, None] + rng.integers(-9, 9, Nout)[:, None]).astype(np.int32)
    sums = xq.astype(np.int64) @ wq.astype(np.int64).T + b_int
    for c in range(0, Nout, 5):
        thr[c] += np.int32(sums[c % M, c] - thr[c, c % n])             # a reference that some sum equals
    _run(xq, wq, b_int, thr, bits_w, bits_a, bits_y)
    up = np.arange(n)
    for channel in (up * 3, up * 4 + (up == 1), up * 8 + 3 * (up == 1), up * 8 + 4 * (up == 1), up * 16 - 7 * (up == n // 2),
                    2 ** 22 - 9 * n + up * 8, 2 ** 22 - 7 * n + up * 8, 2 ** 20 - 7 * n + up * 8, -2 ** 22 - 1 + up * 8,
                    2 ** 31 - 1 - up[::-1] * 8, -2 ** 31 + up * 8, -2 ** 22 + up * (2 ** 23 // n)):
        some = thr.copy()
        some[7] = np.asarray(channel, np.int64).astype(np.int32)
        _run(xq, wq, b_int, some, bits_w, bits_a, bits_y)


@pytest.mark.parametrize("bits_w,bits_a,bits_y", [(4, 4, 4), (8, 8, 4), (2, 4, 4), (4, 4, 3), (4, 4, 2)])
def test_one_reference_off_its_place_is_seen_wherever_it_is(bits_w, bits_a, bits_y):
    """Evenly spaced tables but for one reference, at every place of the row and in channels all over the tile: nearer to a
    neighbour's place than to its own, so that a count taken from the even spacing would be wrong for sums beside it."""
    M, K, Nout = 200, 160, 144
    xq, wq, _, _ = _operands(77 + bits_y, M, K, Nout, bits_w, bits_a)
    n = (1 << bits_y) - 1
    b_int = np.random.default_rng(78).integers(-50, 50, Nout).astype(np.int32)
    std = float(np.std(xq.astype(np.int64) @ wq.astype(np.int64).T))
    gap = max(16, int(2.5 * std) * 2 // n)
    even = np.tile(((np.arange(n) - n // 2) * gap).astype(np.int32), (Nout, 1))
    _run(xq, wq, b_int, even, bits_w, bits_a, bits_y, want_acc=False)
    for at in range(n):
        for side in (-1, 1):
            thr = even.copy()
            thr[(37 * at + (64 if side > 0 else 0)) % Nout, at] += side * (gap * 3 // 4)
            _run(xq, wq, b_int, thr, bits_w, bits_a, bits_y, want_acc=False)


@pytest.mark.parametrize("bits_w,bits_a,bits_y,K,sign", [(8, 8, 4, 1024, -1), (8, 8, 4, 1024, 1), (8, 8, 3, 1024, -1), (4, 4, 4, 65536, -1),
                                                         (2, 4, 4, 65536, 1), (2, 4, 3, 65536, -1)])
def test_narrowest_even_references_far_from_the_bias(bits_w, bits_a, bits_y, K, sign):
    """Where the rounding of the nearest reference's index is largest: spacings from 4 on that are no dyadic numbers, references as
    far off their places as still counts as even, as far from the bias as they may be, a sum at every integer between them."""
    n, tail, M, Nout = (1 << bits_y) - 1, 9, 128, 128
    reach = 2 ** 20 if bits_w == 2 else 2 ** 22
    lo_a, hi_a = vqo.qrange(bits_a)
    lo_w, _ = vqo.qrange(bits_w)
    rng = np.random.default_rng(K + bits_w + bits_y)
    x = np.zeros((M, K), np.int64)
    x[:, :tail] = np.arange(-M // 2, M // 2)[:, None] // tail                # consecutive sums from token to token
    x[:, :tail] += np.arange(tail)[None, :] < (np.arange(-M // 2, M // 2) % tail)[:, None]
    w = np.full((Nout, K), lo_w)
    w[:, :tail] = 1
    full = min((reach - 512) // (-lo_w * max(-lo_a, hi_a)), K - tail - 1)
    x[:, tail:tail + full] = lo_a if sign > 0 else hi_a
    sums = x[:, :tail].sum(1) + lo_w * int(x[0, tail:].sum())
    assert np.array_equal(np.diff(sums), np.ones(M - 1)) and abs(sums).max() < reach and abs(sums).min() > 0.7 * reach
    b_int = rng.integers(-900, 900, Nout)
    thr = np.empty((Nout, n), np.int64)
    for c in range(Nout):
        width = int(rng.integers(4 * (n - 1), 4 * (n - 1) + 4))
        at = np.arange(n) * width / (n - 1)
        off = rng.choice([-0.375, 0.375, 0.0], n) * width / (n - 1)
        ref = np.where(off < 0, np.ceil(at + off), np.floor(at + off))
        ref[0], ref[-1] = 0, width
        assert (abs(ref - at) <= 0.375 * width / (n - 1)).all() and (np.diff(ref) >= 0).all()
        thr[c] = sums[0] + int(rng.integers(2, M - 2 - width)) + ref + b_int[c]
    ref = _run(x.astype(np.int8), w.astype(np.int8), b_int.astype(np.int32), thr.astype(np.int32), bits_w, bits_a, bits_y)
    assert len(np.unique(ref["yq"])) == n + 1


def test_equivalent_bias_at_the_int32_limits():
    """b_int is clamped to int32 by the preparation step, so a near-dead channel carries INT32_MAX or
    INT32_MIN; the sum with an accumulator of the same sign then leaves 32 bits, and the oracle
    compares it in 64 bits.  Accumulators of both signs, references at and next to the limits."""
    xq, wq, _, _ = _operands(21, 160, 192, 48, 4, 4)
    rng = np.random.default_rng(22)
    thr = np.sort(rng.integers(-3000, 3000, size=(48, 15)), axis=1).astype(np.int32)
    b_int = rng.integers(-50, 50, 48).astype(np.int32)
    imax, imin = 2 ** 31 - 1, -2 ** 31
    b_int[0], thr[0, :] = imax, imax                     # exceeded only by sums above INT32_MAX
    b_int[1], thr[1, :] = imin, imin                     # exceeded unless the sum is INT32_MIN or below
    b_int[2], thr[2, :] = imax, np.sort(np.r_[np.full(8, imax - 1), np.full(7, imax)])
    b_int[3], thr[3, :] = imin, np.sort(np.r_[np.full(5, imin), np.full(10, imin + 40)])
    b_int[4], thr[4, :] = imax - 1000, imax - np.arange(15)[::-1] * 150
    b_int[5], thr[5, :] = imin + 1000, imin + np.arange(15) * 150
    b_int[17], thr[17, :] = imax, np.sort(rng.integers(-3000, 3000, 15))   # ordinary references, huge bias
    b_int[33], thr[33, :] = imin, np.sort(rng.integers(-3000, 3000, 15))
    ref = _run(xq, wq, b_int, thr, 4, 4, 4, sum_may_leave_int32=True)
    acc = ref["acc"]
    assert (acc[:, 0] > 0).any() and (acc[:, 0] < 0).any()                 # both signs meet the limits
    assert len(np.unique(ref["yq"][:, 0])) == 2 and len(np.unique(ref["yq"][:, 1])) == 2
    assert np.all(ref["yq"][:, 17] == 7) and np.all(ref["yq"][:, 33] == -8)
    # the same through the two-level table of more than fifteen references per channel
    thr8 = np.sort(rng.integers(-3000, 3000, size=(48, 255)), axis=1).astype(np.int32)
    thr8[0, :], thr8[1, :] = imax, imin
    thr8[2, :128], thr8[2, 128:] = imax - 1, imax
    _run(xq, wq, b_int, thr8, 4, 4, 8, sum_may_leave_int32=True)


@pytest.mark.parametrize("bits_w,bits_a,bits_y,K", [
    (8, 8, 4, 1024), (8, 8, 8, 1024), (8, 8, 4, 65536), (8, 8, 8, 65536), (4, 4, 4, 65536), (4, 4, 8, 65536), (2, 4, 4, 65536)])
def test_largest_accumulators_with_biases_near_the_int32_limits(bits_w, bits_a, bits_y, K):
    """Accumulators of both signs up to the largest that the operands allow (2^30 with 8-bit pairs of 65,536 values), beside
    biases at distances from the limits from which the sum leaves 32 bits or just does not."""
    M, Nout = 40, 80
    lo_a, hi_a = vqo.qrange(bits_a)
    lo_w, hi_w = vqo.qrange(bits_w)
    rng = np.random.default_rng(K + bits_w + bits_y)
    xq = rng.integers(lo_a, hi_a + 1, size=(M, K)).astype(np.int8)
    wq = rng.integers(lo_w, hi_w + 1, size=(Nout, K)).astype(np.int8)
    xq[0], xq[1], xq[2, : K // 2], xq[33] = lo_a, hi_a, lo_a, lo_a
    wq[::2] = lo_w
    wq[1::4] = hi_w
    imax, imin = 2 ** 31 - 1, -2 ** 31
    n = (1 << bits_y) - 1
    for near in (1, 2 ** 20, 2 ** 22, 3 * 2 ** 22, 2 ** 24, 3 * 2 ** 28, 2 ** 30):     # (one distance for all channels of a tile)
        off = rng.integers(near - 1, near + 2, Nout)
        b_int = np.where(np.arange(Nout) & 2, imax - off, imin + off).astype(np.int32)
        thr = np.sort(rng.integers(-3000, 3000, size=(Nout, n)), axis=1).astype(np.int32)
        at_limit = np.clip(b_int[:, None].astype(np.int64) + np.sort(rng.integers(-2 ** 30, 2 ** 30, (Nout, n)), axis=1), imin, imax)
        thr[6::3] = at_limit[6::3]
        thr[7], thr[8] = imax, imin
        ref = _run(xq, wq, b_int, thr, bits_w, bits_a, bits_y, sum_may_leave_int32=True)
        assert (ref["overflow"] > 0) == (near <= K << (bits_w + bits_a - 2)) and set(vqo.qrange(bits_y)) <= set(np.unique(ref["yq"]))
        spaced = np.clip(b_int.astype(np.int64), imin + 2 ** 20, imax - 2 ** 20)[:, None] + 16 * (np.arange(n) - n // 2)
        _run(xq, wq, b_int, spaced.astype(np.int32), bits_w, bits_a, bits_y, sum_may_leave_int32=True)


def test_argument_errors():
    xq, wq, s_w, bias = _operands(3, 8, 64, 24, 4, 4)       # 24 output channels: not a multiple of 16
    b_int, thr = vitq.vq_absorb_thresholds(0.05, s_w, bias, [0.1], 4)
    xd, wd = to_qmat(xq, 4), to_qmat(wq, 4)
    out = vitq.QMat.empty(8, 24, 4)
    td = torch.from_numpy(thr).cuda()
    with pytest.raises(vitq.VitqError) as e:
        vitq.vq_linear_absorbed(xd, wd, None, td, None, out)
    assert e.value.status == vitq.STATUS_NAMES.index("VQ_ERR_UNSUPPORTED")
    with pytest.raises(vitq.VitqError) as e:
        vitq.vq_linear_absorbed(xd, wd, None, None, None, out)
    assert e.value.status == vitq.STATUS_NAMES.index("VQ_ERR_NULL")
    with pytest.raises(vitq.VitqError) as e:
        vitq.vq_absorb_thresholds(0.05, s_w, bias, [0.0], 4)
    assert e.value.status == vitq.STATUS_NAMES.index("VQ_ERR_STEP")
