"""fp32 scoring: rows split into three bf16 parts against 64-bit results, at the edges of the split."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_08373_amd as lib
    lib.load_library()
    return lib


def raw_scores(S, q, k, n_window, sm_scale, reduce="sum"):
    """Raw scores [Hkv, n] of one layer and one sequence."""
    hkv, n = k.shape[2], k.shape[1]
    p = S.SpecKVParams.for_tensors(q, k, seq_lens=[n], n_window=n_window, pool_k=7, c_max=16, sm_scale=sm_scale, reduce=reduce)
    ws = torch.empty(S.workspace_bytes(p), dtype=torch.uint8, device="cuda")
    out = torch.full((2, 1, hkv * n), -1.0, dtype=torch.float32, device="cuda")
    S.speckv_score(p, q, k, out[0], out[1], ws)
    return out[1].view(hkv, n)


def exact_scores(q, k, n_window, sm_scale, reduce="sum"):
    rows, hq = q.shape[2], q.shape[3]
    n, hkv = k.shape[1], k.shape[2]
    m, group = n - n_window, hq // hkv
    row = torch.arange(rows, device="cuda")
    last = torch.where(row < n_window, m + row, torch.full_like(row, n - 1))
    hidden = torch.arange(n, device="cuda")[None, :] > last[:, None]
    ref = torch.zeros(hkv, n, dtype=torch.float64, device="cuda")
    for h in range(hq):
        logits = (q[0, 0, :, h].double() @ k[0, :, h // group].double().t()) * sm_scale
        p = torch.softmax(logits.masked_fill(hidden, -math.inf), dim=1)
        ref[h // group] += p.sum(0) if reduce == "sum" else p.amax(0)
    return ref


def draw(seed, n, rows, hq, hkv, d):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    q = torch.randn(1, 1, rows, hq, d, generator=gen, device="cuda")
    return q, torch.randn(1, n, hkv, d, generator=gen, device="cuda"), gen


# one and several row blocks per wave, padded rows, chunks of one tile to several, tails of every kind
@pytest.mark.parametrize("d,group,rows,n", [(128, 1, 9, 130), (128, 4, 72, 1193), (128, 8, 33, 577), (64, 2, 17, 259),
                                            (64, 4, 128, 2077), (64, 7, 40, 700)])
@pytest.mark.parametrize("reduce", ["sum", "max"])
def test_every_product_of_the_parts_counts(S, d, group, rows, n, reduce):
    """One channel per query row is not zero, so a logit is one product of two 24-bit numbers of size up to
    40.  Allowed: the product left out (2^-34 of it), one rounding for each of the sums (2^-24 for the last
    one, together less than that for the lower ones), and the same again in the multiply-add of the
    softmax: below 40 * 8 * 2^-24 = 2e-5, in the numerator and in the normaliser, and 1e-6 for sums and
    exp2.  A missing product of the larger parts shows as 40 * 2^-17 = 3e-4."""
    q, k, gen = draw(5, n, rows, group * 2, 2, d)
    keep = torch.randint(0, d, (1, 1, rows, group * 2, 1), generator=gen, device="cuda")
    q = torch.where(torch.arange(d, device="cuda") == keep, 3 + q.abs() / 2, torch.zeros_like(q))
    k = k.clamp(-3, 3)
    scale = 40.0 / float(q.max() * 3)
    got, want = raw_scores(S, q, k, min(rows, 16), scale, reduce).double(), exact_scores(q, k, min(rows, 16), scale, reduce)
    assert ((got - want).abs() <= 4.1e-5 * want).all(), float(((got - want).abs() / want).max())


def test_scaling_by_powers_of_two_changes_no_bit(S):
    """Q * 2^e, K * 2^-e: the parts scale with the number, down to parts of 2^-121."""
    q, k, _ = draw(6, 900, 40, 4, 2, 128)
    k = torch.where(k.abs() < 2.0 ** -6, torch.zeros_like(k), k)
    base = raw_scores(S, q, k, 16, 128 ** -0.5)
    for e in (60, -60, 97):
        assert torch.equal(raw_scores(S, q * 2.0 ** e, k * 2.0 ** -e, 16, 128 ** -0.5), base), e


@pytest.mark.parametrize("d,group,n", [(128, 2, 700), (64, 8, 1100)])
def test_infinities_and_numbers_above_the_bf16_range(S, d, group, n):
    """Keys with an infinite channel against queries that are positive there get the score exp(-inf) = 0; numbers
    that bf16 rounds to infinity, and query channels that have zero parts, give finite products."""
    q, k, _ = draw(7, n, 64, group * 2, 2, d)      # whole row blocks: a zero row times an infinity is NaN in any product
    q[..., 3] = 2.0 ** -126                 # its two smaller parts are zero
    q[..., 5] = q[..., 5].abs() + 1.0
    far = [0, 31, 32, 63, 64, n // 2, n - 60, n - 20, n - 1]       # first and last blocks of tiles, chunk and tail
    k[0, far[::2], :, 3] = 3.4e38           # finite; the nearest bf16 number is infinity
    k[0, far[1::2], 0, 5] = -math.inf
    got, want = raw_scores(S, q, k, 16, d ** -0.5).double(), exact_scores(q, k, 16, d ** -0.5)
    assert (got[0, far[1::2]] == 0).all()
    assert ((got - want).abs() <= 1e-4 * want).all(), float(((got - want).abs() / want.clamp(min=1e-300)).max())


def test_nan_stays_with_its_head(S):
    q, k, _ = draw(8, 500, 24, 4, 2, 128)
    k[0, 77, 1, 9] = math.nan
    got = raw_scores(S, q, k, 16, 128 ** -0.5)
    assert torch.isnan(got[1]).any() and torch.isfinite(got[0]).all()
    want = exact_scores(q, k, 16, 128 ** -0.5)
    assert ((got[0].double() - want[0]).abs() <= 1e-4 * want[0]).all()


def logit_spread(S, q, k, sm_scale):
    """q [H, d], k [n, H, d], one row per head: by how much the logits that the raw scores stand for differ from
    64-bit ones, largest minus smallest per head (which cancels the normaliser), in 2^-24 of the head's largest."""
    n, H, d = k.shape
    p = S.SpecKVParams.for_tensors(q.view(1, 1, 1, H, d), k.view(1, n, H, d), seq_lens=[n], n_window=0, pool_k=1, c_max=16,
                                   sm_scale=sm_scale)
    ws = torch.empty(S.workspace_bytes(p), dtype=torch.uint8, device="cuda")
    out = torch.empty(2, 1, H * n, dtype=torch.float32, device="cuda")
    S.speckv_score(p, q.view(1, 1, 1, H, d), k.view(1, n, H, d), out[0], out[1], ws)
    to_log2 = float(torch.tensor(sm_scale, dtype=torch.float32) * torch.tensor(math.log2(math.e), dtype=torch.float32))
    want = (q.double() * k.double()).sum(-1).t() * to_log2
    err = out[1].view(H, n).double().log2() - want
    return float(((err.amax(1) - err.amin(1)) / (want.abs().amax(1) * 2.0 ** -24)).max())


def narrow(seed, n, H, d, channels):
    """Rows with `channels` non-zero channels in [1, 1.5) and keys in [1, 1.02): with sm_scale 72 / channels the
    logits are near 130 binary orders and differ by three at most, so a row's scores are all ordinary numbers."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    q = torch.zeros(H, d, device="cuda")
    q.scatter_(1, torch.rand(H, d, generator=gen, device="cuda").argsort(1)[:, :channels],
               1 + torch.rand(H, channels, generator=gen, device="cuda") / 2)
    q[0] = torch.where(q[0] != 0, 1 + 2.0 ** -8 - 2.0 ** -17, 0.0)       # both smaller parts as large as they can be
    k = 1 + torch.rand(n, H, d, generator=gen, device="cuda") * 0.02
    k[:64, 0] = 1 + 2.0 ** -8 - 2.0 ** -17
    return q, k


# In 2^-24 of a logit's size, either way: the leading products and their sums are exact here, the addition of the
# lower ones rounds once (1); the lower sum is below 2^-7 of the whole and rounded at that size by at most five
# matrix instructions per non-zero channel or group of 16 channels (0.04 each channel); the softmax's multiply-add
# ends near -11 (half a last place is 2^-21, 0.07 of the unit at 112 binary orders and more) and exp2 is
# good to one (0.03).
@pytest.mark.parametrize("channels,allowed", [(1, 2.3), (2, 2.4), (4, 2.6), (16, 2.9)])
@pytest.mark.parametrize("d", [64, 128])
def test_rows_with_few_channels_are_rounded_as_fp32_products(S, d, channels, allowed):
    q, k = narrow(11, 1024, 16, d, channels)
    assert logit_spread(S, q, k, 72.0 / channels) <= allowed


@pytest.mark.parametrize("e", [-96, -102, -104, -110, -117, -125])
def test_small_operands_keep_their_last_bits(S, e):
    """2^e times the same values on one side, 2^-e on the other: below 2^-103 three bf16 parts no longer hold them."""
    q, k = narrow(12, 512, 8, 128, 1)
    assert logit_spread(S, q * 2.0 ** e, k * 2.0 ** -e, 72.0) <= 2.4
    assert logit_spread(S, q * 2.0 ** -e, k * 2.0 ** e, 72.0) <= 2.4
    empty = torch.where(q == 0, 1.0, 0.0).argmax(1)                        # a channel that its row does not use
    q.scatter_(1, empty[:, None], 1.0)
    k.scatter_(2, empty.expand(512, 8)[..., None], 0.0)
    k[::97] = torch.where(k[::97] == 0, 2.0 ** e, k[::97])                 # some blocks hold such a number
    assert logit_spread(S, q, k, 72.0) <= 2.4


def test_small_products_keep_their_last_bits(S):
    """Logits of 2^-120 before sm_scale: their lower products lie below the smallest normal number."""
    q, k = narrow(13, 512, 8, 128, 1)
    assert logit_spread(S, q * 2.0 ** -60, k * 2.0 ** -60, 72.0 * 2.0 ** 120) <= 2.4
