"""Fused calls large enough to be pruned keep what the complete scores say: the best c_max keys by the library's own scores, which
other tests hold against the oracle.  The two ways add a row's sum in different orders (relative 1e-6), so that keys whose scores
are closer than TIE to the last kept one may change places."""
import math

import numpy as np
import pytest
import torch

from . import test_gpu_parity as parity

pytestmark = pytest.mark.gpu
TIE = 2e-5        # ten times the largest relative difference of two fp32 scores over logits of 10^2 (2e-6)


@pytest.fixture(scope="module")
def S():
    import paper_2506_08373_amd as S
    S.load_library()
    return S


def params(S, q, k, lens, n_window, c_max, **kw):
    return S.SpecKVParams.for_tensors(q, k, seq_lens=lens, n_window=n_window, pool_k=kw.pop("pool_k", 7), c_max=c_max,
                                      sm_scale=kw.pop("sm_scale", k.shape[-1] ** -0.5), **kw)


def rows_of(info, ws):
    """Keys listed, and 1 where every key was computed, of the output rows of the last call that had this workspace."""
    table = ws[info["rows_at"]:][:32 * info["n_rows"]].view(torch.int32).view(-1, 8)
    return table[:, 2], table[:, 3]


def sampled(info, keys):
    """The part of `keys` (dimension 0, whole periods of the sample) that the sample has."""
    period = info["tile_keys"] * info["sample_step"]
    whole = keys[:keys.shape[0] // period * period]
    return whole.view(-1, period, *keys.shape[1:])[:, :info["tile_keys"]]


def check(S, q, k, lens, n_window, c_max, ws=None, **kw):
    L, T, H, d = k.shape
    p = params(S, q, k, lens, n_window, c_max, **kw)
    assert S.prune_info(p)["pruned"]
    KT = S.total_keep(p)
    ws = parity.alloc_ws(S, p) if ws is None else ws
    pooled = torch.empty(L, H * T, device="cuda")
    idx = torch.full((L, H * KT), -7, dtype=torch.int32, device="cuda")
    k_out = torch.empty(L, H * KT, d, dtype=k.dtype, device="cuda")
    S.speckv_score(p, q, k, pooled, None, ws)
    for _ in range(2):                                   # the second one on the first one's workspace
        idx.fill_(-7)
        S.speckv_compress(p, q, k, None, idx, k_out, None, ws)
        t0 = keep0 = 0
        for n in lens:
            m, c = n - n_window, min(c_max, n - n_window)
            sc = pooled[:, H * t0:H * (t0 + n)].view(L, H, n)[..., :m]
            got = idx[:, H * keep0:H * (keep0 + c + n_window)].view(L, H, c + n_window).long()
            assert (got.diff(dim=-1) > 0).all() and (got[..., 0] >= 0).all()
            assert torch.equal(got[..., c:], torch.arange(m, n, device="cuda").expand(L, H, n_window))
            last = sc.topk(c, dim=-1).values[..., -1:]
            kept = torch.zeros(L, H, m, dtype=torch.bool, device="cuda").scatter_(-1, got[..., :c], True)
            assert not (kept & (sc < last * (1 - TIE))).any() and not (~kept & (sc > last * (1 + TIE))).any(), n
            rows = k[:, t0:t0 + n].permute(0, 2, 1, 3).gather(2, got[..., None].expand(-1, -1, -1, d))
            out = k_out[:, H * keep0:H * (keep0 + c + n_window)].view(L, H, c + n_window, d)
            assert torch.equal(rows.view(torch.int16), out.view(torch.int16))
            t0 += n
            keep0 += c + n_window
    return idx, pooled


def tensors(lens, n_layers, heads=8, group=4, rows=128, d=128, dtype=torch.bfloat16, gain=2.0, planted=16, seed=3):
    """Logits with a standard deviation of about `gain`, outlier channels, and keys aligned with query rows."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")
    q = torch.empty(n_layers, len(lens), rows, heads * group, d, dtype=dtype, device="cuda")
    k = torch.empty(n_layers, sum(lens), heads, d, dtype=dtype, device="cuda")
    for layer in range(n_layers):
        scale = torch.exp(r(heads, d) * 0.5)
        scale /= scale.pow(4).mean(-1, keepdim=True).pow(0.25)
        q[layer] = (r(len(lens), rows, heads * group, d) * scale.repeat_interleave(group, 0) * gain).to(dtype)
        kl = r(sum(lens), heads, d) * scale
        for x in torch.randint(0, sum(lens), (planted,), generator=g, device="cuda").tolist():
            kl[x] = 2.5 * q[layer, 0, x % rows, ::group].float() / gain
        k[layer] = kl.to(dtype)
    return q, k


@pytest.mark.parametrize("lens,n_layers,kw", [
    ([24832 + 65], 9, {}),                                              # one chunk a sequence, packed pairs of blocks
    ([24832 + 64], 9, {"reduce": "max"}),
    ([70001], 3, {"pool_k": 1}),                                        # longest sample step, several chunks
    ([9000, 30123, 700, 17999, 12289], 4, {"pool_k": 16}),              # short ones are all sample
    ([13000, 50001], 14, {"rows": 37, "pool_k": 4}),                     # blocks shared by waves beside whole ones
    ([40000], 9, {"rows": 67, "reduce": "max"}),                        # padded heads
    ([33000], 12, {"heads": 4, "group": 7}),                            # two super-blocks
    ([33000], 20, {"heads": 4, "group": 7, "rows": 45, "reduce": "max"}),
    ([65537], 10, {"rows": 41}),                                        # one row block a wave
    ([65537], 10, {"rows": 41, "reduce": "max"}),
    ([30001], 8, {"dtype": torch.float16, "c_max": 100}),
    ([30001], 14, {"c_max": 3700}),
    ([30001], 8, {"gain": 0.2}),                                        # flat attention
    ([30001], 8, {"gain": 12.0}),                                       # one key a row
    ([50001], 6, {"d": 64}),                                            # tiles of 256 keys
    ([50001], 6, {"d": 64, "reduce": "max", "gain": 0.7}),
    ([50001, 20000], 12, {"d": 64, "rows": 45, "gain": 1.0}),           # one row block a wave
    ([66450], 12, {"d": 64, "heads": 2, "rows": 96, "gain": 0.7}),
])
def test_pruned_calls_keep_what_complete_scores_say(S, lens, n_layers, kw):
    kw = dict(kw)
    shape = {x: kw.pop(x) for x in ("heads", "group", "rows", "d", "dtype", "gain") if x in kw}
    q, k = tensors(lens, n_layers, **shape)
    check(S, q, k, lens, 32, kw.pop("c_max", 512), **kw)


def test_rows_whose_sample_misleads_are_computed_whole(S):
    """The best keys of one layer lie in the sample, so that its threshold is too high for the others."""
    q, k = tensors([30001], 8, gain=1.0, planted=0)
    info = S.prune_info(params(S, q, k, [30001], 32, 512))
    sampled(info, k[3]).mul_(4)
    sampled(info, k[5]).mul_(1.5)
    ws = torch.empty(info["workspace_bytes"], dtype=torch.uint8, device="cuda")
    check(S, q, k, [30001], 32, 512, ws=ws)
    whole = rows_of(info, ws)[1].view(8, 8).sum(1)
    assert whole[3] == 8 and whole[[0, 1, 2, 4, 6, 7]].sum() == 0, whole


def test_heavy_keys_outside_the_sample(S):
    """Scores far above a row's reference overflow the sums of their segment, in more segments of one chunk than a list has."""
    q, k = tensors([30001], 8, gain=1.0, planted=0)
    info = S.prune_info(params(S, q, k, [30001], 32, 512))
    keys = [x for x in range(200, 29000, 700) if x // info["tile_keys"] % info["sample_step"]]
    period = info["tile_keys"] * info["sample_step"]
    segments = {(x // period * (info["sample_step"] - 1) + x // info["tile_keys"] % info["sample_step"] - 1) // 8
                for x in keys if x < info["chunk_keys"]}                        # of eight tiles each; a list has room for six
    assert len(segments) > 6
    for i, x in enumerate(keys):
        k[2, x] = 60.0 * q[2, 0, i % 8, ::4]                                    # eight rows of the same wavefront
    k[4, 779] = 60.0 * q[4, 0, 5, ::4]
    for layer, x, row in [(2, x, i % 8) for i, x in enumerate(keys)] + [(4, 779, 5)]:
        products = q[layer, 0, row, ::4].float()[:, None] * k[layer].float().transpose(0, 1)
        scores = products.sum(-1) * (128 ** -0.5 * math.log2(math.e))          # [head][key]
        seen = torch.logsumexp(sampled(info, scores.t()).reshape(-1, 8) * math.log(2), 0) / math.log(2)
        assert (scores[:, x] - seen).min() > 126 + 76 + 8                       # the sums' largest number, what exponents are lowered by, margin
    check(S, q, k, [30001], 32, 512)


@pytest.mark.parametrize("lens,n_layers,kw", [([30001], 9, {}), ([50001], 8, {"d": 64}), ([40000], 9, {"rows": 67, "reduce": "max"})])
def test_rows_of_keys_and_queries_apart_in_memory(S, lens, n_layers, kw):
    """Heads before tokens, every row with room behind it; segments left to the repair, gathered keys and rows by these strides."""
    kw = dict(kw)
    shape = {x: kw.pop(x) for x in ("rows", "d") if x in kw}
    q, k = tensors(lens, n_layers, gain=1.0, **shape)
    k[2, 777] = 40.0 * q[2, 0, 5, ::4]
    L, T, H, d = k.shape
    k2 = torch.full((L, H + 1, T, d + 24), float("nan"), dtype=k.dtype, device="cuda")[:, :H, :, :d].transpose(1, 2)
    q2 = torch.full((q.shape[1], L, q.shape[3], q.shape[2], d + 8), float("nan"), dtype=q.dtype, device="cuda")[..., :d].permute(1, 0, 3, 2, 4)
    k2.copy_(k)
    q2.copy_(q)
    assert torch.equal(check(S, q2, k2, lens, 32, 512, **kw)[0], check(S, q, k, lens, 32, 512, **kw)[0])


def test_more_sequences_than_the_plan_simulates(S):
    """Beyond 16 sequences of a length the chunks are made from an even spread; long and short ones in any order, some all sample."""
    lens = [6001 + 977 * ((7 * s) % 20) for s in range(20)] + [40, 130, 900, 3001]
    q, k = tensors(lens, 4, rows=96)
    info = S.prune_info(params(S, q, k, lens, 32, 256))
    assert info["n_chunks"] >= 22
    check(S, q, k, lens, 32, 256)
    check(S, q, k, lens, 32, 256, reduce="max")


def test_all_scores_alike(S):
    q, k = tensors([30001], 8)
    q.zero_()
    idx, _ = check(S, q, k, [30001], 32, 512)
    want = torch.cat([torch.arange(512), torch.arange(29969, 30001)]).to(idx)
    assert torch.equal(idx, want.expand(8, 8, -1).reshape(8, -1))


def test_numbers_that_are_none(S):
    """Scores of heads with such numbers need not be numbers; the other heads' are what they are without them."""
    q, k = tensors([30001], 8)
    clean, _ = check(S, q, k, [30001], 32, 512)
    k[1, 5000, 2] = float("nan")
    k[3, 7000, 4, 5] = float("inf")
    p = params(S, q, k, [30001], 32, 512)
    idx = torch.empty_like(clean)
    k_out = torch.empty(8, idx.shape[1], 128, dtype=k.dtype, device="cuda")
    S.speckv_compress(p, q, k, None, idx, k_out, None, parity.alloc_ws(S, p))
    same = (idx.view(64, -1) == clean.view(64, -1)).all(-1)
    assert same[[i for i in range(64) if i not in (10, 28)]].all()
    odd = idx.view(64, -1)[[10, 28]]
    assert (odd.diff(dim=-1) > 0).all() and (odd[:, 0] >= 0).all()
    assert torch.equal(odd[:, 512:], torch.arange(30001 - 32, 30001, device="cuda").to(idx).expand(2, 32))


def test_a_workspace_without_room_for_it_is_enough(S):
    q, k = tensors([24897], 9)
    size = S.prune_info(params(S, q, k, [24897], 32, 512))["workspace_bytes"]
    for room in (size, size - 1):
        check(S, q, k, [24897], 32, 512, ws=torch.empty(room, dtype=torch.uint8, device="cuda"))


def test_captured_and_replayed_on_other_inputs(S):
    q, k = tensors([24897], 9)
    p = params(S, q, k, [24897], 32, 512)
    ws = parity.alloc_ws(S, p)
    idx = torch.empty(9, 8 * S.total_keep(p), dtype=torch.int32, device="cuda")
    k_out = torch.empty(9, idx.shape[1], 128, dtype=k.dtype, device="cuda")
    S.speckv_compress(p, q, k, None, idx, k_out, None, ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        S.speckv_compress(p, q, k, None, idx, k_out, None, ws)
    for seed in (4, 5, 6):
        q2, k2 = tensors([24897], 9, seed=seed, gain=float(seed - 3))
        q.copy_(q2), k.copy_(k2)
        graph.replay()
        got = idx.clone()
        S.speckv_compress(p, q, k, None, idx, k_out, None, ws)
        assert torch.equal(got, idx)


@pytest.mark.parametrize("n,n_layers,top_k,kw", [
    (60000, 12, 2048, {"d": 64, "rows": 64, "gain": 3.0}),
    (24000, 20, 1000, {"d": 64, "rows": 65, "gain": 2.0}),               # ranked by one workgroup; blocks shared by waves
    (90001, 13, 8000, {"d": 128, "rows": 33, "dtype": torch.float16}),
    (60000, 20, 8000, {"d": 64, "rows": 64, "gain": 0.02}),              # scores much alike: most keys listed
])
def test_prompt_tokens_are_those_of_complete_scores(S, n, n_layers, top_k, kw):
    q, k = tensors([n], n_layers, planted=200, **kw)
    p = params(S, q, k, [n], 32, 512)
    ids = torch.arange(n, dtype=torch.int32, device="cuda") * 3
    got = []
    most = S.prune_info(p, "tokens", top_k)["workspace_bytes"]
    assert most > 0
    for size in (most, most - 1, most):                                           # (no room for pruning in the second)
        out = [torch.full((n,), -7, dtype=torch.int32, device="cuda") for _ in range(2)] + [torch.zeros(1, dtype=torch.int32, device="cuda")]
        S.specpc_select_tokens(p, top_k, 4, q, k, ids, *out, torch.empty(size, dtype=torch.uint8, device="cuda"))
        count = int(out[2])
        got.append([count, out[0][:count].clone(), out[1][:count].clone()])
    assert all(torch.equal(a[2], ids[a[1].long()]) for a in got)
    assert got[0][0] == got[2][0] and torch.equal(got[0][1], got[2][1])
    # 60000 sums within a few per cent of each other are about 1e-6 apart where the last one is kept, which is what the two ways differ
    # by: a few of the 8000 may change places, each with its neighbours
    close = 4 * (2 * 4 + 1) if kw.get("gain", 2.0) < 1 else 0
    here, there = (set(a[1].tolist()) for a in got[:2])
    assert len(here ^ there) <= close


def test_prompt_tokens_whose_sample_misleads(S):
    n = 60000
    q, k = tensors([n], 12, d=64, rows=64, gain=1.0, planted=0)
    p = params(S, q, k, [n], 32, 512)
    info = S.prune_info(p, "tokens", 4000)
    for layer in range(12):
        sampled(info, k[layer]).mul_(3)
    ids = torch.arange(n, dtype=torch.int32, device="cuda")
    got = []
    most = info["workspace_bytes"]
    assert most > 0
    for size in (most, most - 1):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        out = [torch.full((n,), -7, dtype=torch.int32, device="cuda") for _ in range(2)] + [torch.zeros(1, dtype=torch.int32, device="cuda")]
        S.specpc_select_tokens(p, 4000, 0, q, k, ids, *out, ws)
        assert size < most or rows_of(info, ws)[1].item() == 1
        got.append(out)
    assert all(torch.equal(a, b) for a, b in zip(*got))


@pytest.mark.parametrize("lens,n_layers,c_floor,kw", [
    ([32771], 8, 256, {}),
    ([32771], 9, 0, {"heads": 4, "group": 7}),
    ([32771], 8, 1024, {"gain": 0.7}),                                     # floor = budget: every head keeps as much
    ([9000, 30123, 700, 25000], 6, 100, {"dtype": torch.float16}),
    ([32771], 8, 256, {"mislead": 4}),
    ([32771], 8, 0, {"mislead": 3}),
])
def test_shared_budgets_are_those_of_complete_scores(S, lens, n_layers, c_floor, kw):
    kw = dict(kw)
    mislead = kw.pop("mislead", 0)
    q, k = tensors(lens, n_layers, **kw)
    # heads of different sharpness, so that their shares differ
    q *= torch.linspace(0.6, 1.6, q.shape[3], device="cuda").to(q.dtype)[None, None, None, :, None]
    p = params(S, q, k, lens, 32, 1024)
    info = S.prune_info(p, "ada")
    if mislead:
        sampled(info, k[2]).mul_(mislead)
        sampled(info, k[4])[:, :, 1].mul_(mislead)
    H, KT = k.shape[2], S.total_keep(p)
    most = info["workspace_bytes"]
    assert most > 0
    got = []
    for size in (most, most - 1, most):                                     # (no room for pruning in the second)
        idx = torch.full((n_layers, H * KT), -7, dtype=torch.int32, device="cuda")
        off = torch.full((n_layers, len(lens), H + 1), -7, dtype=torch.int32, device="cuda")
        k_out = torch.empty(n_layers, H * KT, 128, dtype=k.dtype, device="cuda")
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        S.speckv_compress_ada(p, c_floor, q, k, None, idx, off, k_out, None, ws)
        if mislead and size == most:
            assert rows_of(info, ws)[1].view(n_layers, H)[2].all()
        got.append((idx, off, k_out.view(torch.int16)))
    assert got[0][1].diff(dim=-1).unique().numel() > 1 or c_floor >= 1024
    for other in got[1:]:
        assert all(torch.equal(a, b) for a, b in zip(got[0], other))


def test_many_probabilities_below_the_smallest_number_of_a_bound(S):
    """A sink takes nearly all of every row.  The scores that decide are about 2^-28, each from one row, but for 100 keys: 0.4 % of
    their score is from the other 32767 rows, 2^-50 each.  Without that part they are below the threshold and below the keys to be kept."""
    n, n_layers, top_k = 48000, 16, 2000
    q = torch.zeros(n_layers, 1, 64, 32, 64, dtype=torch.bfloat16, device="cuda")
    k = torch.zeros(n_layers, n, 8, 64, dtype=torch.bfloat16, device="cuda")
    few = torch.arange(100, device="cuda") * 384 + 128 + 7                   # in tiles 1, 4, 7 ..: below, only the odd ones are used
    few = few[(few // 128) % 2 == 1]
    others = torch.arange(3, 47000, 11, device="cuda")                       # about twice as many as are kept
    others = others[~torch.isin(others, few)]
    least = math.log2(2.0 ** -28 * (1 + 2 / 32))                             # lower end of a first digit
    # channel 0: the sink, 2^60 in every row; channel 2: the other rows; channels 1 and 3: the row that decides
    q[..., 0] = 1
    q[..., 2] = 1
    k[..., 2] = -40
    k[:, 0, :, 0] = 60
    k[:, few, :, 2] = -50.125 + 60
    q[0, 0, 0, 0, 1:4] = torch.tensor([1, 0, 1], device="cuda")
    k[0, :, 0, 1] = -40
    for keys, score in ((few, least - 0.0058), (others, least + 0.0014)):
        k[0, keys, 0, 1] = 32
        k[0, keys, 0, 3] = score + 60 - 32
    k[:, 0, :, 2] = 0
    k[0, 0, 0, 1] = 0
    sm_scale = math.log(2.0) * (1 + 2e-6)
    p = S.SpecKVParams.for_tensors(q, k, seq_lens=[n], n_window=64, pool_k=1, c_max=512, sm_scale=sm_scale)
    exact = torch.zeros(n, dtype=torch.float64, device="cuda")
    for layer in range(n_layers):
        for h in range(32):
            # (rows of a layer and head are alike but for the first one of head 0 of layer 0; none sees the sink's window)
            row = (q[layer, 0, :2, h].double() @ k[layer, :, h // 4].double().t()) * (sm_scale * math.log2(math.e))
            prob = torch.exp2(row - torch.log2(torch.exp2(row - 60).sum(-1, keepdim=True)) - 60)
            exact += prob[0] + 63 * prob[1]
    want = exact[:n - 64].sort(descending=True, stable=True).indices[:top_k].sort().values
    assert torch.isin(few, want).all() and exact[few].min() > exact[others].max() * (1 + 1e-3)
    ids = torch.arange(n, dtype=torch.int32, device="cuda")
    out = [torch.full((n,), -7, dtype=torch.int32, device="cuda") for _ in range(2)] + [torch.zeros(1, dtype=torch.int32, device="cuda")]
    S.specpc_select_tokens(p, top_k, 0, q, k, ids, *out, torch.empty(S.specpc_workspace_bytes(p, top_k), dtype=torch.uint8, device="cuda"))
    got = out[0][:int(out[2])].long()
    assert torch.equal(got[:-64], want)
