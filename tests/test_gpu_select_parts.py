"""Selection inside the fused call where several workgroups share a row: the kept indices are the exact ranking of the
library's own scores (whole numbers, so every comparison is exact), and the cache holds those rows bit for bit."""
import math

import numpy as np
import pytest
import torch

import workloads
from . import test_gpu_parity as parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import paper_2506_08373_amd as S
    S.load_library()
    return S


def ranked(scores, count):
    """The count best of a row of fp32 scores by their bits (a positive NaN above everything), ties to the lower index."""
    bits = (scores + np.float32(0)).view(np.uint32)
    key = np.where(bits >> 31, ~bits, bits | np.uint32(0x80000000)).astype(np.int64)
    return np.sort(np.argsort(-key, kind="stable")[:count])


def check(S, q, k, lens, n_window, c_max, pool_k=7, n_in_dev=None):
    L, T, H, d = k.shape
    p = S.SpecKVParams.for_tensors(q, k, seq_lens=lens, n_window=n_window, pool_k=pool_k, c_max=c_max,
                                   sm_scale=1.0 / math.sqrt(d), n_in_dev=n_in_dev)
    KT = S.total_keep(p)
    ws = parity.alloc_ws(S, p)
    pooled = torch.empty(L, H * T, device="cuda")
    idx = torch.full((L, H * KT), -7, dtype=torch.int32, device="cuda")
    k_out = torch.empty(L, H * KT, d, dtype=k.dtype, device="cuda")
    S.speckv_score(p, q, k, pooled, None, ws)
    S.speckv_compress(p, q, k, None, idx, k_out, None, ws)
    sc, ix, kc, ko = pooled.cpu().numpy(), idx.cpu().numpy(), k.cpu(), k_out.cpu()
    for layer in range(L):
        t0 = keep0 = 0
        for n in lens:
            live = n if n_in_dev is None else int(n_in_dev)
            m, keep = live - n_window, min(c_max, n - n_window) + n_window
            for g in range(H):
                row = sc[layer, H * t0 + g * n:H * t0 + g * n + m]
                r0 = H * keep0 + g * keep
                want = np.concatenate([ranked(row, min(c_max, m)), np.arange(m, live)])
                got = ix[layer, r0:r0 + keep]
                assert np.array_equal(got[:len(want)], want), (layer, n, g)
                assert (got[len(want):] == -1).all()
                rows = kc[layer, t0 + torch.from_numpy(want), g]
                assert torch.equal(ko[layer, r0:r0 + len(want)].view(torch.int16), rows.view(torch.int16))
            t0 += n
            keep0 += keep


def tensors(lens, n_layers=1, n_heads=2, rows=32, seed=3, gain=1.0):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    q = torch.randn(n_layers, len(lens), rows, 2 * n_heads, 64, generator=g, device="cuda") * gain
    k = torch.randn(n_layers, sum(lens), n_heads, 64, generator=g, device="cuda")
    return q.to(torch.bfloat16), k.to(torch.bfloat16)


# a fifth of the row kept and one more; thousands of candidates with the threshold's first digit, ranked by one workgroup;
# the shortest rows of the rule and one entry less; parts of one step of 4096 entries and of two, the last one short; rows
# that start at every alignment (odd lengths); a batch whose shorter rows leave parts empty; 128 rows and one more
@pytest.mark.parametrize("lens,n_layers,n_heads,c_max", [
    ((16399,), 1, 2, 300), ((16400,), 1, 2, 300), ((20501,), 1, 3, 1), ((50003,), 1, 8, 2048), ((65551,), 2, 4, 8192),
    ((65551,), 1, 1, 8193), ((131085,), 1, 2, 1024), ((40001, 700, 17, 30003), 1, 3, 500), ((17001,), 16, 8, 64),
    ((17001,), 43, 3, 64), ((33001,), 1, 3, 6597), ((33001,), 1, 3, 6598), ((61001,), 1, 2, 9000), ((61001,), 1, 2, 16000),
    ((33001,), 1, 2, 16000), ((131085,), 1, 1, 30000)])
def test_rows_shared_by_workgroups(S, lens, n_layers, n_heads, c_max):
    q, k = tensors(lens, n_layers, n_heads, gain=2.0)
    check(S, q, k, lens, 16, c_max)


@pytest.mark.parametrize("c_max", [1, 4096, 5000])
def test_many_equal_scores(S, c_max):
    """All keys alike: the leading digits hold more entries than the candidate list."""
    q, k = tensors((33001,))
    check(S, q, torch.zeros_like(k), (33001,), 16, c_max)
    k[:, ::7] = 0                                         # pooled with a kernel of 7: plateaus of equal scores everywhere
    check(S, q, k, (33001,), 16, c_max)


def test_scores_that_are_no_numbers(S):
    q, k = tensors((33001,))
    k[0, 9000, 0, 0] = math.inf                           # logits of both signs: every score of the head is NaN
    k[0, 20000:20010, 1] = -1e30 * q[0, 0, 0, 2].sign()   # far below every other
    check(S, q, k, (33001,), 16, 700)


# One query row whose logits spread over hundreds of nats, as an attention sink makes them: the threshold lies around 2^-30, 2^-75
# or among scores that underflowed.  Rows shared by workgroups (8, 128 of them) and not (129, 256; short ones in registers)
@pytest.mark.parametrize("n,n_layers,n_heads", [(16400, 1, 8), (70003, 1, 2), (17001, 16, 8), (17001, 43, 3), (40003, 32, 8),
                                                (9001, 32, 8), (9001, 1, 2)])
@pytest.mark.parametrize("gain", [10.0, 25.0, 60.0])
def test_peaked_rows(S, n, n_layers, n_heads, gain):
    q, k = tensors((n,), n_layers, n_heads, rows=1, gain=gain)
    check(S, q, k, (n,), 1, n // 60)


# Normalisers from the caller that are too small: scores far above what probabilities sum to, some or all of them infinite
@pytest.mark.parametrize("n,n_layers", [(33001, 1), (17001, 65), (9001, 17)])
@pytest.mark.parametrize("lse", [-20.0, -60.0, -84.0])
def test_scores_of_any_size(S, n, n_layers, lse):
    q, k = tensors((n,), n_layers)
    p = S.SpecKVParams.for_tensors(q, k, seq_lens=(n,), n_window=16, pool_k=7, c_max=400, sm_scale=0.125)
    norm = torch.full((n_layers, 1, 32, 4), lse, device="cuda")
    pooled = torch.empty(n_layers, 2 * n, device="cuda")
    idx = torch.empty(n_layers, 2 * 416, dtype=torch.int32, device="cuda")
    k_out = torch.empty(n_layers, 2 * 416, 64, dtype=k.dtype, device="cuda")
    ws = parity.alloc_ws(S, p)
    S.speckv_score_lse(p, q, k, norm, pooled, None, ws)
    S.speckv_compress_lse(p, q, k, None, norm, idx, k_out, None, ws)
    scores, got = pooled.view(n_layers, 2, n).cpu().numpy(), idx.view(n_layers, 2, 416).cpu().numpy()
    for layer in range(n_layers):
        for h in range(2):
            assert np.array_equal(got[layer, h, :400], ranked(scores[layer, h, :n - 16], 400)), (layer, h)


@pytest.mark.parametrize("n_live", [60000, 17003, 900, 16])
def test_a_length_on_the_device(S, n_live):
    q, k = tensors((60000,))
    n_dev = torch.tensor([n_live], dtype=torch.int32, device="cuda")
    check(S, q, k, (60000,), 16, 1500, n_in_dev=n_dev)


# one row of a prompt-token call: ranked by one workgroup up to 32K candidates and above 8192 kept, by several otherwise; the
# expansion with fewer intervals than a workgroup takes, with many workgroups, with none, with intervals that all overlap
@pytest.mark.parametrize("n,top_k,n_neighbor", [
    (3000, 1, 3), (32783, 700, 8), (32784, 700, 8), (20003, 0, 4), (20003, 4096, 1), (40005, 8192, 2), (40005, 8193, 30),
    (70001, 20000, 1), (20003, 20003, 5), (20003, 3, 2**31 - 1)])
def test_prompt_tokens_and_their_neighbours(S, n, top_k, n_neighbor):
    w = 16
    q, k = tensors((n,), 2, 2, gain=2.0)
    p = S.SpecKVParams.for_tensors(q, k, seq_lens=(n,), n_window=w, pool_k=7, c_max=1, sm_scale=0.125)
    ids = torch.randint(0, 1 << 20, (n,), dtype=torch.int32, device="cuda")
    ws = torch.empty(S.specpc_workspace_bytes(p, top_k), dtype=torch.uint8, device="cuda")

    def run(nb):
        idx, out = (torch.full((n,), -5, dtype=torch.int32, device="cuda") for _ in range(2))
        count = torch.zeros(1, dtype=torch.int32, device="cuda")
        S.specpc_select_tokens(p, top_k, nb, q, k, ids, idx, out, count, ws)
        c = int(count)
        assert torch.equal(out[:c], ids[idx[:c].long()]) and bool((idx[c:] == -5).all())
        return idx[:c].cpu().numpy()

    m = n - w
    kept = run(0)
    assert kept[-w:].tolist() == list(range(m, n))
    # the scores again in 64 bits
    score = torch.zeros(n, dtype=torch.float64, device="cuda")
    last = torch.cat([m + torch.arange(w), torch.full((q.shape[2] - w,), n - 1)]).cuda()
    hidden = torch.arange(n, device="cuda")[None, :] > last[:, None]
    for layer in range(2):
        for h in range(4):
            logits = (q[layer, 0, :, h].double() @ k[layer, :, h // 2].double().t()) * 0.125
            score += torch.softmax(logits.masked_fill(hidden, -math.inf), dim=1).sum(0)
    pooled = torch.nn.functional.max_pool1d(score[None, None, :m], 7, 1, 3)[0, 0].cpu().numpy()
    parity.assert_indices_valid(kept, pooled, n, w, top_k, "tokens")
    want = np.zeros(n, bool)
    for t in kept[:len(kept) - w].tolist():
        want[max(0, t - n_neighbor):t + n_neighbor + 1] = True
    want[m:] = True
    assert np.array_equal(run(n_neighbor), np.nonzero(want)[0])


@pytest.mark.parametrize("pool_k", [15, 16, 17, 31, 32, 63, 64, 100, 255])
@pytest.mark.parametrize("n", [40005, 300])
def test_wide_maximum_pooling(S, n, pool_k):
    """Fused calls pool without handing the raw scores out; speckv_score with raw does it entry by entry."""
    q, k = tensors((n,), gain=2.0)
    w = 16
    p = S.SpecKVParams.for_tensors(q, k, seq_lens=(n,), n_window=w, pool_k=pool_k, c_max=5, sm_scale=0.125)
    ws = parity.alloc_ws(S, p)
    raw, pooled, alone = (torch.empty(1, 2 * n, device="cuda") for _ in range(3))
    S.speckv_score(p, q, k, pooled, raw, ws)
    S.speckv_score(p, q, k, alone, None, ws)
    assert torch.equal(pooled, alone)
    x = raw.view(2, n)[:, :n - w]
    padded = torch.nn.functional.pad(x, (pool_k // 2, (pool_k - 1) // 2), value=-1.0)
    assert torch.equal(pooled.view(2, n)[:, :n - w], padded.unfold(1, pool_k, 1).amax(-1))


# Rows of up to 8192 entries with a pooling kernel of up to 16: pooled and ranked in one launch; both sides of both limits,
# one and two planes, one vector to a full row, every entry kept, equal scores, a batch
@pytest.mark.parametrize("lens,rows,c_max,pool_k", [
    ((17,), 32, 5, 7), ((21,), 32, 100, 7), ((300,), 32, 7, 1), ((4113,), 32, 4000, 16), ((4113,), 32, 900, 17),
    ((8192,), 32, 2048, 6), ((8193,), 32, 2048, 7), ((5001, 19, 1234, 8192), 32, 300, 7), ((3001,), 320, 700, 7)])
def test_short_rows_pooled_and_ranked_in_one_launch(S, lens, rows, c_max, pool_k):
    q, k = tensors(lens, 2, 3, rows=rows, gain=2.0)
    check(S, q, k, lens, 16, c_max, pool_k)
    check(S, q, torch.zeros_like(k), lens, 16, c_max, pool_k)
    if len(lens) == 1:
        for n_live in (lens[0] - 1, 17, 16, 1):
            check(S, q, k, lens, 16, c_max, pool_k, n_in_dev=torch.tensor([max(n_live, 16)], dtype=torch.int32, device="cuda"))


# the most heads whose sums stay in LDS, one more, and the most there may be
@pytest.mark.parametrize("H,lens,c_floor", [(16, (5003, 40), 11), (17, (5003, 40), 11), (128, (1200,), 0), (1, (9001,), 60)])
def test_shared_budget_around_the_heads_held_in_lds(S, H, lens, c_floor):
    n_window, c_max = 8, 100
    w = workloads.SpecKVWorkload(name="ada_heads", n_layers=1, n_q_heads=H, n_kv_heads=H, head_dim=64, seq_lens=lens, n_window=n_window,
                                 n_lookahead=1, pool_k=7, c_max=c_max, dtype="bf16", sm_scale=1.0)
    p = parity.make_params(S, w)
    rng = np.random.default_rng(H)
    base = rng.integers(-20, 400, size=(1, H * w.total_tokens)).astype(np.float32) / 400
    for s in range(len(lens)):
        parity.split_scores(w, base, 0, s)[...] *= np.float32(2) ** rng.integers(-2, 3, size=(H, 1))
    idx = torch.full((1, H * S.total_keep(p)), -1, dtype=torch.int32, device="cuda")
    head_off = torch.full((1, len(lens), H + 1), -1, dtype=torch.int32, device="cuda")
    ws = torch.empty(S.ada_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    S.speckv_select_ada(p, c_floor, torch.from_numpy(base).cuda(), idx, head_off, ws)
    got, off = idx.cpu().numpy(), head_off.cpu().numpy()
    for s, n in enumerate(lens):
        rows = parity.split_scores(w, base, 0, s)[:, :n - n_window].astype(np.float64)
        want = parity.orc.ada_keep_indices(rows, n, n_window, c_max, c_floor)
        assert off[0, s].tolist() == np.concatenate([[0], np.cumsum([len(x) for x in want])]).tolist()
        assert parity.ada_block(w, got, 0, s, c_max).tolist() == np.concatenate(want).tolist()
