"""How a scoring sweep is cut up: where the row normalisers are merged, workgroups per chunk, rows that heads share a
block for.  Everything against the float64 oracle at the bars of test_gpu_parity."""
import math

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


def shape(**kw):
    c = dict(name="geometry", n_layers=1, n_q_heads=8, n_kv_heads=4, head_dim=128, seq_lens=(1000,), n_window=16,
             n_lookahead=16, pool_k=7, c_max=200, dtype="bf16", n_planted=4, channel_scale=(0.5, 4.0), seed=5)
    c.update(kw)
    c.setdefault("sm_scale", 1.0 / math.sqrt(c["head_dim"]))
    return workloads.SpecKVWorkload(**c)


# Up to 40 chunks of a sequence the column sweep's workgroups merge the partial pairs themselves: no chunk at all, one,
# both sides of a batch of 16 and of the limit, a short and a long sequence together; with one and with two threads per row,
# with the normalisers in registers and in LDS (fp32, two row blocks)
@pytest.mark.parametrize("kw", [
    dict(seq_lens=(100,)), dict(seq_lens=(700, 20, 1300)), dict(seq_lens=(512 * 17 + 16,)),
    dict(seq_lens=(512 * 40 + 30,)), dict(seq_lens=(512 * 41 + 30,)), dict(seq_lens=(600, 512 * 45)),
    dict(seq_lens=(512 * 41 + 30,), n_q_heads=16, n_window=32, n_lookahead=30),
    dict(seq_lens=(512 * 33 + 30,), n_q_heads=16, n_window=64, n_lookahead=64),
    dict(seq_lens=(512 * 18 + 30,), n_q_heads=16, head_dim=64, n_window=64, n_lookahead=64, dtype="f32"),
], ids=lambda kw: "-".join(str(x) for x in kw.values()))
def test_row_normalisers_merged_in_the_column_sweep(S, kw):
    parity.check_full_path(S, shape(**kw))


# Calls of up to 8 units with chunks shorter than 512 keys: one tile per workgroup, two, three; a last one that is shorter;
# a live length that leaves whole workgroups without keys; 8 and 9 units; every tile size (64 to 256 keys)
@pytest.mark.parametrize("keys,chunks,kw", [
    (128, 0, dict(seq_lens=(130,), n_kv_heads=1, n_q_heads=4)),
    (128, 3, dict(seq_lens=(128 * 3 + 15,), n_kv_heads=1, n_q_heads=4)),
    (128, 9, dict(seq_lens=(128 * 3 + 15, 900), dtype="f32", head_dim=64, n_kv_heads=2)),
    (128, 13, dict(seq_lens=(1700,), dtype="f32")),
    (64, 14, dict(seq_lens=(920,), dtype="f32")),
    (256, 20, dict(seq_lens=(5200,), n_q_heads=16, n_kv_heads=8)),
    (512, 18, dict(seq_lens=(9000,), n_q_heads=16, n_kv_heads=8, dtype="f16")),
    (512, 6, dict(seq_lens=(3000,), n_q_heads=18, n_kv_heads=9)),
    (256, 16, dict(seq_lens=(4133,), n_q_heads=32, n_kv_heads=8, n_window=64, n_lookahead=64)),
    (256, 7, dict(seq_lens=(2100,), n_q_heads=32, n_kv_heads=8, n_window=64, n_lookahead=64, head_dim=64)),
], ids=lambda kw: "-".join(str(x) for x in kw.values()) if isinstance(kw, dict) else str(kw))
@pytest.mark.parametrize("mode", ["online", "fixed"])
def test_workgroups_of_few_tiles(S, keys, chunks, kw, mode, monkeypatch):
    monkeypatch.setenv("SPECKV_ROW_STATISTICS", mode)
    w = shape(**kw)
    info = S.plan_info(parity.make_params(S, w))
    assert (info["chunk_keys"], info["n_chunks"]) == (keys, chunks)
    parity.check_full_path(S, w)


@pytest.mark.parametrize("n_live", [4000, 1100, 200, 40])
def test_workgroups_of_few_tiles_with_a_length_on_the_device(S, n_live):
    w = shape(seq_lens=(4000,), n_q_heads=16, n_kv_heads=8)
    t = workloads.generate(w)
    q, k = t["q"].cuda(), t["k"].cuda()
    n_dev = torch.tensor([n_live], dtype=torch.int32, device="cuda")
    out = []
    for n, extra in ((4000, dict(n_in_dev=n_dev)), (n_live, {})):
        kk = k[:, :n].contiguous()
        p = S.SpecKVParams.for_tensors(q, kk, seq_lens=(n,), n_window=w.n_window, pool_k=w.pool_k, c_max=w.c_max,
                                       sm_scale=w.sm_scale, **extra)
        raw, pooled = (torch.full((1, 8 * n), -1.0, device="cuda") for _ in range(2))
        S.speckv_score(p, q, kk, pooled, raw, parity.alloc_ws(S, p))
        out.append((pooled.view(8, n).double().cpu().numpy(), raw.view(8, n).double().cpu().numpy()))
    for dev, host in zip(*out):
        parity.assert_scores_close(dev[:, :n_live], host, "live %d" % n_live)
        assert (dev[:, n_live:] == 0).all()


# The host length is a bound then: it may call for other chunks than the live length, and for another place where the
# chunks' pairs are merged (up to 40 chunks the column sweep, with one or two threads per row).  Scores have the same bits.
LENGTHS = [
    ("short", 7000, (7000, 4097, 2600, 700, 64), dict(n_q_heads=32, n_kv_heads=8, n_window=64, n_lookahead=64)),
    ("short-shared-rows", 14000, (8000, 4133, 900), dict(n_q_heads=32, n_kv_heads=8, n_window=32, n_lookahead=23)),
    ("short-64", 9000, (8000, 4097, 2600, 1100), dict(n_q_heads=32, n_kv_heads=8, head_dim=64, n_window=64, n_lookahead=64)),
    ("short-64-one-block", 9000, (4097, 2600, 300), dict(n_q_heads=32, n_kv_heads=8, head_dim=64, n_window=16, n_lookahead=4)),
    ("short-f32", 3000, (2600, 1500, 1024, 300), dict(n_q_heads=8, n_kv_heads=2, head_dim=64, dtype="f32")),
    ("short-f32-128", 6000, (5000, 1300, 200), dict(n_q_heads=8, n_kv_heads=2, dtype="f32")),
    ("short-gqa7", 9000, (6000, 3000, 600), dict(n_q_heads=28, n_kv_heads=4, n_window=64, n_lookahead=64)),
    ("merge", 30000, (30000, 15000, 10200), dict(n_q_heads=16, n_kv_heads=4, n_window=64, n_lookahead=64)),
    ("merge-two-threads", 60000, (41000, 20000, 12000), dict(n_q_heads=4, n_kv_heads=2, n_window=16, n_lookahead=39)),
    ("merge-f32", 30000, (17000,), dict(n_q_heads=8, n_kv_heads=4, dtype="f32", n_window=64, n_lookahead=64)),
    ("merge-64", 60000, (18000,), dict(n_q_heads=8, n_kv_heads=2, head_dim=64, n_window=64, n_lookahead=64)),
]


@pytest.mark.parametrize("bound,lives,kw", [x[1:] for x in LENGTHS], ids=[x[0] for x in LENGTHS])
def test_a_length_on_the_device_gives_the_bits_of_a_host_length(S, bound, lives, kw):
    w = shape(seq_lens=(bound,), q_gain=2.0, **kw)
    t = workloads.generate(w)
    q, k = t["q"].cuda(), t["k"].cuda()
    H = w.n_kv_heads

    def scores(kk, n, **extra):
        p = S.SpecKVParams.for_tensors(q, kk, seq_lens=(n,), n_window=w.n_window, pool_k=w.pool_k, c_max=w.c_max,
                                       sm_scale=w.sm_scale, **extra)
        raw, pooled = (torch.full((1, H * n), -1.0, device="cuda") for _ in range(2))
        idx = torch.full((1, H * S.total_keep(p)), -7, dtype=torch.int32, device="cuda")
        k_out = torch.empty((1, H * S.total_keep(p), w.head_dim), dtype=kk.dtype, device="cuda")
        ws = parity.alloc_ws(S, p)
        S.speckv_score(p, q, kk, pooled, raw, ws)
        S.speckv_compress(p, q, kk, None, idx, k_out, None, ws)
        return raw.view(H, n), pooled.view(H, n), idx.view(H, -1)

    for live in lives:
        raw, pooled, idx = scores(k, bound, n_in_dev=torch.tensor([live], dtype=torch.int32, device="cuda"))
        raw_h, pooled_h, idx_h = scores(k[:, :live].contiguous(), live)
        assert torch.equal(raw[:, :live], raw_h) and torch.equal(pooled[:, :live], pooled_h), live
        assert bool((raw[:, live:] == 0).all()) and bool((pooled[:, live:] == 0).all())
        keep = idx_h.shape[1]
        assert torch.equal(idx[:, :keep], idx_h) and bool((idx[:, keep:] == -1).all())


# Row blocks that heads share, and blocks that waves share: 32-row blocks of a group -> what the last waves do
#   1, 2 of 4 waves; 3; 5, 6 of 8 waves; 7; 9, 10 with two blocks a wave; 13, 14; two super-blocks of unequal size; two rows a
#   head; a head longer than a super-block (never packed)
@pytest.mark.parametrize("g,window,lookahead", [
    (1, 16, 9), (2, 16, 24), (4, 16, 1), (4, 16, 24), (4, 16, 32), (4, 32, 23), (4, 64, 1), (4, 32, 40), (4, 32, 48), (5, 16, 64),
    (5, 64, 20), (7, 64, 8), (7, 64, 64), (8, 1, 1), (1, 64, 520)])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("mode", ["online", "fixed"])
def test_rows_packed_and_blocks_shared(S, g, window, lookahead, dtype, d, mode, monkeypatch):
    monkeypatch.setenv("SPECKV_ROW_STATISTICS", mode)
    monkeypatch.setenv("SPECKV_SCORE_KERNEL", "tile")
    parity.check_full_path(S, shape(n_q_heads=2 * g, n_kv_heads=2, head_dim=d, n_window=window, n_lookahead=lookahead,
                                    seq_lens=(1500, 2740), dtype=dtype))


# Groups of many heads with few rows each: fewer row blocks than heads padded to whole blocks would take super-blocks
@pytest.mark.parametrize("g,rows,dtype,d", [(9, 2, "f32", 128), (17, 2, "f32", 128), (17, 2, "bf16", 128), (40, 3, "bf16", 64),
                                            (64, 2, "f16", 128), (33, 17, "f32", 64)])
@pytest.mark.parametrize("mode", ["online", "fixed"])
def test_many_heads_of_few_rows(S, g, rows, dtype, d, mode, monkeypatch):
    monkeypatch.setenv("SPECKV_ROW_STATISTICS", mode)
    parity.check_full_path(S, shape(n_q_heads=2 * g, n_kv_heads=2, head_dim=d, n_window=1, n_lookahead=rows - 1,
                                    seq_lens=(1500, 740), dtype=dtype))


# The same with heads combined by maximum (Alg. 2): 1, 2, 5, 6, 9, 10, 13, 14 packed blocks; 16, taken in pairs; two super-blocks
# of unequal size; heads made of whole blocks; a head longer than a super-block; super-blocks that heads of two rows do not need.
# (fp32: the row statistics share blocks, the column maxima of two blocks a wave do not.)  Pools of one: every score is compared.
@pytest.mark.parametrize("g,window,lookahead", [
    (1, 16, 9), (2, 16, 24), (8, 16, 4), (4, 16, 32), (4, 64, 1), (4, 32, 48), (5, 16, 64), (5, 64, 20), (7, 64, 9), (7, 64, 20), (4, 64, 64),
    (1, 64, 520), (17, 1, 1)])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f16", 64), ("f32", 128), ("f32", 64)])
def test_heads_combined_by_maximum(S, g, window, lookahead, dtype, d):
    n, budget = 2740, 400
    w = shape(n_layers=2, n_q_heads=2 * g, n_kv_heads=2, head_dim=d, n_window=window, n_lookahead=lookahead, seq_lens=(n,),
              dtype=dtype, pool_k=1, c_max=budget)
    t = workloads.generate(w)
    ids = workloads.generate_token_ids(w)
    ref = parity.orc.specpc_compress_prompt(workloads.to_float64(t["q"][:, 0]), workloads.to_float64(t["k"]), ids.numpy(), window,
                                            1, 1, budget, 0, w.sm_scale)
    p = parity.make_params(S, w)
    ws = torch.empty(S.specpc_compress_workspace_bytes(p, 0), dtype=torch.uint8, device="cuda")
    idx, out = (torch.full((budget + window,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    count = torch.zeros(1, dtype=torch.int32, device="cuda")
    S.specpc_compress_prompt(p, 0, 1, t["q"].cuda(), t["k"].cuda(), ids.cuda(), idx, out, count, ws)
    assert int(count) == budget + window and torch.equal(out.cpu(), ids[idx.cpu().long()])
    parity.assert_indices_valid(idx.cpu().numpy().astype("int64"), ref["pooled"], n, window, budget, "alg2")


def test_shared_blocks_behind_outliers_and_the_query_stationary_sweep(S, monkeypatch):
    """Fixed references that overflow (segments are repaired by the waves that share), and partial pairs left by the
    query-stationary kernel, which shares nothing, for a column sweep that does."""
    monkeypatch.setenv("SPECKV_ROW_STATISTICS", "fixed")
    for dtype in ("bf16", "f32"):
        parity.check_full_path(S, shape(n_q_heads=8, n_kv_heads=2, n_window=64, n_lookahead=1, seq_lens=(9000,), dtype=dtype,
                                        q_gain=8.0, n_planted=8))
    parity.check_full_path(S, shape(n_q_heads=8, n_kv_heads=2, head_dim=64, n_window=64, n_lookahead=1, seq_lens=(5000,)))
