"""Selection of rows that one workgroup holds in registers (up to 8192 vectors of four scores, 4096 where the
first digit is counted already): whole numbers, so every comparison with the oracle is exact."""
import numpy as np
import pytest
import torch

import workloads
from . import test_gpu_parity
from oracle import speckv_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import paper_2506_08373_amd as S
    S.load_library()
    return S


# one entry; less than a vector; one wavefront's vectors and the next; a vector per thread and one more; the
# largest row at every alignment, and rows that fit at some alignments only
@pytest.mark.parametrize("m", [1, 3, 5, 255, 257, 4095, 4097, 8193, 16385, 32761, 32765, 32766, 32767, 32768, 32771])
def test_select_on_short_rows(S, m):
    H, n_window = 4, 2 if m % 2 else 1
    n = m + n_window                                    # odd: the four rows start at the four alignments
    rng = np.random.default_rng(m)
    rows = np.full((H, n), 1e30, dtype=np.float32)      # scores of the window are never looked at
    rows[0, :m] = np.exp(4 * rng.standard_normal(m))
    rows[1, :m] = rng.integers(0, 9, m)
    rows[2, :m] = 0.25
    rows[3, :m] = rng.standard_normal(m)
    pooled = torch.from_numpy(rows).reshape(1, -1).cuda()
    for c_max in sorted({1, max(1, m // 7), max(1, m - 1), m}):
        p = S.SpecKVParams(n_layers=1, n_q_heads=H, n_kv_heads=H, head_dim=64, seq_lens=(n,), n_window=n_window,
                           n_lookahead=1, pool_k=7, c_max=c_max, dtype=torch.bfloat16, sm_scale=1.0)
        idx = torch.full((1, H * S.total_keep(p)), -1, dtype=torch.int32, device="cuda")
        S.speckv_select(p, pooled, idx)
        got = idx.cpu().numpy().reshape(H, -1)
        for g in range(H):
            want = orc.keep_indices(rows[g, :m].astype(np.float64), n, n_window, c_max)
            assert np.array_equal(got[g], want), (c_max, g)


@pytest.mark.parametrize("m", [3, 261, 4099, 16390])
def test_every_bit_pattern_has_its_own_rank(S, m):
    """NaNs rank by their bits too, down to the lowest pattern of all, which vectors outside a row share."""
    H, n_window = 4, 1 if m % 2 == 0 else 2
    n = m + n_window
    rng = np.random.default_rng(m)
    bits = rng.choice(np.array([0xffffffff, 0xfffffffe, 0xfffffffd, 0xff800000, 0x7fffffff], np.uint32), (H, n))
    bits[1, :] = 0xffffffff
    pooled = torch.from_numpy(bits.view(np.int32)).cuda().view(torch.float32).reshape(1, -1)
    key = np.where(bits >> 31, ~bits, bits | np.uint32(0x80000000)).astype(np.float64)     # exact: below 2^53
    for c_max in sorted({1, m // 3, m * 2 // 3, m - 1}):
        p = S.SpecKVParams(n_layers=1, n_q_heads=H, n_kv_heads=H, head_dim=64, seq_lens=(n,), n_window=n_window,
                           n_lookahead=1, pool_k=7, c_max=c_max, dtype=torch.bfloat16, sm_scale=1.0)
        idx = torch.full((1, H * S.total_keep(p)), -1, dtype=torch.int32, device="cuda")
        S.speckv_select(p, pooled, idx)
        got = idx.cpu().numpy().reshape(H, -1)
        for g in range(H):
            assert np.array_equal(got[g], orc.keep_indices(key[g, :m], n, n_window, c_max)), (c_max, g)


@pytest.mark.parametrize("n_in", [521, 4099, 16390, 16447, 16450, 16451])
def test_fused_call_selects_what_its_scores_say(S, n_in):
    """The fused call hands selection the first digit's counts; its indices are those of the scores that
    speckv_score gives for the same inputs."""
    w = workloads.llama8b_layer(n_in=n_in, c_max=256, name="short_rows")
    t = workloads.generate(w)
    q, k, v = (t[x].cuda() for x in ("q", "k", "v"))
    p = S.SpecKVParams.for_tensors(q, k, seq_lens=w.seq_lens, n_window=w.n_window, pool_k=w.pool_k, c_max=w.c_max,
                                   sm_scale=w.sm_scale)
    H, m = w.n_kv_heads, n_in - w.n_window
    idx = torch.empty((1, H * S.total_keep(p)), dtype=torch.int32, device="cuda")
    k_out = torch.empty((1, H * S.total_keep(p), w.head_dim), dtype=w.torch_dtype, device="cuda")
    pooled = torch.empty((1, H * n_in), dtype=torch.float32, device="cuda")
    ws = torch.empty(S.workspace_bytes(p), dtype=torch.uint8, device="cuda")
    S.speckv_score(p, q, k, pooled, None, ws)
    S.speckv_compress(p, q, k, v, idx, k_out, torch.empty_like(k_out), ws)
    got, scores = idx.cpu().numpy().reshape(H, -1), pooled.cpu().numpy().reshape(H, n_in)
    for g in range(H):
        want = orc.keep_indices(scores[g, :m].astype(np.float64), n_in, w.n_window, w.c_max)
        assert np.array_equal(got[g], want), g


@pytest.mark.parametrize("in_bin", [40, 4096, 4097])
def test_rows_just_too_long_for_registers(S, in_bin):
    """The limits of the path that reads a row once more, at a length that does not fit registers."""
    test_gpu_parity.test_select_around_the_limits_of_the_one_read_path(S, 32780, in_bin)


def ordered_keys(bits):
    return np.where(bits >> 31, ~bits, bits | np.uint32(0x80000000)).astype(np.float64)      # exact: below 2^53


@pytest.mark.parametrize("m", [32775, 70001, 300000])
@pytest.mark.parametrize("kind", ["one NaN", "two NaNs", "infinities", "minus infinities"])
def test_long_rows_whose_threshold_is_no_ordinary_number(S, m, kind):
    """Rows that do not fit registers (300000: split over workgroups) where the last score kept is a NaN or an
    infinity: ranked by their bits, ties to the lower index, every slot written, as in short rows."""
    H, n = 2, m + 1
    rng = np.random.default_rng(m)
    bits = rng.random((H, n), dtype=np.float32).view(np.uint32)
    if kind == "one NaN":
        bits[:] = 0x7fc00000
    elif kind == "two NaNs":
        bits[:] = np.where(rng.random((H, n)) < 0.5, 0x7fc00000, 0x7fc00001)
    elif kind == "infinities":
        bits[:, ::3] = 0x7f800000
    else:
        bits[:] = np.where(rng.random((H, n)) < 0.001, bits, 0xff800000)
    pooled = torch.from_numpy(bits.view(np.int32)).cuda().view(torch.float32).reshape(1, -1)
    c_max = 500
    p = S.SpecKVParams(n_layers=1, n_q_heads=H, n_kv_heads=H, head_dim=64, seq_lens=(n,), n_window=1, n_lookahead=1,
                       pool_k=7, c_max=c_max, dtype=torch.bfloat16, sm_scale=1.0)
    ws = torch.empty(max(S.select_workspace_bytes(p), 256), dtype=torch.uint8, device="cuda")
    for workspace in (None, ws):
        idx = torch.full((1, H * S.total_keep(p)), -7, dtype=torch.int32, device="cuda")
        S.speckv_select(p, pooled, idx, *(() if workspace is None else (workspace,)))
        got = idx.cpu().numpy().reshape(H, -1)
        for g in range(H):
            assert np.array_equal(got[g], orc.keep_indices(ordered_keys(bits[g, :m]), n, 1, c_max)), g


def test_token_selection_from_scores_that_are_all_nan(S):
    """One NaN key makes every score of a 40000-token prompt NaN: the first tokens are kept, nothing is left unwritten
    for the expansion to read."""
    n, top = 40000, 64
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    q = torch.randn(1, 1, 32, 4, 64, generator=gen, device="cuda").bfloat16()
    k = torch.randn(1, n, 2, 64, generator=gen, device="cuda").bfloat16()
    k[0, 100, :, 7] = float("nan")
    p = S.SpecKVParams.for_tensors(q, k, seq_lens=[n], n_window=32, pool_k=7, c_max=16, sm_scale=0.125)
    ids = torch.arange(n, dtype=torch.int32, device="cuda")
    idx, out, count = torch.full_like(ids, -7), torch.full_like(ids, -7), torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.full((S.specpc_workspace_bytes(p, top),), 0x3f, dtype=torch.uint8, device="cuda")
    S.specpc_select_tokens(p, top, 4, q, k, ids, idx, out, count, ws)
    want = list(range(top + 4)) + list(range(n - 32, n))
    assert int(count) == len(want) and idx[:len(want)].tolist() == want and out[:len(want)].tolist() == want
    assert (idx[len(want):] == -7).all()
