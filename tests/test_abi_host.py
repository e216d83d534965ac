"""Host-side checks that need no GPU: the library loads, exports its ABI, validates arguments."""
import ctypes
import os
import re

import pytest
import torch

import paper_2506_08373_amd as S
from paper_2506_08373_amd import binding


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(S.library_path()):
        from paper_2506_08373_amd import build
        build.build(verbose=False)
    return S.load_library()


PLAN_INFO_WORDS = 11     # SPECKV_PLAN_INFO_WORDS of include/speckv.h


def base_params(**kw):
    args = dict(n_layers=2, n_q_heads=8, n_kv_heads=2, head_dim=64, seq_lens=[300, 500], n_window=16,
                n_lookahead=16, pool_k=7, c_max=64, sm_scale=0.125, dtype=torch.bfloat16)
    args.update(kw)
    return S.SpecKVParams(**args)


def test_every_declared_symbol_is_exported(lib, repo_root):
    header = open(os.path.join(repo_root, "include", "speckv.h")).read()
    declared = set(re.findall(r"\b(speck?v?_[a-z_]+|specpc_[a-z_]+)\s*\(", header))
    declared = {d for d in declared if not d.endswith("_t")}
    assert {"speckv_score", "speckv_select", "speckv_compact", "speckv_compress",
            "specpc_select_tokens"} <= declared
    for name in declared:
        assert hasattr(lib, name), "header declares %s but the library does not export it" % name
    assert set(binding.EXPORTS) == declared


def test_plan_info_word_count_matches_the_header(repo_root):
    header = open(os.path.join(repo_root, "include", "speckv.h")).read()
    assert int(re.search(r"#define SPECKV_PLAN_INFO_WORDS (\d+)", header).group(1)) == PLAN_INFO_WORDS


def test_prune_info_words_match_the_header_and_agree_with_the_queries(lib, repo_root):
    header = open(os.path.join(repo_root, "include", "speckv.h")).read()
    assert int(re.search(r"#define SPECKV_PRUNE_INFO_WORDS (\d+)", header).group(1)) == len(S.prune_info(base_params())) == 9
    assert set(S.prune_info(base_params()).values()) == {0}
    shape = dict(n_layers=16, n_q_heads=32, n_kv_heads=8, n_window=64, n_lookahead=64, sm_scale=0.1, dtype=torch.bfloat16)
    for lens in ([131072], [70001], [60000, 5000, 300], [40000] * 3):
        p = S.SpecKVParams(head_dim=128, seq_lens=lens, pool_k=7, c_max=1024, **shape)
        info, ada = S.prune_info(p), S.prune_info(p, "ada")
        assert info["pruned"] == ada["pruned"] == 1 and info["n_rows"] == 16 * 8 * len(lens) and info["tile_keys"] == 128
        assert info["rows_at"] + 32 * info["n_rows"] < info["workspace_bytes"] <= S.workspace_bytes(p)
        assert info["workspace_bytes"] < ada["workspace_bytes"] <= S.ada_workspace_bytes(p)
        assert info["sample_step"] in (4, 8, 16) and info["n_chunks"] >= len([n for n in lens if n > 1000])
        assert info["chunk_keys"] % (128 * info["sample_step"]) == 0
    # a size that hides in the rounding of the token list's: 24000 tokens, 1000 kept
    small = S.SpecKVParams(head_dim=64, seq_lens=[24000], pool_k=7, c_max=512, **{**shape, "n_layers": 4})
    assert S.prune_info(small, "tokens", 1000)["pruned"] == 0
    large = S.SpecKVParams(head_dim=64, seq_lens=[60000], pool_k=7, c_max=512, **shape)
    assert S.prune_info(large, "tokens", 1000)["pruned"] == 1 and S.prune_info(large, "tokens", 59000)["pruned"] == 0
    assert S.prune_info(large, "tokens", 1000)["n_rows"] == 1


def test_the_environment_chooses_the_kernels_of_fused_calls_too(lib, monkeypatch):
    p = S.SpecKVParams(n_layers=16, n_q_heads=32, n_kv_heads=8, head_dim=128, seq_lens=[70001], n_window=64, n_lookahead=64, pool_k=7,
                       c_max=1024, sm_scale=0.1, dtype=torch.bfloat16)
    need = S.workspace_bytes(p)
    for name, value in (("SPECKV_SCORE_KERNEL", "qs"), ("SPECKV_SCORE_KERNEL", "tile"), ("SPECKV_ROW_STATISTICS", "online")):
        assert S.prune_info(p)["pruned"] == 1
        with monkeypatch.context() as m:
            m.setenv(name, value)
            assert S.prune_info(p)["pruned"] == 0 and S.workspace_bytes(p) == need


def test_status_strings(lib):
    assert lib.speckv_status_string(0) == b"ok"
    assert b"workspace" in lib.speckv_status_string(-3)


def test_keep_counts_follow_the_budget_rule(lib):
    p = base_params(seq_lens=[300, 20, 500], c_max=64, n_window=16)
    assert [S.n_keep(p, s) for s in range(3)] == [80, 20, 80]     # min(c_max, m) + n_window
    assert S.total_keep(p) == 180
    assert S.n_keep(p, 3) == -1
    assert S.workspace_bytes(p) > 0 and S.workspace_bytes(p) % 256 == 0


@pytest.mark.parametrize("kw", [
    dict(n_q_heads=7),                       # not a multiple of n_kv_heads
    dict(pool_k=0),
    dict(c_max=-1),
    dict(sm_scale=0.0),
    dict(sm_scale=float("nan")),
    dict(n_window=0, n_lookahead=0),         # no observation rows
    dict(seq_lens=[300, 10]),                # shorter than the window
    dict(seq_lens=[300, 0]),
    dict(n_layers=0),
    dict(q_strides=(1, 1, 1, 3)),            # rows not 16-byte aligned
])
def test_invalid_arguments_are_rejected_before_any_launch(lib, kw):
    p = base_params(**kw)
    assert S.workspace_bytes(p) == 0
    # pointers are never touched when validation fails: dummy non-null values are safe here
    st = lib.speckv_compress(p.ref(), 256, 256, 256, 256, 256, 256, 256, 1 << 40, None)
    assert st == -1


@pytest.mark.parametrize("kw", [dict(head_dim=96), dict(pool_k=257), dict(seq_lens=[64] * 129),
                                dict(n_q_heads=64, n_kv_heads=1, n_lookahead=100)])
def test_unsupported_configurations(lib, kw):
    p = base_params(**kw)
    st = lib.speckv_compress(p.ref(), 256, 256, 256, 256, 256, 256, 256, 1 << 40, None)
    assert st == -2


def test_select_workspace_is_small_and_checked(lib):
    """Selection needs scratch only when few, very long rows are split over workgroups; the size is
    a few MiB, far below the scoring workspace, and a smaller buffer is refused before any launch."""
    short = base_params()
    assert S.select_workspace_bytes(short) == 0
    long_rows = base_params(n_layers=1, seq_lens=[600000], c_max=4096)
    need = S.select_workspace_bytes(long_rows)
    assert 0 < need < S.workspace_bytes(long_rows) and need % 256 == 0 and need < (16 << 20)
    assert S.plan_info(long_rows)["select_parts"] > 1
    assert lib.speckv_select(long_rows.ref(), 256, 256, 256, need - 1, None) == -3
    assert lib.speckv_select(long_rows.ref(), 256, 256, 257, need, None) == -3      # misaligned


def test_device_side_count_needs_one_sequence_and_supported_entry_points(lib):
    """n_in_dev is validated on the host like everything else (the pointer itself is never read
    there): one sequence only, 4-byte aligned, and not for the entry points that do not honour it."""
    p = base_params(seq_lens=[500])
    p.c.n_in_dev = 1024
    need = S.workspace_bytes(p)
    assert need > 0
    two = base_params()
    two.c.n_in_dev = 1024
    assert S.workspace_bytes(two) == 0
    assert lib.speckv_compress(two.ref(), 256, 256, 256, 256, 256, 256, 256, 1 << 40, None) == -2
    p.c.n_in_dev = 1026
    assert lib.speckv_compress(p.ref(), 256, 256, 256, 256, 256, 256, 256, 1 << 40, None) == -1
    p.c.n_in_dev = 1024
    assert lib.specpc_select_tokens(p.ref(), 10, 1, 256, 256, 256, 256, 256, 256, 256, 1 << 40, None) == -2


def test_null_misaligned_and_workspace_errors(lib):
    p = base_params()
    need = S.workspace_bytes(p)
    ok = 256
    assert lib.speckv_compress(p.ref(), None, ok, ok, ok, ok, ok, ok, need, None) == -1
    assert lib.speckv_compress(p.ref(), ok + 2, ok, ok, ok, ok, ok, ok, need, None) == -1     # q misaligned
    assert lib.speckv_compress(p.ref(), ok, ok, ok, ok, ok, None, ok, need, None) == -1       # v without v_out
    assert lib.speckv_compress(p.ref(), ok, ok, ok, ok, ok, ok, None, need, None) == -3
    assert lib.speckv_compress(p.ref(), ok, ok, ok, ok, ok, ok, ok, need - 1, None) == -3
    assert lib.speckv_compress(p.ref(), ok, ok, ok, ok, ok, ok, ok + 16, need, None) == -3    # ws misaligned
    assert lib.speckv_score(p.ref(), ok, ok, None, None, ok, need, None) == -1
    assert lib.speckv_select(p.ref(), None, ok, None, 0, None) == -1
    assert lib.speckv_compact(p.ref(), ok, ok, None, ok, ok, None) == -1
    assert lib.specpc_select_tokens(p.ref(), 10, 2, ok, ok, ok, ok, ok, ok, ok, 1 << 40, None) == -2  # 2 sequences
    one = base_params(seq_lens=[300])
    assert lib.specpc_select_tokens(one.ref(), -1, 2, ok, ok, ok, ok, ok, ok, ok, 1 << 40, None) == -1
    assert lib.specpc_select_tokens(one.ref(), 10, 2, ok, ok, ok, ok, ok, ok, ok, 16, None) == -3
    evs = (ctypes.c_void_p * 7)()
    assert lib.speckv_compress_events(p.ref(), ok, ok, ok, ok, ok, ok, ok, need, None, evs, 7) == -1  # null events
    assert lib.speckv_compress_events(p.ref(), ok, ok, ok, ok, ok, ok, ok, need, None, None, 7) == -1


def test_number_types(lib):
    for dt in (torch.bfloat16, torch.float16, torch.float32):
        assert S.workspace_bytes(base_params(dtype=dt)) > 0
    p = base_params()
    p.c.dtype = 3                                            # not a speckv_dtype
    assert S.workspace_bytes(p) == 0


def test_shared_budget_entry_points_validate(lib):
    p = base_params()
    ok = 256
    need = S.ada_workspace_bytes(p)
    assert need > S.workspace_bytes(p)
    assert lib.speckv_select_ada(p.ref(), -1, ok, ok, ok, ok, need, None) == -1           # negative floor
    assert lib.speckv_select_ada(p.ref(), 3, ok, ok, None, ok, need, None) == -1          # no head_off
    assert lib.speckv_select_ada(p.ref(), 3, ok, ok, ok, ok, need - 1, None) == -3
    assert lib.speckv_compact_ada(p.ref(), ok, ok, ok, None, ok, ok, None) == -1
    assert lib.speckv_compress_ada(p.ref(), 3, ok, ok, ok, ok, ok, ok, ok, None, need, None) == -3
    assert lib.speckv_compress_ada(p.ref(), 3, ok, ok, None, ok, ok, ok, ok, ok, need, None) == -1   # v_out without v
    many = base_params(n_q_heads=256, n_kv_heads=256)
    assert S.ada_workspace_bytes(many) == 0
    assert lib.speckv_select_ada(many.ref(), 3, ok, ok, ok, ok, 1 << 40, None) == -2


def test_binding_refuses_host_tensors(lib):
    p = base_params()
    x = torch.zeros(4)
    with pytest.raises(ValueError):
        S.speckv_select(p, x, x.to(torch.int32))


def test_bench_refuses_more_than_one_gpu(repo_root):
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(repo_root, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True)
    assert r.returncode != 0 and "ONE GPU" in r.stderr


# --------------------------------------------------------------------------- #
# The host's launch plan (no GPU needed)
# --------------------------------------------------------------------------- #
def test_plan_of_the_benchmark_configurations(lib):
    import workloads
    def plan(w):
        return S.plan_info(S.SpecKVParams(
            n_layers=w.n_layers, n_q_heads=w.n_q_heads, n_kv_heads=w.n_kv_heads, head_dim=w.head_dim,
            seq_lens=list(w.seq_lens), n_window=w.n_window, n_lookahead=w.n_lookahead, pool_k=w.pool_k,
            c_max=w.c_max, sm_scale=w.sm_scale, dtype=w.torch_dtype))
    c3 = plan(workloads.llama8b_full_128k())
    # 512 rows per KV group: 8 waves x 2 blocks, one super-block; 4 equal chunks per (layer, head)
    # = 1024 identical workgroups = 4 whole rounds on 256 CUs
    assert (c3["waves"], c3["blocks_per_wave"], c3["row_super_blocks"]) == (8, 2, 1)
    assert c3["chunk_keys"] == 32768 and c3["n_chunks"] == 4 and c3["tile_keys"] == 128
    assert c3["select_parts"] == 1
    c4 = plan(workloads.ragged_batch())
    # G = 7: two super-blocks; ragged lengths: chunks shortened to balance the last round
    assert c4["row_super_blocks"] == 2 and c4["chunk_keys"] == 8192
    c5 = plan(workloads.specpc_draft())
    assert c5["tile_keys"] == 256 and (c5["waves"], c5["blocks_per_wave"]) == (8, 1)
    tiny = plan(workloads.tiny_fp32())
    assert (tiny["waves"], tiny["blocks_per_wave"]) == (4, 1) and tiny["tile_keys"] == 128
    # one layer of the 8B shape: the chunk workgroups and the 8 masked-tail workgroups of a sweep share
    # one launch and fit one round of the 256 CUs together (chunks a little longer than 1/32 of the prompt)
    for n_in in (32768, 131072):
        one = plan(workloads.llama8b_layer(n_in=n_in, n_layers=1))
        kc, kt = one["chunk_keys"], one["tile_keys"]
        unmasked = (n_in - 64 + 1) // kt * kt                       # keys every observation row may see, whole tiles
        assert kc % kt == 0 and one["n_chunks"] == -(-unmasked // kc)
        assert one["n_chunks"] * 8 + 8 <= 256 < -(-unmasked // (kc - kt)) * 8 + 8      # one tile shorter would not fit
        assert one["fixed_reference_rows"] == 0          # one round of workgroups: online step, no repair launch
    # sweeps of several rounds sum their row statistics against fixed references; the Q-stationary
    # kernel (row statistics at d = 64) has its own step
    assert c3["fixed_reference_rows"] == 1 and c4["fixed_reference_rows"] == 1
    assert c5["q_stationary"] & 1 and c5["fixed_reference_rows"] == 0 and tiny["fixed_reference_rows"] == 0


def test_plan_of_small_calls(lib):
    """Up to 8 units: as few tiles a workgroup as keeps a prompt to 20 chunks and the call to one round of the CUs."""
    def plan(units, n, rows, dtype=torch.bfloat16, d=128, G=4):
        info = S.plan_info(S.SpecKVParams(n_layers=1, n_q_heads=G * units, n_kv_heads=units, head_dim=d, seq_lens=[n], n_window=16,
                                          n_lookahead=rows - 16, pool_k=7, c_max=64, sm_scale=0.1, dtype=dtype))
        return info["chunk_keys"], info["n_chunks"]
    assert plan(2, 1024, 32, torch.float32, 64) == (128, 7)
    assert plan(8, 4133, 55) == (256, 16)
    assert plan(8, 2560 + 15, 55) == (128, 20) and plan(8, 2560 + 128 + 15, 55) == (256, 11)
    assert plan(8, 7680 + 15, 55) == (384, 20) and plan(8, 7680 + 128 + 15, 55) == (512, 16)
    assert plan(1, 1280 + 15, 55, torch.float32) == (64, 20) and plan(1, 1280 + 64 + 15, 55, torch.float32) == (128, 11)
    assert plan(8, 2560 + 15, 30, d=64) == (128, 20) and plan(8, 2560 + 15, 128, d=64) == (256, 10)     # tiles of half a row length in LDS
    assert plan(9, 4133, 55) == (512, 8)
    # a length on the device: the kernels cut it; the grid has room for the most chunks of any length up to the bound
    for units, bound in ((8, 7000), (2, 1000), (1, 60000)):
        most = max(plan(units, n, 55)[1] for n in list(range(16, bound, 53)) + [bound])
        p = S.SpecKVParams(n_layers=1, n_q_heads=4 * units, n_kv_heads=units, head_dim=128, seq_lens=[bound], n_window=16,
                           n_lookahead=39, pool_k=7, c_max=64, sm_scale=0.1, dtype=torch.bfloat16)
        need = S.workspace_bytes(p)
        p.c.n_in_dev = 1024
        info = S.plan_info(p)
        assert info["chunk_keys"] == plan(units, bound, 55)[0] and info["n_chunks"] == most
        assert S.workspace_bytes(p) == need


@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 64), (torch.bfloat16, 128), (torch.float32, 128)])
def test_every_super_block_has_rows(lib, dtype, d):
    """Many heads of few rows: what heads padded to whole row blocks need is more than what they need packed."""
    for G in range(1, 129):
        for rows in (2, 3, 7, 17, 31, 33, 40, 65):
            if G * rows > 4096:
                continue
            info = S.plan_info(S.SpecKVParams(n_layers=1, n_q_heads=2 * G, n_kv_heads=2, head_dim=d, seq_lens=[3000], n_window=1,
                                              n_lookahead=rows - 1, pool_k=7, c_max=64, sm_scale=0.1, dtype=dtype))
            blocks, rows_per_wg = -(-G * rows // 32), info["waves"] * info["blocks_per_wave"] * 32
            if -(-rows // 32) * 32 <= rows_per_wg:
                assert info["row_super_blocks"] <= blocks <= info["row_super_blocks"] * rows_per_wg // 32, (G, rows)


def test_row_statistics_mode_follows_the_environment(lib, monkeypatch):
    import workloads
    w = workloads.llama8b_layer(n_in=32768, n_layers=1)
    p = S.SpecKVParams(n_layers=w.n_layers, n_q_heads=w.n_q_heads, n_kv_heads=w.n_kv_heads, head_dim=w.head_dim,
                       seq_lens=list(w.seq_lens), n_window=w.n_window, n_lookahead=w.n_lookahead, pool_k=w.pool_k,
                       c_max=w.c_max, sm_scale=w.sm_scale, dtype=w.torch_dtype)
    assert S.plan_info(p)["fixed_reference_rows"] == 0
    monkeypatch.setenv("SPECKV_ROW_STATISTICS", "fixed")
    assert S.plan_info(p)["fixed_reference_rows"] == 1
    monkeypatch.setenv("SPECKV_ROW_STATISTICS", "online")
    full = workloads.llama8b_full_128k()
    pf = S.SpecKVParams(n_layers=full.n_layers, n_q_heads=full.n_q_heads, n_kv_heads=full.n_kv_heads,
                        head_dim=full.head_dim, seq_lens=list(full.seq_lens), n_window=full.n_window,
                        n_lookahead=full.n_lookahead, pool_k=full.pool_k, c_max=full.c_max, sm_scale=full.sm_scale,
                        dtype=full.torch_dtype)
    assert S.plan_info(pf)["fixed_reference_rows"] == 0


def test_plan_invariants_over_random_shapes(lib):
    import numpy as np
    rng = np.random.default_rng(0)
    for _ in range(300):
        G = int(rng.choice([1, 2, 4, 5, 7, 8, 16]))
        Hkv = int(rng.choice([1, 2, 4, 8]))
        d = int(rng.choice([64, 128]))
        dt = [torch.bfloat16, torch.float16, torch.float32][int(rng.integers(0, 3))]
        w_ = int(rng.choice([0, 16, 64]))
        a_ = int(rng.choice([1, 16, 64, 200]))
        n_seqs = int(rng.choice([1, 1, 3, 16]))
        lens = [int(x) for x in rng.integers(max(1, w_), int(rng.choice([2000, 70000, 1200000])), size=n_seqs)]
        L = int(rng.choice([1, 2, 32]))
        if sum(lens) * L * Hkv > 1 << 31:
            continue
        p = S.SpecKVParams(n_layers=L, n_q_heads=G * Hkv, n_kv_heads=Hkv, head_dim=d, seq_lens=lens,
                           n_window=w_, n_lookahead=a_, pool_k=7, c_max=1024, sm_scale=0.1, dtype=dt)
        out = (ctypes.c_int64 * PLAN_INFO_WORDS)()
        st = lib.speckv_plan_info(p.ref(), out)
        if st == -2:
            continue                                           # outside the supported envelope
        assert st == 0
        info = S.plan_info(p)
        tile, kc = info["tile_keys"], info["chunk_keys"]
        # chunks are whole tiles; below 512 keys, in small calls only, whole tiles as they pass through LDS
        units = L * Hkv * info["row_super_blocks"]
        if kc < 512:
            lds_tile = 128 if tile == 256 and info["blocks_per_wave"] == 1 else tile
            assert units <= 8 and kc % lds_tile == 0 and (info["n_chunks"] + n_seqs) * units <= 256
        else:
            assert kc % tile == 0
        rows_per_wg = info["waves"] * info["blocks_per_wave"] * 32
        rp = (w_ + a_ + 31) // 32 * 32
        if rp > rows_per_wg or (w_ + a_) % 32 == 0 or w_ + a_ == 1:
            assert info["row_super_blocks"] * rows_per_wg >= G * min(rp, rows_per_wg) or rp > rows_per_wg
        else:       # heads share row blocks: room for all of them, and no super-block without any
            assert info["row_super_blocks"] * rows_per_wg >= G * (w_ + a_)
            assert info["row_super_blocks"] <= -(-G * (w_ + a_) // 32)
        # the unmasked chunks cover exactly the whole tiles visible to every row
        want_chunks = 0
        for n in lens:
            visible = min(n, n - w_ + 1)
            want_chunks += -(-(visible // tile * tile) // kc)
        assert info["n_chunks"] == want_chunks
        # rows are split for selection only when they are long and few
        rows = L * n_seqs * Hkv
        if info["select_parts"] > 1:
            assert max(lens) - w_ >= 1 << 18 and rows * info["select_parts"] <= 512 + rows
            assert info["select_parts"] * info["select_part_keys"] >= max(lens) - w_
        assert S.workspace_bytes(p) > 0


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("units", range(1, 9))
def test_workspace_of_a_prompt_suffices_for_every_shorter_one(lib, units, d, dtype):
    """Calls of few (layer, head, super-block) units cut short prompts into shorter chunks than longer ones.  Up to 512 keys
    for every workgroup of the first round; beyond, chunks grow with the prompt."""
    for G, rows in ((4, 32), (4, 128), (1, 600)):
        def need(*lens):
            p = S.SpecKVParams(n_layers=1, n_q_heads=G * units, n_kv_heads=units, head_dim=d, seq_lens=lens, n_window=16,
                               n_lookahead=rows - 16, pool_k=7, c_max=64, sm_scale=0.1, dtype=dtype)
            info = S.plan_info(p)
            return S.workspace_bytes(p), S.ada_workspace_bytes(p), info["row_super_blocks"] * units
        for lens in ([(n,) for n in range(16, 15900, 61)],
                     [(n, 700, 3000) for n in range(16, 9000, 97)] + [(9000, n, 3000) for n in range(700, 1900, 61)]):
            before = (0, 0)
            for ls in lens:
                *now, n_units = need(*ls)
                if n_units > 8:
                    break
                assert now[0] >= before[0] and now[1] >= before[1], (ls, now, before)
                before = now


@pytest.mark.parametrize("heads,kv_heads,d,rows,n_layers,c_max", [
    (32, 8, 128, 128, 3, 512), (32, 8, 128, 128, 32, 2048), (32, 8, 128, 128, 1, 1024), (28, 4, 128, 69, 13, 2048), (28, 4, 128, 128, 28, 512),
    (16, 1, 128, 80, 27, 256), (16, 1, 128, 88, 1, 256), (32, 8, 64, 128, 18, 512), (32, 8, 64, 128, 2, 1024), (8, 2, 64, 96, 67, 256),
    (8, 2, 64, 96, 29, 256),
])
def test_workspace_of_a_long_prompt_suffices_for_every_shorter_one(lib, heads, kv_heads, d, rows, n_layers, c_max):
    """How many chunks a prompt is cut into goes up and down with its length, and with it the scratch of a call, pruned or not."""
    def params(*lens):
        return S.SpecKVParams(n_layers=n_layers, n_q_heads=heads, n_kv_heads=kv_heads, head_dim=d, seq_lens=lens, n_window=64,
                              n_lookahead=rows - 64, pool_k=7, c_max=c_max, sm_scale=0.1, dtype=torch.bfloat16)
    for lens in ([(n,) for n in range(700, 140000, 509)] + [(n,) for n in range(140000, 600000, 9973)],
                 [(n, 17001, 700) for n in range(700, 90000, 1021)]):
        before = (0, 0, 0)
        for ls in lens:
            p = params(*ls)
            now = (S.workspace_bytes(p), S.ada_workspace_bytes(p), S.specpc_workspace_bytes(p, c_max) if len(ls) == 1 else 0)
            assert all(x >= y for x, y in zip(now, before)), (ls, now, before)
            before = now


def test_plain_c_caller(lib, repo_root, tmp_path):
    """The header and the library from a C99 program (host-side entry points only)."""
    import shutil
    import subprocess
    cc = shutil.which("gcc")
    if cc is None:
        pytest.skip("no C compiler")
    pkg = os.path.join(repo_root, "paper_2506_08373_amd")
    exe = str(tmp_path / "c_abi_check")
    subprocess.run([cc, "-std=c99", "-Wall", "-Werror", "-I", os.path.join(repo_root, "include"),
                    os.path.join(repo_root, "tests", "c_abi_check.c"), "-o", exe,
                    "-L", pkg, "-lspeckv", "-Wl,-rpath," + pkg, "-Wl,-rpath,/opt/rocm/lib",
                    "-L", "/opt/rocm/lib", "-lamdhip64"], check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stderr)
    assert "workspace" in r.stdout
