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
