"""What the bf16 attention kernel's plan chooses for the shapes of the GPU tests that are meant for one of its forms, and that it stays within its
workspace.  Host only: nothing is launched."""
import random

import pytest

import paper_2602_08722_amd as pk
from tests import test_gpu_kernel_edges as E
from tests.test_abi import _shape


def _case_shape(case, d=None):
    t_max = max(max(case["kv_lens"]), 1)
    return _shape(pk, batch=case.get("batch", 1), n_q_heads=case["n_q"], n_kv_heads=case["n_kv"], head_dim=d or case["d"],
                  chunk_len=case["chunk"], max_kv_len=t_max, max_budget=min(max(case["budgets"]), t_max))


@pytest.mark.parametrize("cases", ["BF16_SPLIT_CASES", "MERGE_CASES", "MANY_TILES_CASES", "WHOLE_CASES", "ROW_CASES", "UNIT_CASES"])
def test_cases_run_the_form_they_are_meant_for(cases):
    for case in getattr(E, cases):
        for d in (case["d"],) if "d" in case else (64, 128):
            assert pk.quoka_probe_attn_plan(_case_shape(case, d), True) == case["plan"], (case, d)


def test_every_form_of_the_kernel_has_a_case():
    forms = {(d, rows, splits > 1) for name in ("BF16_SPLIT_CASES", "MERGE_CASES", "MANY_TILES_CASES", "WHOLE_CASES", "ROW_CASES", "UNIT_CASES")
             for case in getattr(E, name) for d in ((case["d"],) if "d" in case else (64, 128)) for rows, splits in [case["plan"]]}
    assert forms == {(d, rows, split) for d in (64, 128) for rows in (4, 8) for split in (False, True)}
    assert {2, 3, 4, 5, 8, 9, 32} <= {case["plan"][1] for case in E.MERGE_CASES}


def test_a_shape_or_pointer_that_is_wrong_is_refused():
    assert pk.quoka_probe_attn_plan(_shape(pk, dtype=pk.QUOKA_F32), True) == (0, 0)
    assert pk.quoka_probe_attn_plan(_shape(pk, chunk_len=1), True) == (0, 0)   # decode-sized
    with pytest.raises(pk.QuokaError):
        pk.quoka_probe_attn_plan(_shape(pk, head_dim=96), True)
    import ctypes
    assert pk.load_library().quoka_probe_attn_plan(ctypes.byref(_shape(pk)), 1, None, None) == 1


def test_partials_fit_the_workspace_over_the_range_of_shapes():
    """A split list writes (heads x row blocks x splits) records of 32 rows; the workspace of the shape, and of the same shape with
    longer chunks (a prompt's chunks share one), holds them."""
    rng = random.Random(5)
    for _ in range(3000):
        n_kv, g = rng.choice([(8, 4), (4, 8), (4, 3), (2, 7), (1, 16), (8, 1), (1, 1)])
        d, batch = rng.choice([64, 128]), rng.choice([1, 1, 2, 3, 8, 13, 64])
        chunk, cap = int(2 ** rng.uniform(0, 13)), int(2 ** rng.uniform(0, 17))
        t_max = rng.randint(cap, 2 * cap)
        shape = _shape(pk, batch=batch, n_q_heads=n_kv * g, n_kv_heads=n_kv, head_dim=d, chunk_len=chunk, max_kv_len=t_max, max_budget=cap)
        for sparse in (False, True):
            rows, splits = pk.quoka_probe_attn_plan(shape, sparse)
            if rows == 0:
                assert g * chunk <= 32
                continue
            assert rows in (4, 8) and 1 <= splits <= 32
            records = batch * n_kv * g * -(-chunk // 32) * splits
            tile = 64 if rows == 8 else 128
            assert splits <= -(-(cap if sparse else t_max) // tile) + -(-chunk // tile)   # every share has a tile of a full list
            if splits > 1:
                assert records <= 2048
                assert records * 32 * (d + 2) * 4 <= pk.quoka_workspace_bytes(shape)
                longer = _shape(pk, batch=batch, n_q_heads=n_kv * g, n_kv_heads=n_kv, head_dim=d, chunk_len=min(8192, 2 * chunk),
                                max_kv_len=t_max, max_budget=cap)
                assert records * 32 * (d + 2) * 4 <= pk.quoka_workspace_bytes(longer)


def _plan(n_q, n_kv, d, chunk, cap, batch=1):
    return pk.quoka_probe_attn_plan(_shape(pk, batch=batch, n_q_heads=n_q, n_kv_heads=n_kv, head_dim=d, chunk_len=chunk, max_kv_len=cap,
                                           max_budget=cap), False)


@pytest.mark.parametrize("d", [64, 128])
def test_whole_lists_take_the_block_form_of_their_size(d):
    # few row blocks: four; eight only where blocks of four are more than 256 (260 and 312 here), and in a batch only with room for few keys
    assert _plan(8, 2, d, 65, 130) == (4, 1) and _plan(14, 2, d, 9, 60) == (4, 1)
    assert _plan(12, 4, d, 187, 454, batch=13) == (8, 1)
    assert _plan(12, 4, d, 174, 2616, batch=13)[0] == 4 and _plan(8, 8, d, 279, 2251, batch=13)[0] == 4
    # more than 1024 row blocks: a batch by the number of its groups of eight, one sequence by theirs and, at d 64, by whose keys they are
    assert _plan(32, 8, d, 257, 3000, batch=7) == (8, 1) and _plan(32, 8, d, 160, 3000, batch=8) == (4, 1)
    assert _plan(32, 8, d, 1064, 3000) == (8, 1)
    assert _plan(12, 4, d, 3203, 1) == ((4 if d == 64 else 8), 1)
    assert _plan(32, 8, d, 2240, 3000) == (4, 1)                                   # 280 groups
    assert _plan(32, 8, d, 3500, 1) == ((4 if d == 64 else 8), 1)                  # 440 groups, the chunk's own keys
    assert _plan(32, 8, d, 3500, 9000) == (8, 1) and _plan(32, 8, d, 4800, 1) == (8, 1)
