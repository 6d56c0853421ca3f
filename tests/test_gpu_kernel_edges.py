"""Kernel variants at the sizes where they can go wrong -- edges of tiles and units, remainders, the smallest and largest
of their range -- against the oracle, at the bars of tests/parity.py (float32 sums and bf16 operands respectively)."""
import numpy as np
import pytest
import torch

import gen
from oracle import quoka_oracle as O
from tests import parity as P
from tests.bf16_round import round_to_bf16
from tests.test_gpu_stages import _buffers, _pk

pytestmark = pytest.mark.gpu


def _id(c):
    return "-".join(f"{k}{v}" for k, v in c.items())


def check_attention(case, rows=None, score_flags=0, tol=None):
    """Sparse attention over seeded random index lists of the stated budgets, then dense attention, each with its
    softmax normaliser, against the oracle (every row, or the chunk positions `rows`)."""
    case = dict(case)
    plan, dense_plan = case.pop("plan", None), case.pop("dense_plan", None)
    batch = case.setdefault("batch", 1)
    w = gen.make_custom(n_retain=8, seed=21, **case)
    buf = _buffers(w, score_flags=score_flags)
    if plan is not None:
        assert _pk().quoka_probe_attn_plan(buf.shape, True) == plan
    if dense_plan is not None:
        assert _pk().quoka_probe_attn_plan(buf.shape, False) == dense_plan
    tol = tol or P.TOL_OUT[w.dtype]
    tol_lse = 1e-4 if w.dtype == "f32" else 2e-2
    rng = np.random.default_rng(3)
    lists = []
    for b in range(batch):
        n = min(w.budgets[b], w.kv_lens[b])
        lists.append(np.stack([np.sort(rng.choice(w.kv_lens[b], size=n, replace=False)) if n else np.zeros(0, np.int64)
                               for _ in range(w.n_kv)]))
    host = np.zeros(tuple(buf.k_idx.shape), dtype=np.int32)
    for b in range(batch):
        host[b, :, :lists[b].shape[1]] = lists[b]
    buf.k_idx.copy_(torch.from_numpy(host))
    buf.k_cnt.copy_(torch.from_numpy(np.array([[x.shape[1]] * w.n_kv for x in lists], dtype=np.int32)))
    at = slice(None) if rows is None else rows
    for name in ("sparse", "dense"):
        buf.workspace.fill_(0xA5)
        buf.out.fill_(float("nan"))
        buf.lse.fill_(float("nan"))
        (buf.sparse_attn if name == "sparse" else buf.dense_attn)()
        torch.cuda.synchronize()
        out, lse = gen.from_torch(buf.out), gen.from_torch(buf.lse)
        assert not np.isnan(out).any() and not np.isnan(lse).any()
        for b in range(batch):
            K, V = w.K[b][:, :w.kv_lens[b]], w.V[b][:, :w.kv_lens[b]]
            if name == "sparse":
                want, want_lse = O.sparse_attn(w.Q[b], K, V, lists[b], w.Kc[b], w.Vc[b], True, rows=rows)
            else:
                want, want_lse = O.dense_attn(w.Q[b], K, V, w.Kc[b], w.Vc[b], True, rows=rows)
            err, err_lse = P.max_abs(out[b][:, at], want), P.max_abs(lse[b][:, at], want_lse)
            assert err <= tol and err_lse <= tol_lse, f"{name} b{b}: out {err}, lse {err_lse}"


F32_ATTN_CASES = [
    dict(n_q=2, n_kv=1, d=64, chunk=1, kv_lens=[1], budgets=[1]),            # one row, two keys
    dict(n_q=3, n_kv=1, d=128, chunk=11, kv_lens=[31], budgets=[31]),        # 33 rows; one unit short of full
    dict(n_q=2, n_kv=2, d=64, chunk=32, kv_lens=[33], budgets=[32]),         # exact units, then one key more
    dict(n_q=2, n_kv=1, d=128, chunk=17, kv_lens=[5000], budgets=[2000]),    # 34 rows, the key list split over blocks
    dict(n_q=4, n_kv=1, d=64, chunk=1, kv_lens=[9000], budgets=[513]),       # decode-sized, most splits
    dict(n_q=5, n_kv=1, d=128, chunk=70, kv_lens=[300, 0, 7], budgets=[64, 3, 7], batch=3),
    dict(n_q=16, n_kv=8, d=64, chunk=600, kv_lens=[40], budgets=[5]),        # more row blocks than compute units: no split
    dict(n_q=8, n_kv=2, d=128, chunk=8, kv_lens=[26, 0, 3], budgets=[26, 1, 9], batch=3),   # short lists: one wave per row, up to
    dict(n_q=3, n_kv=3, d=64, chunk=1, kv_lens=[24], budgets=[24]),                          # the line, and one key beyond it
    dict(n_q=3, n_kv=3, d=64, chunk=1, kv_lens=[25], budgets=[25]),
    dict(n_q=4, n_kv=1, d=128, chunk=5, kv_lens=[33], budgets=[32]),
    dict(n_q=4, n_kv=2, d=128, chunk=16, kv_lens=[10], budgets=[3]),
]


@pytest.mark.parametrize("case", F32_ATTN_CASES, ids=_id)
def test_float32_attention_units_rows_and_splits(case):
    check_attention(dict(case, dtype="f32"))


# K rows of float32 units at d 128 go through LDS beyond four units: four, and five, the last one of a single key; eight, and nine and ten, of
# which one and two waves have a second one; a split list (seven units a share, and one where the sequence has but four); and d 64, where none do
@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("case", [
    dict(n_q=2, n_kv=1, chunk=16, kv_lens=[300], budgets=[96]),
    dict(n_q=2, n_kv=1, chunk=16, kv_lens=[300], budgets=[97]),
    dict(n_q=3, n_kv=1, chunk=33, kv_lens=[300], budgets=[192]),
    dict(n_q=300, n_kv=300, chunk=33, kv_lens=[300], budgets=[224]),     # (more row blocks than compute units: not split)
    dict(n_q=300, n_kv=300, chunk=33, kv_lens=[300], budgets=[225]),
    dict(n_q=4, n_kv=2, chunk=70, kv_lens=[900, 31], budgets=[800, 31], batch=2),
], ids=_id)
def test_float32_attention_keys_through_lds(case, d):
    check_attention(dict(case, dtype="f32", d=d), rows=[0, 15] if case["chunk"] == 16 else [0, 31, 32])


# the merge of key splits takes four records at a time, in one group of threads or eight: 2, 4, 5 and 9 splits, the most there are,
# and sequences with fewer units than splits
@pytest.mark.parametrize("case", [
    dict(n_q=2, n_kv=1, d=128, chunk=33, kv_lens=[400], budgets=[300]),
    dict(n_q=2, n_kv=1, d=64, chunk=40, kv_lens=[1000], budgets=[960]),
    dict(n_q=2, n_kv=1, d=128, chunk=3, kv_lens=[1200], budgets=[1100]),
    dict(n_q=5, n_kv=1, d=64, chunk=31, kv_lens=[2300], budgets=[2200]),
    dict(n_q=1, n_kv=1, d=128, chunk=1, kv_lens=[17000], budgets=[16500]),
    dict(n_q=4, n_kv=2, d=64, chunk=9, kv_lens=[4000, 1, 0, 270], budgets=[3900, 1, 2, 40], batch=4),
], ids=_id)
def test_float32_attention_merge_of_splits(case):
    check_attention(dict(case, dtype="f32"))


@pytest.mark.parametrize("n_retain,kv_len,d", [(1, 1, 64), (32, 127, 128), (33, 129, 128), (64, 64, 64), (65, 1000, 128),
                                               (128, 33, 64), (40, 70001, 64)])
def test_float32_scores_query_blocks_and_key_tails(n_retain, kv_len, d):
    w = gen.make_custom(dtype="f32", n_q=2, n_kv=1, d=d, chunk=140, kv_lens=[kv_len], budgets=[1], n_retain=n_retain, seed=22)
    buf = _buffers(w)
    qbar = O.group_mean_queries(w.Q[0], O.select_queries(w.Q[0], n_retain), 1).astype(np.float32)
    buf.qbar.copy_(torch.from_numpy(qbar[None]))
    buf.scores.fill_(float("nan"))
    buf.score_keys()
    torch.cuda.synchronize()
    got = gen.from_torch(buf.scores)[0]
    want = O.key_scores_preagg(qbar.astype(np.float64), w.K[0])
    assert not np.isnan(got).any() and P.max_abs(got, want) <= P.TOL_SCORE


# few queries: plain FMAs up to a number of queries that rises with the keys (3 at first, 26 at most), either side of the line
@pytest.mark.parametrize("score_flags", [0, 1, 2, 8])
@pytest.mark.parametrize("n_q,n_retain,kv_lens,d", [(2, 3, [1, 255, 257], 64), (2, 4, [255], 128), (4, 26, [70001], 64),
                                                    (4, 17, [70001, 0], 64), (4, 27, [70001], 64), (4, 23, [70001], 128), (2, 1, [513], 128)])
def test_float32_scores_of_few_queries(n_q, n_retain, kv_lens, d, score_flags):
    n_kv = 1 if n_q == 2 else 4
    w = gen.make_custom(dtype="f32", n_q=n_q, n_kv=n_kv, d=d, chunk=140, kv_lens=kv_lens, budgets=[1] * len(kv_lens),
                        n_retain=n_retain, batch=len(kv_lens), seed=24)
    buf = _buffers(w, score_flags=score_flags)
    qbar = np.stack([O.group_mean_queries(w.Q[b], O.select_queries(w.Q[b], n_retain), n_kv) for b in range(w.batch)]).astype(np.float32)
    buf.qbar.copy_(torch.from_numpy(qbar))
    buf.scores.fill_(float("nan"))
    buf.score_keys()
    torch.cuda.synchronize()
    q = round_to_bf16(qbar) if score_flags & 8 else qbar
    for b in range(w.batch):
        got = gen.from_torch(buf.scores)[b][:, :w.kv_lens[b]]
        K = w.K[b][:, :w.kv_lens[b]].astype(np.float64)
        dots = np.einsum("hrd,htd->hrt", q[b].astype(np.float64), K)
        want = dots.mean(axis=1) if score_flags & 2 else dots.max(axis=1)
        if not score_flags & 1:
            want = want / np.maximum(np.linalg.norm(K, axis=-1), 1e-8)
        # (float32 sums of d products: about sqrt(d) 2^-24 of |q| |k|, and |k| is about sqrt(d))
        assert not np.isnan(got).any() and (not got.size or P.max_abs(got, want) <= P.TOL_SCORE * (np.sqrt(d) * 1.5 if score_flags & 1 else 1))


# The bf16 prefill kernel chooses blocks of eight or four row blocks and how many of them share a key list by a model of the call.
# `plan` says what a case is meant to run, (row blocks per block, splits) of the sparse call: a change of the model that takes a case
# elsewhere fails (tests/test_attn_plan.py, without a GPU), and the case is to be chosen anew.
# Key lists split over blocks (few row blocks); the second sequence of a batch has fewer tiles than there are splits, so some blocks
# get none
BF16_SPLIT_CASES = [
    dict(n_q=8, n_kv=2, d=128, chunk=9, kv_lens=[6000, 3], budgets=[1500, 3], batch=2, plan=(4, 13)),
    dict(n_q=2, n_kv=1, d=64, chunk=33, kv_lens=[4097], budgets=[640], plan=(4, 6)),
    dict(n_q=7, n_kv=1, d=128, chunk=65, kv_lens=[2500], budgets=[2500], plan=(4, 11)),
    dict(n_q=2, n_kv=2, d=128, chunk=129, kv_lens=[1, 5000, 0], budgets=[1, 1100, 9], batch=3, plan=(4, 11)),
    dict(n_q=2, n_kv=1, d=128, chunk=33, kv_lens=[1000], budgets=[640], plan=(8, 11)),   # a tile each
]


@pytest.mark.parametrize("scale_f32", [False, True], ids=["", "scale-f32"])
@pytest.mark.parametrize("case", BF16_SPLIT_CASES, ids=_id)
def test_bf16_attention_key_splits(case, scale_f32):
    check_attention(dict(case, dtype="bf16"), score_flags=16 if scale_f32 else 0)


def test_bf16_attention_key_splits_of_a_batch_in_one_round():
    # 104 blocks of two row blocks: the dense call's lists are shared by two blocks, one round
    check_attention(dict(dtype="bf16", n_q=16, n_kv=8, d=64, chunk=17, kv_lens=[3000 - 230 * i for i in range(13)],
                         budgets=[700] * 13, batch=13, plan=(4, 1), dense_plan=(4, 2)), rows=[0, 8, 16])


def test_bf16_attention_key_splits_of_eight_row_blocks():
    # 48 groups of eight row blocks on 256 compute units, which the plan splits five ways
    check_attention(dict(dtype="bf16", n_q=8, n_kv=8, d=128, chunk=1341, kv_lens=[5000], budgets=[3000], plan=(8, 5)),
                    rows=[0, 1, 31, 32, 700, 1311, 1312, 1340])


# the merge of key splits takes four records at a time and up to eight waves: 2 to 5 splits, 7 to 9, and the most there are
MERGE_CASES = [
    dict(n_q=32, n_kv=8, d=64, chunk=333, kv_lens=[2000], budgets=[1990], plan=(4, 2)),
    dict(n_q=7, n_kv=1, d=128, chunk=333, kv_lens=[300], budgets=[299], plan=(4, 3)),
    dict(n_q=14, n_kv=2, d=128, chunk=65, kv_lens=[300], budgets=[290], plan=(4, 1)),
    dict(n_q=2, n_kv=1, d=64, chunk=333, kv_lens=[150], budgets=[150], plan=(4, 1)),
    dict(n_q=4, n_kv=1, d=128, chunk=130, kv_lens=[700], budgets=[640], plan=(4, 4)),
    dict(n_q=1, n_kv=1, d=64, chunk=33, kv_lens=[300], budgets=[290], plan=(4, 4)),
    dict(n_q=4, n_kv=1, d=128, chunk=130, kv_lens=[300], budgets=[290], plan=(8, 4)),
    dict(n_q=1, n_kv=1, d=64, chunk=130, kv_lens=[300], budgets=[290], plan=(4, 5)),
    dict(n_q=7, n_kv=1, d=128, chunk=130, kv_lens=[1000], budgets=[1000], plan=(4, 5)),
    dict(n_q=1, n_kv=1, d=64, chunk=33, kv_lens=[700], budgets=[700], plan=(4, 7)),
    dict(n_q=1, n_kv=1, d=64, chunk=130, kv_lens=[700], budgets=[700], plan=(4, 8)),
    dict(n_q=1, n_kv=1, d=128, chunk=130, kv_lens=[300], budgets=[290], plan=(8, 8)),
    dict(n_q=1, n_kv=1, d=64, chunk=333, kv_lens=[700], budgets=[690], plan=(4, 9)),
    dict(n_q=1, n_kv=1, d=128, chunk=333, kv_lens=[200], budgets=[129], plan=(8, 9)),
    dict(n_q=1, n_kv=1, d=128, chunk=33, kv_lens=[20000], budgets=[19000], plan=(4, 30)),      # one token in the second row block
    dict(n_q=1, n_kv=1, d=64, chunk=1000, kv_lens=[19000], budgets=[19000], plan=(4, 32)),
    dict(n_q=3, n_kv=1, d=64, chunk=33, kv_lens=[9000, 2, 0, 4000], budgets=[8000, 2, 1, 40], batch=4, plan=(4, 22)),   # neutral records
]


@pytest.mark.parametrize("case", MERGE_CASES, ids=_id)
def test_bf16_attention_merge_of_splits(case):
    check_attention(dict(case, dtype="bf16"), rows=[0, 31, 32, 500, 999] if case["chunk"] == 1000 else None)


# shares of many tiles in blocks of eight row blocks, at d 64 staged through registers: 131 tiles over four blocks, whose shares begin
# at tiles of either stage; a sequence whose shares differ by a tile and one with fewer tiles than blocks
MANY_TILES_CASES = [
    dict(n_q=12, n_kv=4, d=64, chunk=333, kv_lens=[8000, 5003, 64], budgets=[8000, 5003, 64], batch=3, plan=(8, 4)),
    dict(n_q=32, n_kv=8, d=128, chunk=333, kv_lens=[5000], budgets=[5000], plan=(8, 5)),
]


@pytest.mark.parametrize("scale_f32", [False, True], ids=["", "scale-f32"])
@pytest.mark.parametrize("case", MANY_TILES_CASES, ids=_id)
def test_bf16_attention_shares_of_many_tiles(case, scale_f32):
    check_attention(dict(case, dtype="bf16"), rows=[0, 31, 32, 63, 64, 100, 200, 320, 332], score_flags=16 if scale_f32 else 0)


# a wave works in units of 32 keys, the first of them formed ahead of the loop, the last without a successor: lists that end within and
# at the end of the first and second unit of the first and second tile, chunks whose row blocks start in either unit of a tile;
# blocks of four row blocks (chunk 97: the second wave set sees nothing of the first chunk tile) and of eight (batches of 32 heads)
UNIT_CASES = [
    dict(n_q=4, n_kv=2, chunk=97, kv_lens=[1, 33, 64, 65], budgets=[1, 33, 64, 65], batch=4, plan=(4, 1)),
    dict(n_q=4, n_kv=2, chunk=128, kv_lens=[127, 128, 129, 0], budgets=[127, 128, 129, 0], batch=4, plan=(4, 1)),
    # nothing for the second set in the last cache tile
    dict(n_q=4, n_kv=2, chunk=289, kv_lens=[1, 64, 130, 0], budgets=[1, 64, 130, 0], batch=4, plan=(4, 1)),
    dict(n_q=64, n_kv=16, chunk=289, kv_lens=[31, 32, 63, 130], budgets=[31, 32, 63, 130], batch=4, plan=(8, 1)),
]


@pytest.mark.parametrize("scale_f32", [False, True], ids=["", "scale-f32"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("case", UNIT_CASES, ids=_id)
def test_bf16_attention_units_and_runs_of_tiles(case, d, scale_f32):
    check_attention(dict(case, dtype="bf16", d=d), score_flags=16 if scale_f32 else 0)


# bf16 rounds every probability but 1: those of the keys that hold a row's largest score are exact where that score is the row's
# reference point.  Chunks whose first 64 keys are all that counts (half of them at probability 1, half at 3/4, whose values cancel) and
# whose other keys, a few octaves below, have values of zero: a sum of exact probabilities is exactly zero, while a reference point taken
# from another tile first scales both by 2^4.55, which rounds the one up and the other down and leaves up to 1e-3.
@pytest.mark.parametrize("score_flags", [0, 16])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("chunk,kv_len", [(1100, 0), (1100, 100), (2240, 0), (2240, 257)])
def test_bf16_attention_takes_the_reference_point_from_the_first_keys(chunk, kv_len, d, score_flags):
    n_q, n_kv = 32, 8
    r = np.float32(1.4426950408889634) / np.sqrt(np.float32(d))
    if not score_flags:
        r = round_to_bf16(np.array([r]))[0]
    shift = 4.55

    def key(log2p):   # q = (1, 2^-8, 2^-16): the score in three pieces of eight bits
        rest, pieces = log2p / float(r), []
        for i in range(3):
            piece = float(round_to_bf16(np.array([rest * 256.0 ** i], dtype=np.float32))[0])
            pieces.append(piece)
            rest -= piece / 256.0 ** i
        return torch.tensor(pieces)

    for p in (2.0 ** shift, 0.75 * 2.0 ** shift):   # (what the shifted probabilities round to)
        assert abs(float(round_to_bf16(np.array([p], dtype=np.float32))[0]) / p - 1) > 1e-3
    q = torch.zeros(1, n_q, chunk, d)
    q[..., :3] = torch.tensor([1.0, 2.0 ** -8, 2.0 ** -16])
    kc = torch.zeros(1, n_kv, chunk, d)
    kc[..., 1:64:2, :3] = key(np.log2(0.75))
    kc[..., 64:, :3] = key(-shift)
    vc = torch.zeros(1, n_kv, chunk, d)
    vc[..., 0:64:2, :], vc[..., 1:64:2, :] = 0.75, -1.0
    k = torch.zeros(1, n_kv, max(kv_len, 1), d)
    k[..., :3] = key(-shift)
    dev = lambda t: t.to("cuda:0", torch.bfloat16)
    buf = _pk().ChunkBuffers(dev(q), dev(k), dev(torch.zeros_like(k)), dev(kc), dev(vc), [kv_len], [0], 8, score_flags=score_flags)
    four = chunk == 2240   # blocks of four row blocks, of eight
    assert _pk().quoka_probe_attn_plan(buf.shape, False) == (4 if four else 8, 1)
    buf.dense_attn()
    torch.cuda.synchronize()
    assert bool((buf.out[:, :, 64:] == 0).all()), float(buf.out[:, :, 64:].abs().max())


# whole key lists of one sequence: one round of blocks of eight row blocks (130 of them, the last one not full), two rounds of
# blocks of four at d 64 (lists of the chunk's own keys), three at either head size (264 groups of eight), two rounds of blocks of eight
WHOLE_CASES = [
    dict(n_q=16, n_kv=1, d=64, chunk=2070, kv_lens=[3000], budgets=[2500], plan=(8, 1)),
    dict(n_q=16, n_kv=1, d=64, chunk=2070, kv_lens=[0], budgets=[1], plan=(4, 1)),
    dict(n_q=7, n_kv=1, d=128, chunk=4803, kv_lens=[700], budgets=[129], plan=(8, 1)),
    dict(n_q=32, n_kv=8, d=64, chunk=2081, kv_lens=[100], budgets=[65], plan=(4, 1)),
    dict(n_q=28, n_kv=4, d=128, chunk=2400, kv_lens=[300], budgets=[65], plan=(4, 1)),
    dict(n_q=28, n_kv=4, d=64, chunk=2400, kv_lens=[300], budgets=[129], plan=(4, 1)),
    dict(n_q=64, n_kv=4, d=128, chunk=1569, kv_lens=[130], budgets=[100], plan=(8, 1)),
]


@pytest.mark.parametrize("case", WHOLE_CASES, ids=_id)
def test_bf16_attention_whole_lists_of_one_sequence(case):
    check_attention(dict(case, dtype="bf16"), rows=[0, 31, 32, 1000, case["chunk"] - 33, case["chunk"] - 1])


# rows go out through LDS, which the waves' hand-over records (blocks of four) or the tiles (blocks of eight) held before: every row,
# the last row block not full, into contiguous outputs and into rows that lie apart, whose gaps stay as they are
ROW_CASES = [
    dict(n_q=16, n_kv=2, d=128, chunk=2070, kv_lens=[50], budgets=[40], plan=(8, 1)),
    dict(n_q=16, n_kv=2, d=64, chunk=2070, kv_lens=[50], budgets=[40], plan=(4, 1)),
    dict(n_q=28, n_kv=4, d=128, chunk=2400, kv_lens=[50], budgets=[40], plan=(4, 1)),      # rounds of blocks of four
    dict(n_q=14, n_kv=2, d=64, chunk=5, kv_lens=[129], budgets=[129], plan=(4, 1)),        # few rows: stored as the registers lie; 63 of
    dict(n_q=14, n_kv=2, d=128, chunk=9, kv_lens=[130], budgets=[129], plan=(4, 1)),       # them, and 64, which go out whole
    dict(n_q=16, n_kv=2, d=128, chunk=8, kv_lens=[130], budgets=[129], plan=(4, 1)),
    dict(n_q=4, n_kv=2, d=64, chunk=31, kv_lens=[60], budgets=[50], plan=(4, 1)),          # 62, one head a row block
    dict(n_q=4, n_kv=2, d=64, chunk=97, kv_lens=[70], budgets=[65], plan=(4, 1)),
    dict(n_q=14, n_kv=2, d=128, chunk=9, kv_lens=[60], budgets=[50], plan=(4, 1)),
    dict(n_q=16, n_kv=2, d=128, chunk=8, kv_lens=[60], budgets=[50], plan=(4, 1)),
    dict(n_q=16, n_kv=2, d=128, chunk=2070, kv_lens=[3000], budgets=[2500], plan=(8, 1)),
    dict(n_q=16, n_kv=2, d=64, chunk=2070, kv_lens=[3000], budgets=[2500], plan=(8, 1)),   # (as the registers lie)
]


@pytest.mark.parametrize("scale_f32", [False, True], ids=["", "scale-f32"])
@pytest.mark.parametrize("case", ROW_CASES, ids=_id)
def test_bf16_attention_rows_of_whole_lists(case, scale_f32):
    flags, rows = 16 if scale_f32 else 0, sorted({0, 1, case["chunk"] // 2, case["chunk"] - 2, case["chunk"] - 1})
    check_attention(dict(case, dtype="bf16"), rows=rows, score_flags=flags)
    w = gen.make_custom(dtype="bf16", n_retain=8, seed=22, batch=1, **{k: v for k, v in case.items() if k != "plan"})
    buf = _buffers(w, score_flags=flags)
    n, d = w.budgets[0], w.d
    buf.k_idx.copy_(torch.arange(n, dtype=torch.int32).expand(1, w.n_kv, n))
    buf.k_cnt.fill_(n)
    buf.sparse_attn()
    wide = torch.full((1, w.n_q, w.chunk, d + 24), 7.0, dtype=torch.bfloat16, device="cuda:0")
    buf.shape.o_stride[:] = wide.stride()[:3]
    buf.sparse_attn(out=wide[..., :d])
    torch.cuda.synchronize()
    assert torch.equal(wide[..., :d], buf.out) and bool((wide[..., d:] == 7.0).all())


# the first fetches of a block with a whole list leave before its length is known: lists that fill their first tile, one short of it, and empty, in
# arrays whose unused entries are out of range, in every form of the kernel and with queries whose tokens lie apart
@pytest.mark.parametrize("scale_f32", [False, True], ids=["", "scale-f32"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("case,counts", [
    (dict(n_q=16, n_kv=2, chunk=9, kv_lens=[200], budgets=[129], plan=(4, 1)), [129, 128, 127, 65, 1, 0]),
    (dict(n_q=16, n_kv=2, chunk=2070, kv_lens=[3000], budgets=[2500], plan=(8, 1)), [2500, 65, 64, 63, 1, 0]),
    (dict(n_q=14, n_kv=2, chunk=5, kv_lens=[200], budgets=[129], plan=(4, 1)), [129, 128, 127, 65, 1, 0]),     # rows stored as the registers lie
    (dict(n_q=14, n_kv=2, chunk=40, kv_lens=[3000], budgets=[2500], plan=(4, 11)), [2500, 129, 127, 64, 1, 0]),   # shared lists
    (dict(n_q=12, n_kv=4, chunk=1421, kv_lens=[3000], budgets=[2500], plan=(8, 3)), [2500, 65, 64, 63, 1, 0]),
], ids=["four", "eight", "four-few-rows", "four-shared", "eight-shared"])
def test_bf16_attention_lists_shorter_than_their_array(case, counts, d, scale_f32):
    case = dict(case)
    plan, chunk = case.pop("plan"), case["chunk"]
    w = gen.make_custom(dtype="bf16", d=d, n_retain=8, batch=1, seed=4, **case)
    buf = _buffers(w, score_flags=16 if scale_f32 else 0)
    got = _pk().quoka_probe_attn_plan(buf.shape, True)
    assert got == plan, got
    apart = torch.full((1, w.n_q, chunk, d + 8), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    apart[..., :d] = buf.q
    buf.q = apart[..., :d]
    buf.shape.q_stride[:] = buf.q.stride()[:3]
    rows = sorted({0, 1, chunk // 2, chunk - 1})
    rng = np.random.default_rng(d)
    n_most, n_keys = w.budgets[0], w.kv_lens[0]
    for n in counts:
        lists = np.stack([np.sort(rng.choice(n_keys, size=n, replace=False)) for _ in range(w.n_kv)]).astype(np.int32)
        host = np.full(tuple(buf.k_idx.shape), 0x7FFFFFFF, dtype=np.int32)
        host[0, :, n:n_most:2] = -1
        host[0, :, :n] = lists
        buf.k_idx.copy_(torch.from_numpy(host))
        buf.k_cnt.fill_(n)
        buf.out.fill_(float("nan"))
        buf.sparse_attn()
        torch.cuda.synchronize()
        out = gen.from_torch(buf.out[0])
        assert not np.isnan(out).any()
        want = O.sparse_attn(w.Q[0], w.K[0], w.V[0], lists, w.Kc[0], w.Vc[0], rows=rows)
        assert P.max_abs(out[:, rows], want) <= P.TOL_OUT["bf16"], n


# no room for selected keys at all: the entry that the kernels fetch ahead is none of a list's, in units and a wave a row (float32), decode of one
# sequence and of a batch, blocks of four and of eight
@pytest.mark.parametrize("case", [
    dict(dtype="f32", n_q=4, n_kv=2, d=64, chunk=40, kv_lens=[70], budgets=[0]),
    dict(dtype="f32", n_q=4, n_kv=2, d=128, chunk=200, kv_lens=[70], budgets=[0]),
    dict(dtype="f32", n_q=4, n_kv=2, d=128, chunk=2, kv_lens=[70], budgets=[0]),
    dict(dtype="bf16", n_q=4, n_kv=2, d=128, chunk=1, kv_lens=[70], budgets=[0]),
    dict(dtype="bf16", n_q=4, n_kv=2, d=64, chunk=8, kv_lens=[70, 9], budgets=[0, 0], batch=2),
    dict(dtype="bf16", n_q=14, n_kv=2, d=64, chunk=9, kv_lens=[70], budgets=[0]),
    dict(dtype="bf16", n_q=14, n_kv=2, d=128, chunk=300, kv_lens=[70], budgets=[0]),
    dict(dtype="bf16", n_q=52, n_kv=52, d=128, chunk=700, kv_lens=[70], budgets=[0]),
], ids=_id)
def test_attention_without_room_for_selected_keys(case):
    check_attention(case, rows=sorted({0, case["chunk"] // 2, case["chunk"] - 1}))


# decode kernel: single slots, tiles of 32 short of and past full, fewer tiles than waves or blocks, batches whose shares
# of the blocks differ, batches beyond one wave's lanes
DECODE_CASES = [
    dict(n_q=1, n_kv=1, d=64, chunk=1, kv_lens=[0], budgets=[1]),
    dict(n_q=4, n_kv=1, d=128, chunk=8, kv_lens=[31], budgets=[24]),
    dict(n_q=8, n_kv=2, d=128, chunk=1, kv_lens=[4100], budgets=[127]),
    dict(n_q=16, n_kv=1, d=64, chunk=2, kv_lens=[20000], budgets=[20000]),
    dict(n_q=8, n_kv=4, d=128, chunk=3, kv_lens=[9000, 1, 700, 0, 3333], budgets=[1000, 1, 96, 5, 333], batch=5),
    dict(n_q=8, n_kv=8, d=64, chunk=3, kv_lens=[9000, 100, 6000], budgets=[9000, 50, 700], batch=3),   # two blocks a unit
    dict(n_q=16, n_kv=8, d=64, chunk=2, kv_lens=[300 + 11 * i for i in range(20)], budgets=[90] * 20, batch=20),
    dict(n_q=2, n_kv=1, d=64, chunk=1, kv_lens=[(97 * i) % 1511 for i in range(66)],
         budgets=[(97 * i) % 1511 // 4 + 1 for i in range(66)], batch=66),
]


@pytest.mark.parametrize("case", DECODE_CASES, ids=lambda c: _id({k: v for k, v in c.items() if k not in ("kv_lens", "budgets")}))
def test_decode_attention_tiles_and_shares(case):
    check_attention(dict(case, dtype="bf16"))


# more than two tiles a wave have a form of their own: two, and one tile more, of one sequence (two blocks a head) and of a ragged batch (six)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("case", [
    dict(n_q=256, n_kv=256, chunk=1, kv_lens=[520], budgets=[511]),
    dict(n_q=256, n_kv=256, chunk=1, kv_lens=[511], budgets=[511]),
    dict(n_q=256, n_kv=256, chunk=1, kv_lens=[520], budgets=[512]),
    dict(n_q=512, n_kv=128, chunk=2, kv_lens=[766, 95], budgets=[766, 40], batch=2),
    dict(n_q=512, n_kv=128, chunk=2, kv_lens=[780, 95], budgets=[767, 40], batch=2),
], ids=_id)
def test_decode_attention_two_tiles_a_wave_and_more(case, d):
    check_attention(dict(case, dtype="bf16", d=d))


# one sequence: the kernels look a full list up before they know its length; lists that are full, one short of it, of fewer tiles or
# splits, and empty, in arrays whose unused entries are out of range, and partials left by a longer list
@pytest.mark.parametrize("count", [1600, 1599, 1500, 400, 127, 32, 1, 0])
@pytest.mark.parametrize("d,chunk", [(128, 1), (64, 8), (128, 5)])
def test_decode_attention_lists_of_one_sequence_shorter_than_their_array(d, chunk, count):
    w = gen.make_custom(dtype="bf16", n_q=8, n_kv=2, d=d, chunk=chunk, n_retain=8, kv_lens=[2000], budgets=[1600], batch=1, seed=4)
    buf = _buffers(w)
    rng = np.random.default_rng(count)
    lists = np.stack([np.sort(rng.choice(2000, size=1600, replace=False)) for _ in range(w.n_kv)]).astype(np.int32)
    full = np.full(tuple(buf.k_idx.shape), 0x7FFFFFFF, dtype=np.int32)
    for n in (1600, count):   # (the full list first: its partials are still there when the short one is merged)
        host = full.copy()
        host[0, :, :n] = lists[:, :n]
        buf.k_idx.copy_(torch.from_numpy(host))
        buf.k_cnt.fill_(n)
        buf.out.fill_(float("nan"))
        buf.lse.fill_(float("nan"))
        buf.sparse_attn()
        torch.cuda.synchronize()
        want, want_lse = O.sparse_attn(w.Q[0], w.K[0], w.V[0], lists[:, :n], w.Kc[0], w.Vc[0], True)
        assert P.max_abs(gen.from_torch(buf.out[0]), want) <= P.TOL_OUT["bf16"]
        assert P.max_abs(gen.from_torch(buf.lse[0]), want_lse) <= 2e-2


# entries are fetched a unit or a tile ahead, for slots that hold a chunk row or nothing too: float32 units and decode tiles of a batch, lists
# around whole units, of one entry and empty, in arrays whose unused entries are out of range
@pytest.mark.parametrize("dtype,d,chunk", [("f32", 64, 40), ("f32", 128, 7), ("bf16", 128, 3), ("bf16", 64, 8)])
def test_entries_fetched_ahead_of_their_use(dtype, d, chunk):
    w = gen.make_custom(dtype=dtype, n_q=4, n_kv=2, d=d, chunk=chunk, n_retain=8, kv_lens=[700, 650], budgets=[600, 600], batch=2, seed=5)
    buf = _buffers(w)
    rng = np.random.default_rng(d)
    for counts in ((600, 257), (256, 0), (1, 255), (0, 33)):
        host = np.full(tuple(buf.k_idx.shape), 0x7FFFFFFF, dtype=np.int32)
        host[:, :, 1::2] = -1
        lists = []
        for b, n in enumerate(counts):
            lists.append(np.stack([np.sort(rng.choice(w.kv_lens[b], size=n, replace=False)) for _ in range(w.n_kv)]).astype(np.int32))
            host[b, :, :n] = lists[b]
        buf.k_idx.copy_(torch.from_numpy(host))
        buf.k_cnt.copy_(torch.tensor([[n] * w.n_kv for n in counts], dtype=torch.int32))
        buf.out.fill_(float("nan"))
        buf.sparse_attn()
        torch.cuda.synchronize()
        for b in range(2):
            want = O.sparse_attn(w.Q[b], w.K[b], w.V[b], lists[b], w.Kc[b], w.Vc[b])
            assert P.max_abs(gen.from_torch(buf.out[b]), want) <= P.TOL_OUT[dtype], (b, counts)


# top-B: the fused call and the stage calls against a sort of the same scores, bit for bit, whatever the scores look
# like (ties at the cut, one score only, more keys in the cut bin than LDS takes, edges of the keys held per thread)
BINNED_CASES = [
    ("normal", dict(kv_lens=[1024, 33, 1], budgets=[100, 32, 1], batch=3)),
    ("normal", dict(kv_lens=[1025, 1, 0], budgets=[1024, 9, 3], batch=3)),
    ("normal", dict(kv_lens=[32768], budgets=[3932])),
    ("normal", dict(kv_lens=[16385], budgets=[16384])),
    ("pairs", dict(kv_lens=[20480, 20000], budgets=[2481, 19999], batch=2)),   # 20, 24, 28 keys a thread, full and not
    ("normal", dict(kv_lens=[20481], budgets=[700])),
    ("normal", dict(kv_lens=[24576, 24577], budgets=[24575, 3], batch=2)),
    ("pairs", dict(kv_lens=[16384], budgets=[5001])),
    ("normal", dict(kv_lens=[5000], budgets=[1], chunk=1, n_retain=8)),
    ("pairs", dict(kv_lens=[6001], budgets=[777])),            # every score twice: ties at the cut
    ("equal", dict(kv_lens=[9000], budgets=[4000])),           # one score only: more keys in the cut's bin than LDS takes
    ("normal", dict(kv_lens=[3000], budgets=[400], dtype="f32", d=64)),
    ("pairs", dict(kv_lens=[20000, 7], budgets=[5000, 7], batch=2, dtype="f32")),
]


@pytest.mark.parametrize("kind,case", BINNED_CASES, ids=lambda x: _id(x) if isinstance(x, dict) else x)
def test_top_b_cut_bins_ties_and_shares(kind, case):
    case = dict(dict(dtype="bf16", n_q=4, n_kv=2, d=128, chunk=40, n_retain=16, batch=1), **case)
    w = gen.make_custom(seed=23, **case)
    if kind == "equal":
        w.K[:] = w.K[:, :, :1]
    elif kind == "pairs":
        n = w.K.shape[2] // 2 * 2
        w.K[:, :, 1:n:2] = w.K[:, :, 0:n:2]
    for fused in (False, True):
        buf = _buffers(w)
        buf.workspace.fill_(0xA5)
        buf.k_idx.fill_(-1)
        buf.k_cnt.fill_(-1)
        if fused:
            buf.chunk_attn()
        else:
            buf.select_queries()
            buf.score_keys()
            buf.topk_keys()
        torch.cuda.synchronize()
        scores, idx, cnt = gen.from_torch(buf.scores), gen.from_torch(buf.k_idx), gen.from_torch(buf.k_cnt)
        for b in range(w.batch):
            want = O.topk_keys(scores[b][:, :w.kv_lens[b]], w.budgets[b])
            assert np.all(cnt[b] == want.shape[1])
            assert np.array_equal(idx[b][:, :want.shape[1]], want), f"fused {fused} b{b}"


@pytest.mark.parametrize("T,B", [(700, 90), (1024, 1023), (9001, 4500), (20011, 300), (32768, 32767)])
def test_top_b_of_scores_that_are_not_finite(T, B):
    """A NaN score ranks as the infinity of its sign; the list stays full, ascending and inside the cache."""
    w = gen.make_custom(dtype="bf16", n_q=2, n_kv=2, d=64, chunk=40, n_retain=16, kv_lens=[T], budgets=[B], batch=1, seed=3)
    rng = np.random.default_rng(11)
    for share in (0.0, 0.001, 0.5, 1.0):
        buf = _buffers(w)
        s = rng.standard_normal((2, T)).astype(np.float32)
        odd = rng.random((2, T)) < share
        s[odd] = rng.choice(np.array([np.nan, -np.nan, np.inf, -np.inf], dtype=np.float32), size=int(odd.sum()))
        buf.scores.copy_(torch.from_numpy(s)[None])
        buf.k_idx.fill_(-1)
        buf.topk_keys()
        torch.cuda.synchronize()
        ranked = np.where(np.isnan(s), np.copysign(np.float32(np.inf), s), s)
        want = np.stack([np.sort(np.argsort(-r, kind="stable")[:B]) for r in ranked])
        assert np.array_equal(gen.from_torch(buf.k_idx)[0][:, :B], want), share


@pytest.mark.parametrize("T,B", [(9001, 4500), (32768, 20000), (32769, 20000), (70001, 30000)])
def test_top_b_ties_of_signed_zeros_and_nan_on_both_sides_of_the_register_path(T, B):
    """Equal scores go to the lower position, whatever the sign of a zero, and a NaN ranks as the infinity of its sign:
    the register path (up to 32768 scores) and the multi-block path alike."""
    w = gen.make_custom(dtype="bf16", n_q=2, n_kv=2, d=64, chunk=40, n_retain=16, kv_lens=[T], budgets=[B], batch=1, seed=3)
    rng = np.random.default_rng(12)
    zeros = rng.choice(np.array([0.0, -0.0], dtype=np.float32), size=(2, T))
    zeros[:, ::9] = rng.choice(np.array([1.5, -1.5], dtype=np.float32), size=zeros[:, ::9].shape)
    odd = rng.standard_normal((2, T)).astype(np.float32)
    at = rng.random((2, T)) < 0.5 * B / T   # (the cut lies among the infinities where B is small)
    odd[at] = rng.choice(np.array([np.nan, -np.nan, np.inf, -np.inf], dtype=np.float32), size=int(at.sum()))
    odd[:, 5:T:max(1, 2 * T // (3 * B))] = np.inf
    for s in (zeros, odd):
        buf = _buffers(w)
        buf.scores.copy_(torch.from_numpy(s)[None])
        buf.workspace.fill_(0xA5)
        buf.k_idx.fill_(-1)
        buf.topk_keys()
        torch.cuda.synchronize()
        ranked = np.where(np.isnan(s), np.copysign(np.float32(np.inf), s), s)
        want = np.stack([np.sort(np.argsort(-r, kind="stable")[:B]) for r in ranked])
        assert np.array_equal(gen.from_torch(buf.k_idx)[0][:, :B], want)


def check_crowded_top_b(T, crowd):
    """Two heads of T scores, `crowd` of them within a thousandth of a bin around the cut, a third of these equal."""
    rng = np.random.default_rng(T + crowd)
    s = rng.standard_normal((2, T)).astype(np.float32)
    B = max(1, T // 3)
    if crowd:
        at = np.stack([rng.choice(T, size=crowd, replace=False) for _ in range(2)])
        cut = np.sort(s, axis=1)[:, T - B][:, None]
        near = (cut + rng.choice(np.array([0, 0, 1, 2, 3, 4], dtype=np.float32), size=at.shape) * np.float32(1e-7)).astype(np.float32)
        np.put_along_axis(s, at, near, axis=1)
    w = gen.make_custom(dtype="bf16", n_q=2, n_kv=2, d=64, chunk=40, n_retain=16, kv_lens=[T], budgets=[B], batch=1, seed=3)
    buf = _buffers(w)
    buf.scores.copy_(torch.from_numpy(s)[None])
    buf.k_idx.fill_(-1)
    buf.topk_keys()
    torch.cuda.synchronize()
    want = np.stack([np.sort(np.argsort(-r, kind="stable")[:B]) for r in s])
    assert np.array_equal(gen.from_torch(buf.k_idx)[0][:, :B], want), f"{crowd} keys"


# threads and keys a thread: the sizes on either side of every line; scores that fill one bin with few, up to 256 or more keys
@pytest.mark.parametrize("T,crowd", [
    (T, crowd) for T in (2, 63, 511, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193, 12288, 12289, 16384, 28672, 28673)
    for crowd in (0, 200, 256, 257) if crowd < T])
def test_top_b_threads_keys_and_crowded_bins(T, crowd):
    check_crowded_top_b(T, crowd)


# how many keys of the cut's bin are ranked (`line`; the bin holds a few more than the crowd), one or four at a time, and how many are
# radix-selected
@pytest.mark.parametrize("T,line", [(500, 128), (2048, 128), (2049, 256), (12288, 256), (16384, 320), (20480, 384), (24576, 448),
                                    (28672, 512), (32768, 512)])
def test_top_b_ranked_and_radix_selected_bins(T, line):
    few = 32 if line == 128 else 64
    for crowd in [few - 2, few - 1, few, few + 1, few + 2, few + 3, 2 * few - 1] + [line + i for i in range(-12, 3)]:
        check_crowded_top_b(T, min(crowd, T - 1))
