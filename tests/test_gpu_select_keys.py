"""quoka_select_keys (scoring + top-B as one stage; Alg. 1 S = Qbar K^T, max, topk) against the oracle and against the
two separate calls.  On long bf16 caches the stage scores every key with one bf16 term first and re-scores only the
keys near the cut exactly; its index lists must still be the top-B of the exact scores."""
import numpy as np
import pytest
import torch

import gen
from oracle import quoka_oracle as O
from tests import parity as P

pytestmark = pytest.mark.gpu


def _pk():
    import paper_2602_08722_amd as pk
    pk.load_library()
    return pk


def _buffers(pk, w, t=None):
    t = gen.to_torch(w, "cuda:0") if t is None else t
    mb = min(max(w.budgets), w.t_max)
    return pk.ChunkBuffers(t["q"], t["k"], t["v"], t["kc"], t["vc"], w.kv_lens, w.budgets, w.n_retain, max_budget=mb)


def _staged(buf):
    buf.select_queries()
    buf.scores.fill_(float("nan"))
    buf.k_idx.fill_(-1)
    buf.score_keys()
    buf.topk_keys()
    torch.cuda.synchronize()
    return buf.scores.clone(), buf.k_idx.clone(), buf.k_cnt.clone()


def _fused(buf, dirty=0x5A):
    buf.select_queries()
    buf.scores.fill_(float("nan"))
    buf.k_idx.fill_(-1)
    buf.k_cnt.fill_(-1)
    buf.workspace.fill_(dirty)       # the stage clears what it needs itself
    buf.select_queries()             # (its workspace region was just overwritten; Q-bar is an input of the stage)
    buf.select_keys()
    torch.cuda.synchronize()
    return buf.scores.clone(), buf.k_idx.clone(), buf.k_cnt.clone()


def _compare(pk, w, t=None, oracle=True):
    buf = _buffers(pk, w, t)
    sc_s, idx_s, cnt_s = _staged(buf)
    sc_f, idx_f, cnt_f = _fused(buf)
    assert torch.equal(cnt_f, cnt_s)
    qbar = gen.from_torch(buf.qbar)
    q_idx = gen.from_torch(buf.q_idx)
    n_exact = n_all = 0
    for b in range(w.batch):
        T, n = w.kv_lens[b], int(cnt_s[b, 0])
        assert n == min(w.budgets[b], T, buf.shape.max_budget)
        # the same index lists, bit for bit, as the two separate calls
        assert torch.equal(idx_f[b, :, :n], idx_s[b, :, :n]), f"sequence {b}: index lists differ from the staged calls"
        if T == 0:
            continue
        got, exact = sc_f[b, :, :T], sc_s[b, :, :T]
        assert not torch.isnan(got).any()
        same = got.view(torch.int32) == exact.view(torch.int32)
        n_exact += int(same.sum())
        n_all += same.numel()
        if oracle:
            want = O.key_scores(w.Q[b], q_idx[b], w.K[b][:, :T], w.n_kv)
            for kv in range(w.n_kv):
                if P.two_pass_scores(w):
                    P.check_two_pass_scores(got[kv].cpu().numpy(), want[kv], qbar[b, kv], w.budgets[b],
                                            what=f"b{b} kv{kv}")
                else:
                    assert P.max_abs(got[kv].cpu().numpy(), want[kv]) <= P.TOL_SCORE
                P.check_topk_set(idx_f[b, kv, :n].cpu().numpy(), want[kv], w.budgets[b], what=f"b{b} kv{kv}")
    return n_exact, n_all


CASES = [
    # just past the single-block limit; budgets on both sides of the tile size; N_Q variants 4 / 2 / 1 query blocks
    dict(n_q=8, n_kv=2, d=128, chunk=256, n_retain=128, kv_lens=[33000], budgets=[4000]),
    dict(n_q=8, n_kv=2, d=128, chunk=256, n_retain=64, kv_lens=[40000], budgets=[1]),
    dict(n_q=4, n_kv=2, d=128, chunk=64, n_retain=20, kv_lens=[36111], budgets=[36110]),
    dict(n_q=4, n_kv=4, d=64, chunk=96, n_retain=40, kv_lens=[50001], budgets=[7777]),
    dict(n_q=4, n_kv=1, d=64, chunk=200, n_retain=128, kv_lens=[34000], budgets=[3000]),
    # ragged batch: an empty cache, one shorter than a tile, a full-budget one and a budget beyond the cache
    dict(n_q=8, n_kv=2, d=128, chunk=128, n_retain=32, kv_lens=[45000, 0, 1500, 33333, 70000],
         budgets=[5000, 10, 150, 33333, 99999], batch=5),
    # one head per group (Q-bar rows are single unit queries), decode-sized chunk (identity selection)
    dict(n_q=2, n_kv=2, d=128, chunk=4, n_retain=16, kv_lens=[65537], budgets=[8000]),
    # short caches go through the stage too (it is then the two separate launches)
    dict(n_q=8, n_kv=2, d=128, chunk=100, n_retain=16, kv_lens=[3000, 32768], budgets=[300, 4000], batch=2),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()))
def test_select_keys_matches_the_oracle_and_the_staged_calls(case):
    pk = _pk()
    case = dict(case)
    batch = case.pop("batch", 1)
    w = gen.make_custom(dtype="bf16", batch=batch, seed=31, **case)
    n_exact, n_all = _compare(pk, w)
    if P.two_pass_scores(w):
        assert n_exact < 0.7 * n_all, (n_exact, n_all)   # the cheaper pass really ran: most keys keep their provisional score
    else:
        assert n_exact == n_all                          # short caches: the stage is the two separate launches


def test_select_keys_with_planted_exact_ties_and_repeated_keys():
    """Equal exact scores go to the lower position, also when they straddle the cut and sit in different tiles: rows
    of the cache are repeated (identical keys score identically in both passes) so that the cut falls inside a group
    of equal scores."""
    pk = _pk()
    w = gen.make_custom(dtype="bf16", n_q=8, n_kv=2, d=128, chunk=128, n_retain=64, kv_lens=[40000], budgets=[500],
                        seed=32)
    # find a key that ranks near the budget, then copy it to many positions spread over the cache
    q_idx = O.select_queries(w.Q[0], w.n_retain)
    sc = O.key_scores(w.Q[0], q_idx, w.K[0], w.n_kv)
    for kv in range(w.n_kv):
        order = np.argsort(-sc[kv], kind="stable")
        src = order[480]
        dst = np.arange(17, 40000, 1301)       # 31 copies: more than the 20 places left below rank 480
        w.K[0, kv, dst] = w.K[0, kv, src]
    _compare(pk, w)


def test_select_keys_when_every_key_is_a_candidate():
    """A cache of identical keys: every score ties, the band is the whole cache, and the first B positions win."""
    pk = _pk()
    w = gen.make_custom(dtype="bf16", n_q=4, n_kv=2, d=128, chunk=64, n_retain=32, kv_lens=[33500], budgets=[1000],
                        seed=33)
    w.K[0, :, :] = w.K[0, :, :1]
    buf = _buffers(pk, w)
    _, idx_f, cnt_f = _fused(buf)
    assert cnt_f.tolist() == [[1000, 1000]]
    assert torch.equal(idx_f[0, :, :1000].cpu(), torch.arange(1000, dtype=torch.int32).expand(2, 1000))
    _compare(pk, w, oracle=False)


@pytest.mark.parametrize("name,kw", [("c4", {}), ("c5", dict(n_retain=128, budget_frac=0.12))])
def test_select_keys_full_size(name, kw):
    pk = _pk()
    w = gen.make_workload(name, **kw)
    n_exact, n_all = _compare(pk, w, oracle=(name == "c4"))
    assert n_exact < 0.5 * n_all


def test_select_keys_token_major_cache():
    """Strided (token-major) caches give the same lists as their head-major copies."""
    pk = _pk()
    w = gen.make_custom(dtype="bf16", n_q=8, n_kv=4, d=128, chunk=64, n_retain=32, kv_lens=[40000], budgets=[3000],
                        seed=34)
    t = gen.to_torch(w, "cuda:0")
    tm = dict(t)
    for k in ("k", "v"):
        tm[k] = t[k].permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    a, b = _buffers(pk, w, t), _buffers(pk, w, tm)
    ra, rb = _fused(a), _fused(b)
    for x, y in zip(ra, rb):
        assert torch.equal(x.view(torch.int32), y.view(torch.int32))


# up to eight retained queries: all three terms in one operand, exact scores from the streaming launch, the cut found by the
# emitting blocks (edges of the tiles, of the list of candidates held in LDS, and of the rule's sizes)
PACKED = [
    ("normal", dict(n_q=32, n_kv=8, d=128, chunk=1, n_retain=16, kv_lens=[32769], budgets=[3000])),
    ("normal", dict(n_q=12, n_kv=4, d=64, chunk=8, n_retain=8, kv_lens=[65537, 0, 1500, 2048, 40000],
                    budgets=[7000, 4, 1500, 2047, 1], batch=5)),
    ("normal", dict(n_q=2, n_kv=2, d=128, chunk=40, n_retain=7, kv_lens=[131072], budgets=[131071])),
    ("pairs", dict(n_q=8, n_kv=2, d=128, chunk=3, n_retain=64, kv_lens=[110001], budgets=[9001])),
    ("equal", dict(n_q=8, n_kv=2, d=64, chunk=2, n_retain=64, kv_lens=[100000], budgets=[50001])),
    ("half", dict(n_q=4, n_kv=2, d=128, chunk=1, n_retain=1, kv_lens=[100003], budgets=[60001])),
]


@pytest.mark.parametrize("kind,case", PACKED, ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()) if isinstance(c, dict) else c)
def test_few_queries_select_exactly_from_one_pass(kind, case):
    pk = _pk()
    case = dict(case)
    w = gen.make_custom(dtype="bf16", seed=41, **dict(dict(batch=1), **case))
    if kind == "equal":
        w.K[:] = w.K[:, :, :1]
    elif kind == "half":      # more equal candidates at the cut than the emitting blocks hold
        w.K[:, :, 30000:70000] = w.K[:, :, 30000:30001]
    elif kind == "pairs":
        n = w.K.shape[2] // 2 * 2
        w.K[:, :, 1:n:2] = w.K[:, :, 0:n:2]
    n_exact, n_all = _compare(pk, w, oracle=kind == "normal")
    assert n_exact == n_all
    buf = _buffers(pk, w)
    buf.select_queries()
    torch.cuda.synchronize()
    qbar, q_idx = buf.qbar.clone(), buf.q_idx.clone()
    for b in (buf.qbar, buf.q_idx, buf.k_idx):
        b.fill_(-1)
    buf.chunk_attn()
    torch.cuda.synchronize()
    assert torch.equal(buf.qbar, qbar) and torch.equal(buf.q_idx, q_idx)
    for b in range(w.batch):
        n = int(buf.k_cnt[b, 0])
        want = O.topk_keys(buf.scores[b, :, :w.kv_lens[b]].cpu().numpy(), w.budgets[b])
        assert np.array_equal(buf.k_idx[b, :, :n].cpu().numpy(), want)


@pytest.mark.parametrize("case", [
    dict(n_q=4, n_kv=2, d=128, chunk=1, n_retain=16, kv_lens=[1000, 0, 129], budgets=[100, 5, 128], batch=3),
    dict(n_q=16, n_kv=1, d=64, chunk=8, n_retain=8, kv_lens=[32768], budgets=[5000]),
    dict(n_q=6, n_kv=2, d=64, chunk=5, n_retain=32, kv_lens=[1], budgets=[1]),
], ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()))
def test_scoring_launch_forms_the_queries_of_a_few_tokens(case):
    """chunk_attn leaves the query stage to the scoring launch here: the same bits as the separate calls."""
    pk = _pk()
    w = gen.make_custom(dtype="bf16", seed=43, **dict(dict(batch=1), **case))
    buf = _buffers(pk, w)
    sc, idx, cnt = _staged(buf)
    qbar, q_idx = buf.qbar.clone(), buf.q_idx.clone()
    for b in (buf.qbar, buf.q_idx, buf.k_idx, buf.k_cnt):
        b.fill_(-1)
    buf.scores.fill_(float("nan"))
    buf.chunk_attn()
    torch.cuda.synchronize()
    assert torch.equal(buf.qbar, qbar) and torch.equal(buf.q_idx, q_idx) and torch.equal(buf.k_cnt, cnt)
    for b in range(w.batch):
        T, n = w.kv_lens[b], int(cnt[b, 0])
        assert torch.equal(buf.scores[b, :, :T], sc[b, :, :T]) and torch.equal(buf.k_idx[b, :, :n], idx[b, :, :n])


@pytest.mark.parametrize("crowd", [0, 40, 64, 300, 900, 1100, 3000])
@pytest.mark.parametrize("n_q,chunk", [(4, 2), (4, 60)], ids=["one-pass", "two-pass"])
def test_select_keys_with_many_candidates_near_the_cut(n_q, chunk, crowd):
    """`crowd` keys differ from the one at the cut by a few bf16 steps of some elements, so that they share its bin, or its part of
    a bin: more or fewer than a block holds in registers or ranks one by one.  The list is that of the scores themselves."""
    pk = _pk()
    T, B = 100000, 9000
    w = gen.make_custom(dtype="bf16", n_q=n_q, n_kv=2, d=128, chunk=chunk, n_retain=32, kv_lens=[T], budgets=[B], seed=47)
    rng = np.random.default_rng(6)
    sc = O.key_scores(w.Q[0], O.select_queries(w.Q[0], w.n_retain), w.K[0], w.n_kv)
    for kv in range(w.n_kv):
        src = np.argsort(-sc[kv], kind="stable")[B - crowd // 3]
        dst = rng.choice(T, size=crowd, replace=False)
        rows = np.repeat(w.K[0, kv, src:src + 1], crowd, axis=0)
        rows *= 1.0 + (rng.integers(-1, 2, size=rows.shape) * (rng.random(rows.shape) < 0.05)) * 2.0 ** -7
        w.K[0, kv, dst] = rows
    t = gen.to_torch(w, "cuda:0")     # (rounds the rows to bf16)
    buf = _buffers(pk, w, t)
    _, idx_s, cnt_s = _staged(buf)
    exact = gen.from_torch(buf.scores)[0]
    _, idx_f, cnt_f = _fused(buf)
    assert torch.equal(cnt_f, cnt_s) and torch.equal(idx_f, idx_s)
    assert np.array_equal(gen.from_torch(idx_f)[0], O.topk_keys(exact, B))


# chunk_attn, in sizes where it scores every key exactly and selects from the histogram of the exact scores
@pytest.mark.parametrize("kind", ["normal", "pairs", "equal"])
@pytest.mark.parametrize("case", [
    dict(n_q=4, n_kv=1, d=128, chunk=40, n_retain=9, kv_lens=[32769], budgets=[1]),                  # one query block; a tile of one key
    dict(n_q=4, n_kv=2, d=64, chunk=70, n_retain=64, kv_lens=[40960], budgets=[40959]),              # two; full tiles; all but one
    dict(n_q=4, n_kv=2, d=128, chunk=200, n_retain=100, kv_lens=[131072], budgets=[9000]),           # four; the longest cache
    dict(n_q=2, n_kv=2, d=128, chunk=3, n_retain=16, kv_lens=[65537], budgets=[8000]),               # all queries kept, few positions
    dict(n_q=8, n_kv=2, d=128, chunk=128, n_retain=32, kv_lens=[45000, 0, 1500, 33333, 70000], budgets=[5000, 10, 150, 33333, 99999],
         batch=5),
], ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()))
def test_chunk_attn_selects_from_exact_scores(kind, case):
    pk = _pk()
    w = gen.make_custom(dtype="bf16", seed=44, **dict(dict(batch=1), **case))
    if kind == "equal":
        w.K[:] = w.K[:, :, :1]
    elif kind == "pairs":
        n = w.K.shape[2] // 2 * 2
        w.K[:, :, 1:n:2] = w.K[:, :, 0:n:2]
    buf = _buffers(pk, w)
    sc, idx, cnt = _staged(buf)
    buf.scores.fill_(float("nan"))
    buf.k_idx.fill_(-1)
    buf.k_cnt.fill_(-1)
    buf.workspace.fill_(0x5A)
    buf.chunk_attn()
    torch.cuda.synchronize()
    assert torch.equal(buf.k_cnt, cnt)
    for b in range(w.batch):
        T, n = w.kv_lens[b], int(cnt[b, 0])
        assert torch.equal(buf.scores[b, :, :T], sc[b, :, :T]) and torch.equal(buf.k_idx[b, :, :n], idx[b, :, :n])


# The exact route's scoring blocks share out what the caches hold: caches with room to spare, with nothing, one key, and tiles of 128
# just short of, at and past full; batches with one long sequence, with empty ones, and with more than a wave has lanes
@pytest.mark.parametrize("n_kv,d,T_max,lens", [
    (2, 128, 70000, [0]), (2, 128, 70000, [1]), (2, 64, 70000, [127]), (2, 128, 70000, [128]), (1, 64, 131072, [129]),
    (8, 128, 40000, [8000]), (2, 128, 70000, [69999]),
    (2, 64, 70000, [70000, 0, 1, 128, 129, 5000]), (1, 128, 50000, [0, 0, 50000]), (2, 64, 33000, [0, 0, 0]),
    (4, 64, 33000, [3, 33000, 0, 77, 20000]),
    (1, 64, 33000, [33000 - 517 * i for i in range(64)]), (1, 64, 32800, [32800 - 499 * i for i in range(65)]),
], ids=lambda v: f"{len(v)}x{v[0]}" if isinstance(v, list) else str(v))
def test_chunk_attn_of_caches_with_room_to_spare(n_kv, d, T_max, lens):
    pk = _pk()
    b, C = len(lens), 40
    g = torch.Generator(device="cuda").manual_seed(50)
    q, k, v, kc, vc = (torch.randn(b, n, t, d, device="cuda", generator=g, dtype=torch.float32).bfloat16()
                       for n, t in ((2 * n_kv, C), (n_kv, T_max), (n_kv, T_max), (n_kv, C), (n_kv, C)))
    buf = pk.ChunkBuffers(q, k, v, kc, vc, lens, [t // 9 + 1 for t in lens], 16, max_budget=T_max // 8)
    sc, idx, cnt = _staged(buf)
    buf.scores.fill_(float("nan"))
    buf.k_idx.fill_(-1)
    buf.k_cnt.fill_(-1)
    buf.workspace.fill_(0x5A)
    buf.chunk_attn()
    torch.cuda.synchronize()
    assert torch.equal(buf.k_cnt, cnt)
    for i, T in enumerate(lens):
        n = int(cnt[i, 0])
        assert n == min(T // 9 + 1, T)
        assert torch.equal(buf.scores[i, :, :T], sc[i, :, :T]) and torch.equal(buf.k_idx[i, :, :n], idx[i, :, :n])


# Beyond 250 MB of keys (up to 32 queries: 300 MB) the streaming launch scores exactly (up to 64 queries): the scores and lists of the two separate calls bit for bit;
# one query block and two, not full and full; steps of 256 keys just short of, at and past full, empty sequences, more than a wave has lanes
@pytest.mark.parametrize("kind", ["normal", "pairs", "equal"])
@pytest.mark.parametrize("n_kv,d,T_max,lens,n_retain", [
    (4, 128, 33000, [33000, 0, 1, 255, 256, 257, 5000, 32768], 9),
    (4, 128, 33000, [2, 511, 513, 0, 33000, 33000, 777, 12345], 64),
    (8, 64, 33000, [33000, 0, 1, 255, 256, 257, 5000, 32768], 33),
    (1, 128, 131072, [131072, 100001, 3, 65536, 0, 131071, 5, 90000], 32),
    (1, 64, 32800, [32800 - 499 * (i % 65) for i in range(66)], 40),
    (4, 128, 40000, [40000, 0, 1, 255, 256, 257, 5000, 32768], 9),
    (1, 128, 131072, [131072, 100001, 3, 65536, 0, 131071, 5, 90000, 777], 32),
], ids=lambda v: f"{len(v)}x{v[0]}" if isinstance(v, list) else str(v))
def test_chunk_attn_streams_exact_scores(kind, n_kv, d, T_max, lens, n_retain):
    pk = _pk()
    b, C = len(lens), 70
    assert b * n_kv * T_max * d * 2 > 250_000_000
    g = torch.Generator(device="cuda").manual_seed(53)
    q, k, v, kc, vc = (torch.randn(b, n, t, d, device="cuda", generator=g, dtype=torch.float32).bfloat16()
                       for n, t in ((2 * n_kv, C), (n_kv, T_max), (n_kv, T_max), (n_kv, C), (n_kv, C)))
    if kind == "equal":
        k[:] = k[:, :, :1].clone()
    elif kind == "pairs":
        n = T_max // 2 * 2
        k[:, :, 1:n:2] = k[:, :, 0:n:2]
    buf = pk.ChunkBuffers(q, k, v, kc, vc, lens, [t // 9 + 1 for t in lens], n_retain, max_budget=T_max // 8)
    sc, idx, cnt = _staged(buf)
    buf.scores.fill_(float("nan"))
    buf.k_idx.fill_(-1)
    buf.k_cnt.fill_(-1)
    buf.workspace.fill_(0x5A)
    buf.chunk_attn()
    torch.cuda.synchronize()
    assert torch.equal(buf.k_cnt, cnt)
    for i, T in enumerate(lens):
        n = int(cnt[i, 0])
        assert torch.equal(buf.scores[i, :, :T], sc[i, :, :T]) and torch.equal(buf.k_idx[i, :, :n], idx[i, :, :n])


# More candidates than a block holds in registers, listed in memory and fetched in runs of 2048 (8192 where one block selects for a
# head): lists just short of, at and past whole runs; all scores equal, or eight values of which the cut's is an eighth
@pytest.mark.parametrize("values", [1, 8])
@pytest.mark.parametrize("call,chunk", [("chunk_attn", 40), ("chunk_attn", 2), ("select_keys", 40)], ids=["exact", "one-pass", "two-pass"])
def test_candidates_listed_in_memory(call, chunk, values):
    pk = _pk()
    lens = [1025, 2047, 2048, 2049, 4096 * 8 + 1, 8191, 8192, 8193] if values == 1 else [33000, 16384, 16392, 8200, 40, 20000, 30000, 24576]
    g = torch.Generator(device="cuda").manual_seed(51)
    q, k, v, kc, vc = (torch.randn(8, n, t, 64, device="cuda", generator=g).bfloat16()
                       for n, t in ((2, chunk), (1, 33000), (1, 33000), (1, chunk), (1, chunk)))
    k = k[:, :, torch.randint(0, values, (33000,), device="cuda", generator=g)].contiguous()
    buf = pk.ChunkBuffers(q, k, v, kc, vc, lens, [t // 2 + 1 for t in lens], 16)
    sc, idx, cnt = _staged(buf)
    buf.select_queries()
    buf.k_idx.fill_(-1)
    buf.k_cnt.fill_(-1)
    getattr(buf, call)()
    torch.cuda.synchronize()
    assert torch.equal(buf.k_cnt, cnt)
    for i, T in enumerate(lens):
        n = int(cnt[i, 0])
        want = O.topk_keys(gen.from_torch(sc)[i][:, :T], n)
        assert np.array_equal(gen.from_torch(idx)[i][:, :n], want) and np.array_equal(gen.from_torch(buf.k_idx)[i][:, :n], want)


@pytest.mark.parametrize("left_out", [30000, 45, 3])
@pytest.mark.parametrize("case", [dict(n_q=4, n_kv=1, chunk=40, n_retain=32), dict(n_q=8, n_kv=8, chunk=2, n_retain=16)], ids=["exact", "one-pass"])
def test_keys_whose_scores_overflow(case, left_out):
    """Keys so long that their squared norm is infinite (their score is then zero), and so long that the product is too (not a
    number: below every other score, on every route of long caches).  The cut lies among ordinary scores, or among those without
    a number, of which the lower positions are taken."""
    pk = _pk()
    T = 40000
    w = gen.make_custom(dtype="bf16", d=128, kv_lens=[T], budgets=[T - left_out], batch=1, seed=52, **case)
    buf = _buffers(pk, w)
    buf.select_queries()
    qbar = gen.from_torch(buf.qbar)[0]
    rng = np.random.default_rng(9)
    for kv in range(w.n_kv):
        at = rng.choice(T, size=40, replace=False)
        w.K[0, kv, at[:20]] *= 2.0 ** 90
        w.K[0, kv, at[20:]] = np.where(qbar[kv, 0] > 0, 1.0, -1.0) * 255 / 256 * 2.0 ** 128   # (product with row 0: its 1-norm times that)
        assert np.abs(qbar[kv, 0]).sum() > 1.1
    buf = _buffers(pk, w)
    exact = gen.from_torch(_staged(buf)[0])[0]
    lists = []
    for call in (buf.chunk_attn, buf.select_keys):
        buf.k_idx.fill_(-1)
        call()
        torch.cuda.synchronize()
        lists.append(gen.from_torch(buf.k_idx)[0])
    assert np.array_equal(*lists)
    nan = np.isnan(exact)
    assert (nan.sum(axis=1) == 20).all()
    assert np.array_equal(lists[0], O.topk_keys(np.where(nan, np.float32(-2.0), exact), T - left_out))
