"""GPU parity of the multi-chunk prefill driver (Alg. 2's loop) against the oracle."""
import numpy as np
import pytest
import torch

import gen
from oracle import quoka_oracle as O
from tests import parity as P

pytestmark = pytest.mark.gpu


def _prompt(seed, n_q, n_kv, d, L):
    """A whole prompt as one 'chunk' of the seeded generator: Q [1, n_q, L, d], K / V [1, n_kv, L, d] (bf16-exact)."""
    w = gen.make_custom(dtype="bf16", n_q=n_q, n_kv=n_kv, d=d, chunk=L, n_retain=1, kv_lens=[0], budgets=[0],
                        batch=1, seed=seed)
    return w.Q[0], w.Kc[0], w.Vc[0]


def _full_causal(Q, K, V):
    """Plain causal attention over the whole prompt in float64: the definition dense chunked prefill must reach."""
    n_q, L, d = Q.shape
    g = n_q // K.shape[0]
    out = np.empty((n_q, L, d))
    mask = np.tril(np.ones((L, L), dtype=bool))
    for h in range(n_q):
        s = (Q[h].astype(np.float64) @ K[h // g].astype(np.float64).T) / np.sqrt(d)
        s = np.where(mask, s, -np.inf)
        p = np.exp(s - s.max(axis=1, keepdims=True))
        out[h] = (p / p.sum(axis=1, keepdims=True)) @ V[h // g].astype(np.float64)
    return out


def _to_dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to(torch.bfloat16).to("cuda:0")[None]


@pytest.mark.parametrize("L,chunk", [(640, 128), (700, 192), (96, 128), (130, 128), (1027, 256)])  # the last two end in a decode-sized chunk
def test_dense_chunked_prefill_is_full_causal_attention(L, chunk):
    import paper_2602_08722_amd as pk
    pk.load_library()
    Q, K, V = _prompt(31, 8, 2, 128, L)
    pb = pk.PrefillBuffers(_to_dev(Q), _to_dev(K), _to_dev(V), chunk, n_retain=16, budget=0)
    out = pb.run(sparse=False)
    torch.cuda.synchronize()
    got = out[0].float().cpu().numpy()
    assert P.max_abs(got, _full_causal(Q, K, V)) <= P.TOL_OUT["bf16"]


@pytest.mark.parametrize("L,chunk,n_retain,budget", [(768, 128, 16, 96), (700, 192, 32, 64), (1027, 256, 16, 200)])
def test_sparse_chunked_prefill_matches_oracle(L, chunk, n_retain, budget):
    import paper_2602_08722_amd as pk
    pk.load_library()
    Q, K, V = _prompt(32, 8, 2, 128, L)
    pb = pk.PrefillBuffers(_to_dev(Q), _to_dev(K), _to_dev(V), chunk, n_retain=n_retain, budget=budget)
    out = pb.run(sparse=True)
    torch.cuda.synchronize()
    got = out[0].float().cpu().numpy()
    want = O.chunked_prefill(Q, K, V, chunk, n_retain=n_retain, budget=budget)
    assert P.max_abs(got, want) <= P.TOL_OUT["bf16"]
    # the scratch buffers hold the last chunk's selection: it must be the oracle's for that chunk
    s = (L - 1) // chunk * chunk
    _, _, k_idx = O.quoka_select(Q[:, s:], K[:, :s], n_retain, budget)
    cnt = pb.k_cnt[0].cpu().numpy()
    got_idx = pb.k_idx[0].cpu().numpy()
    scores = O.key_scores(Q[:, s:], O.select_queries(Q[:, s:], n_retain), K[:, :s], K.shape[0])
    for kv in range(K.shape[0]):
        assert cnt[kv] == min(budget, s)
        P.check_topk_set(got_idx[kv, :cnt[kv]], scores[kv], min(budget, s), what=f"last chunk kv{kv}")


@pytest.mark.parametrize("dtype,batch,n_q,n_kv,d,L,chunk,n_retain,sparse", [
    ("bf16", 1, 8, 2, 128, 700, 192, 32, True),      # a short last chunk goes along
    ("bf16", 1, 8, 2, 128, 1027, 256, 16, True),     # a decode-sized one does not
    ("bf16", 1, 6, 2, 64, 2600, 200, 48, True),      # every chunk full length, three heads a group
    ("bf16", 2, 8, 2, 128, 2111, 128, 16, True),     # two sequences, 17 chunks each
    ("bf16", 1, 32, 8, 128, 9000, 100, 64, True),    # 90 chunks: two groups
    ("bf16", 1, 4, 1, 64, 36000, 2048, 32, True),    # the two-pass selection, no key splits
    ("bf16", 1, 8, 2, 64, 800, 4, 16, True),         # decode-sized chunks
    ("bf16", 1, 8, 2, 128, 1500, 256, 16, False),
    ("f32", 1, 4, 2, 64, 900, 128, 16, True),        # float32: the short last chunk runs by itself
    ("f32", 2, 4, 2, 128, 1024, 128, 16, True),
    ("bf16", 1, 4, 2, 64, 60000, 1024, 8, True),     # few queries, few keys in all: no packed scoring in any group
    ("bf16", 1, 8, 8, 64, 36000, 600, 8, True),      # few queries, packed scoring in chunks of every length
])
def test_chunks_that_share_launches_match_chunk_after_chunk(dtype, batch, n_q, n_kv, d, L, chunk, n_retain, sparse):
    """The same prompt with the workspace of one chunk (chunk after chunk) and with the full one (chunks as a batch)."""
    import paper_2602_08722_amd as pk
    pk.load_library()
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    rng = torch.Generator(device="cuda").manual_seed(5)
    q, k, v = (torch.randn(batch, n, L, d, device="cuda", generator=rng).to(dt) for n in (n_q, n_kv, n_kv))
    def run(full):
        pb = pk.PrefillBuffers(q, k, v, chunk, n_retain, lambda t: t // 8)
        if not full:
            small = pk.quoka_workspace_bytes(pb.shape)
            assert small < pb.workspace.numel()
            pb.workspace = pb.workspace[:small]
        for t in (pb.k_idx, pb.q_idx, pb.k_cnt):
            t.fill_(-1)
        pb.run(sparse=sparse)
        torch.cuda.synchronize()
        return pb
    one, many = run(False), run(True)
    # two roundings of the output to dt, and of the probabilities (bf16) on either side
    tol = P.TOL_OUT["bf16"] if dtype == "bf16" else 2e-5
    assert (one.out.float() - many.out.float()).abs().max().item() <= tol
    if sparse:   # the last chunk's intermediates are the caller's either way
        n_keep = min(n_retain, L - (L - 1) // chunk * chunk, chunk)
        if n_keep == min(n_retain, chunk):
            assert torch.equal(one.q_idx, many.q_idx)
        assert torch.equal(one.k_cnt, many.k_cnt) and int(one.k_cnt.min()) > 0
        cnt = int(one.k_cnt[0, 0])
        assert torch.equal(one.k_idx[:, :, :cnt], many.k_idx[:, :, :cnt])
        t = (L - 1) // chunk * chunk
        assert torch.equal(one.scores[:, :, :t], many.scores[:, :, :t])
        assert (one.qbar - many.qbar).abs().max().item() <= 1e-6 or n_keep < min(n_retain, chunk)


def _prompt_on_device(batch, n_q, n_kv, d, L, q_scale=1.0, seed=5):
    rng = torch.Generator(device="cuda").manual_seed(seed)
    q, k, v = (torch.randn(batch, n, L, d, device="cuda", generator=rng) for n in (n_q, n_kv, n_kv))
    return (q * q_scale).bfloat16(), k.bfloat16(), v.bfloat16()


@pytest.mark.parametrize("n_q,n_kv,d,L,chunk,n_retain,sparse", [
    (2, 2, 64, 212, 64, 16, True),       # one head a group, last chunk of 20 tokens
    (8, 2, 128, 1029, 256, 4, True),     # four heads a group, last chunk of 5
    (8, 2, 128, 1029, 256, 4, False),
])
def test_decode_sized_last_chunk_is_scaled_in_float32(n_q, n_kv, d, L, chunk, n_retain, sparse):
    """A last chunk that retains as many queries as the others but fits the decode kernel takes that kernel, which leaves Q
    alone: logits of eight times unit variance, at the usual bar (the kernel for larger chunks is off by 0.06 there)."""
    import paper_2602_08722_amd as pk
    pk.load_library()
    q, k, v = _prompt_on_device(1, n_q, n_kv, d, L, q_scale=8.0)
    outs = []
    for full in (False, True):
        pb = pk.PrefillBuffers(q, k, v, chunk, n_retain, lambda t: t // 8)
        if not full:
            pb.workspace = pb.workspace[:pk.quoka_workspace_bytes(pb.shape)]
        pb.run(sparse=sparse)
        torch.cuda.synchronize()
        outs.append(pb.out)
    tail = (L - 1) // chunk * chunk
    assert torch.equal(outs[0][:, :, tail:], outs[1][:, :, tail:])   # the same launches
    if not sparse:
        want = _full_causal(gen.from_torch(q)[0], gen.from_torch(k)[0], gen.from_torch(v)[0])[:, tail:]
        assert P.max_abs(gen.from_torch(outs[1])[0][:, tail:], want) <= P.TOL_OUT["bf16"]


@pytest.mark.parametrize("n_retain", [15, 16, 17])
def test_last_chunk_of_as_many_tokens_as_are_retained(n_retain):
    """Up to n_retain tokens all are kept, in position order (16 tokens of four heads a group: not decode-sized)."""
    import paper_2602_08722_amd as pk
    pk.load_library()
    q, k, v = _prompt_on_device(1, 8, 2, 64, 3 * 256 + 16)
    got = []
    for full in (False, True):
        pb = pk.PrefillBuffers(q, k, v, 256, n_retain, lambda t: t // 8)
        if not full:
            pb.workspace = pb.workspace[:pk.quoka_workspace_bytes(pb.shape)]
        pb.run()
        torch.cuda.synchronize()
        n = min(n_retain, 16)
        # (where the last chunk retains fewer queries than the others, its arrays are packed by its own number)
        q_idx, qbar = pb.q_idx.flatten()[:8 * n].view(8, n), pb.qbar.flatten()[:2 * n * 64]
        got.append((q_idx, qbar, pb.k_cnt, pb.k_idx[:, :, :int(pb.k_cnt[0, 0])]))
        if n == 16:
            assert torch.equal(q_idx, torch.arange(16, device="cuda", dtype=torch.int32).expand(8, 16))
    for a, b in zip(*got):
        assert torch.equal(a, b)


def test_short_last_chunk_keeps_its_query_route():
    """128 heads, full chunks beyond what one block per head holds, a last chunk within: cosines so close together that the
    last bits of the mean decide ranks."""
    import paper_2602_08722_amd as pk
    pk.load_library()
    L, chunk = 6 * 1024 + 300, 1024
    q, k, v = _prompt_on_device(4, 32, 8, 128, L)
    rng = torch.Generator(device="cuda").manual_seed(6)
    lean = 30.0 * torch.randn(4, 32, 1, 128, device="cuda", generator=rng)
    q = (lean + q.float()).bfloat16()
    got = []
    for full in (False, True):
        pb = pk.PrefillBuffers(q, k, v, chunk, 64, lambda t: t // 8)
        if not full:
            pb.workspace = pb.workspace[:pk.quoka_workspace_bytes(pb.shape)]
        pb.run()
        torch.cuda.synchronize()
        got.append((pb.q_idx, pb.qbar, pb.k_cnt, pb.k_idx[:, :, :int(pb.k_cnt[0, 0])]))
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("chunk,tail", [(1024, 65), (1024, 200), (1024, 256), (1024, 257), (700, 300), (2000, 512), (1024, 513)])
def test_short_last_chunk_selects_alike_in_one_block_and_in_tiles(d, chunk, tail):
    """Few heads, full chunks beyond one block per head: a last chunk of up to 512 tokens takes one block per head by itself and the
    tiled launches among the others.  Cosines so close together that the last bits of the mean decide ranks: the same bits."""
    import paper_2602_08722_amd as pk
    pk.load_library()
    L = 5 * chunk + tail
    q, k, v = _prompt_on_device(1, 8, 2, d, L, seed=tail)
    rng = torch.Generator(device="cuda").manual_seed(6)
    lean = 30.0 * torch.randn(1, 8, 1, d, device="cuda", generator=rng)
    q = (lean + q.float()).bfloat16()
    got = []
    for full in (False, True):
        pb = pk.PrefillBuffers(q, k, v, chunk, 64, lambda t: t // 8)
        if not full:
            pb.workspace = pb.workspace[:pk.quoka_workspace_bytes(pb.shape)]
        pb.q_idx.fill_(-1)
        pb.run()
        torch.cuda.synchronize()
        got.append((pb.q_idx, pb.qbar, pb.k_cnt, pb.k_idx[:, :, :int(pb.k_cnt[0, 0])]))
    for a, b in zip(*got):
        assert torch.equal(a, b)


# (what is compared is what the last chunk leaves; one of up to n_retain = 64 tokens runs by itself, keeps them all and writes no more
# entries than it has, so the rest of the lists is then another chunk's: tails begin at 65)
@pytest.mark.parametrize("d,chunk,tail", [(128, 1024, 1024), (128, 513, 65), (128, 1000, 577), (64, 1024, 1023), (64, 640, 66), (128, 1025, 700)])
def test_queries_of_many_heads_are_selected_as_in_tiles(d, chunk, tail):
    """Chunks that share a launch give it enough heads for one block per head and up to 1024 tokens; one chunk at a time takes the tiled
    launches.  Query rows that lie apart, cosines so close together that the last bits of the mean decide ranks: the same bits."""
    import paper_2602_08722_amd as pk
    pk.load_library()
    n_q, L = 16, 5 * chunk + tail
    _, k, v = _prompt_on_device(1, n_q, 4, d, L, seed=tail)
    rng = torch.Generator(device="cuda").manual_seed(7)
    lean = 30.0 * torch.randn(1, 1, n_q, d, device="cuda", generator=rng)
    q = (lean + torch.randn(1, L, n_q, d, device="cuda", generator=rng)).bfloat16().transpose(1, 2)
    got = []
    for full in (False, True):
        pb = pk.PrefillBuffers(q, k, v, chunk, 64, lambda t: t // 8)
        if not full:
            pb.workspace = pb.workspace[:pk.quoka_workspace_bytes(pb.shape)]
        pb.q_idx.fill_(-1)
        pb.run()
        torch.cuda.synchronize()
        got.append((pb.q_idx, pb.qbar, pb.k_cnt, pb.k_idx[:, :, :int(pb.k_cnt[0, 0])]))
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("dtype,n_q,n_kv,L,chunk,sparse", [
    ("bf16", 4, 1, 300, 8, False),      # decode kernel
    ("bf16", 4, 1, 300, 8, True),
    ("bf16", 4, 2, 900, 64, False),     # key lists split over blocks
    ("f32", 4, 2, 500, 32, False),
])
@pytest.mark.parametrize("full", [False, True], ids=["chunk-after-chunk", "grouped"])
def test_cache_lengths_beyond_the_prompt_position_are_cut(dtype, n_q, n_kv, L, chunk, sparse, full):
    """No chunk sees cache rows that its launch was not sized for (every partial result that is added up has been written:
    the workspace holds NaN).  Chunk after chunk that is the chunk's own position."""
    import paper_2602_08722_amd as pk
    pk.load_library()
    q, k, v = (x if dtype == "bf16" else x.float() for x in _prompt_on_device(1, n_q, n_kv, 64, L))
    outs = []
    for beyond in (False, True):
        pb = pk.PrefillBuffers(q, k, v, chunk, 4, lambda t: t // 4)
        if beyond:
            pb.kv_lens_all.fill_(L)
        if not full:
            pb.workspace = pb.workspace[:pk.quoka_workspace_bytes(pb.shape)]
        pb.workspace.fill_(0xFF)
        pb.run(sparse=sparse)
        torch.cuda.synchronize()
        outs.append(pb.out)
    assert not torch.isnan(outs[1].float()).any()
    if not full:
        assert torch.equal(outs[0], outs[1])
