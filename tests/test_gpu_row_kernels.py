"""Branches of the per-row kernels.

Greedy sampling: rows cut into chunks against whole rows (by vocabulary and
batch), ties across chunk edges to the lowest index, NaN and -inf, rows that do
not start 16-byte aligned; exact against numpy.

V pages: passes of 64 rows and more write V 16 rows at a time (eight slots of a
page with one store where they line up), smaller ones a row at a time.  The same
tokens appended in passes of both kinds leave the same layer-0 pages: K and V
depend there on the token's own row alone, so the values differ by the summation
order of one fp32 product, at most one step of the storage type.
"""

import dataclasses

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _engine(shape, dtype, **kw):
    import paper_2609_36899_amd as P
    from workload import make_weights
    w = P.weights_to_device(make_weights(shape, seed=3, bf16=dtype == P.BF16), dtype)
    per_tok = P.kv_bytes_per_token(shape, dtype, kw.get("kv_fp8"))
    return P.Engine(shape, w, dtype, 64 * 16 * per_tok, max_seqs=4, max_seq_len=512, max_batch=4,
                    max_chunk=160, **kw)


@pytest.mark.parametrize("vocab,offset", [(1024, 0), (32768, 0), (32771, 0), (128256, 0), (128256, 1)])
def test_greedy_chunks(vocab, offset):
    import paper_2609_36899_amd as P
    from workload import TINY
    E = _engine(dataclasses.replace(TINY, n_layers=1, d_model=64, ffn_dim=64, vocab=vocab), P.F32)
    rng = np.random.default_rng(vocab)
    for B in (1, 5, 64, 127, 128):
        z = rng.standard_normal((B, vocab)).astype(np.float32)
        z[0] = np.round(z[0])                      # ties everywhere
        if B > 4:
            z[1] = -np.inf
            z[2, ::2] = np.nan
            z[3] = 1.0                             # all equal
            z[4] = -np.inf
            z[4, vocab - 1] = -3.0
        want = [int(np.argmax(np.where(np.isnan(r), -np.inf, r))) for r in z]
        buf = torch.empty(offset + B * vocab, device="cuda")
        zd = buf[offset:].view(B, vocab)
        zd.copy_(torch.from_numpy(z))
        tok = torch.full((B,), -1, dtype=torch.int32, device="cuda")
        E.sample(zd, tok)
        np.testing.assert_array_equal(tok.cpu().numpy(), want)


@pytest.mark.parametrize("held", [-1, 0, 77777, 128255, 128256, 2 ** 31 - 1, -2 ** 31])
def test_greedy_whatever_the_buffer_held(held):
    """Chunks merge in the output: what it held before, a token of the row or not, must
    not matter, with numbers, ties, -inf, NaN in parts and NaN throughout."""
    import paper_2609_36899_amd as P
    from workload import TINY
    V = 128256
    E = _engine(dataclasses.replace(TINY, n_layers=1, d_model=64, ffn_dim=64, vocab=V), P.F32)
    z = torch.randn((8, V), device="cuda", generator=torch.Generator("cuda").manual_seed(4))
    z[1].round_()
    z[2] = -float("inf")
    z[3] = float("nan")
    z[4] = float("nan")
    z[4, V - 1] = -float("inf")
    z[5, :77777] = float("nan")
    z[6] = 2.0
    z[7, V // 2:] = float("nan")
    want = [int(np.argmax(np.where(np.isnan(r), -np.inf, r))) for r in z.cpu().numpy()]
    want[4] = V - 1  # -inf is a number, NaN is none
    for _ in range(3):
        tok = torch.full((8,), held, dtype=torch.int32, device="cuda")
        E.sample(z, tok)
        np.testing.assert_array_equal(tok.cpu().numpy(), want)


def test_greedy_more_rows_than_a_grid_axis():
    """70000 rows: only the first grid axis takes that many work groups."""
    import paper_2609_36899_amd as P
    from workload import TINY
    E = _engine(dataclasses.replace(TINY, n_layers=1, d_model=64, ffn_dim=64, vocab=64), P.F32)
    z = torch.randn((70000, 64), device="cuda", generator=torch.Generator("cuda").manual_seed(2))
    tok = torch.full((70000,), -1, dtype=torch.int32, device="cuda")
    E.sample(z, tok)
    assert torch.equal(tok.long(), z.argmax(dim=1))


@pytest.mark.parametrize("vocab,B", [(128256, 48), (65536, 3)])
def test_greedy_calls_may_overlap(vocab, B):
    """24 outstanding calls over two streams that wait for nothing, eight of them
    replays of one captured call: each gives its own rows' tokens."""
    from workload import TINY
    import paper_2609_36899_amd as P
    E = _engine(dataclasses.replace(TINY, n_layers=1, d_model=64, ffn_dim=64, vocab=vocab), P.F32)
    n = 24
    z = torch.randn((n, B, vocab), device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    tok = torch.full((n, B), -1, dtype=torch.int32, device="cuda")
    replayed = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    sides = [torch.cuda.Stream(), torch.cuda.Stream()]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        E.set_stream(torch.cuda.current_stream())
        E.sample(z[0], replayed)
    torch.cuda.synchronize()
    seen = []
    for i in range(n):
        E.set_stream(sides[i % 2])
        E.sample(z[i], tok[i])
        if i % 3 == 0:  # in order among themselves, beside the calls of the other stream
            with torch.cuda.stream(sides[0]):
                replayed.fill_(-1)
                graph.replay()
                seen.append(replayed.clone())
    torch.cuda.synchronize()
    E.set_stream(torch.cuda.current_stream())
    want = z.argmax(dim=2)
    assert torch.equal(tok.long(), want)
    assert all(torch.equal(s.long(), want[0]) for s in seen)


@pytest.mark.parametrize("kind", ["f32", "bf16", "fp8"])
@pytest.mark.parametrize("before", [0, 5, 8, 16, 27])
def test_v_rows_match_single_rows(kind, before):
    import paper_2609_36899_amd as P
    from workload import SMALL_BF16, TINY, random_tokens
    shape, dtype = (TINY, P.F32) if kind == "f32" else (SMALL_BF16, P.BF16)
    toks = random_tokens(before + 139, shape.vocab, 5)
    pages = []
    for chunk in (160, 16):  # one pass of 139 rows; passes of at most 16
        E = _engine(shape, dtype, kv_fp8=(0.02, 0.03) if kind == "fp8" else None)
        s = E.kv_alloc(0)
        if before:
            E.kv_append_prefix(s, toks[:before], chunk_tokens=16)
        E.kv_append_prefix(s, toks[before:], chunk_tokens=chunk)
        at = torch.arange(len(toks), device="cuda")
        pg = torch.from_numpy(E.kv_block_table(s)).cuda().long()[at // 16]
        view = lambda t: (t.view(torch.float8_e4m3fn) if kind == "fp8" else t).float()
        pages.append((view(E.k_pages(0))[pg, :, at % 16], view(E.v_pages(0))[pg, :, :, at % 16]))
    step = {"f32": 2.0 ** -20, "bf16": 2.0 ** -7, "fp8": 2.0 ** -3}[kind]
    for a, b in zip(*pages):
        floor = 2.0 ** -9 if kind == "fp8" else 1e-6  # the smallest code
        assert torch.all((a - b).abs() <= step * torch.maximum(a.abs(), b.abs()) + floor)
        assert (a != b).float().mean() < (1.0 if kind == "f32" else 0.01)
        assert a.abs().max() > 0


@pytest.mark.parametrize("kind", ["f32", "bf16", "fp8"])
def test_v_of_a_large_decode_batch(kind):
    """72 trajectories decoded in one step and in three leave the same layer-0 pages."""
    import paper_2609_36899_amd as P
    from workload import SMALL_BF16, TINY, make_weights, random_tokens
    shape, dtype = (TINY, P.F32) if kind == "f32" else (SMALL_BF16, P.BF16)
    fp8 = (0.02, 0.03) if kind == "fp8" else None
    w = P.weights_to_device(make_weights(shape, seed=3, bf16=kind != "f32"), dtype)
    n, pages = 72, []
    last = torch.tensor(random_tokens(n, shape.vocab, 9), dtype=torch.int32, device="cuda")
    for batch in (72, 24):
        E = P.Engine(shape, w, dtype, 3 * n * 16 * P.kv_bytes_per_token(shape, dtype, fp8), max_seqs=n,
                     max_seq_len=64, max_batch=n, max_chunk=64, kv_fp8=fp8)
        ids = [E.kv_alloc(0) for _ in range(n)]
        for i, s in enumerate(ids):
            E.kv_append_prefix(s, random_tokens(1 + i % 33, shape.vocab, i), chunk_tokens=64)
        logits = torch.empty((n, shape.vocab), device="cuda")
        for b in range(0, n, batch):
            E.decode_step(ids[b:b + batch], last[b:b + batch], logits[b:b + batch])
        at = torch.tensor([1 + i % 33 for i in range(n)], device="cuda")
        pg = torch.tensor([int(E.kv_block_table(s)[(1 + i % 33) // 16]) for i, s in enumerate(ids)],
                          device="cuda")
        view = lambda t: (t.view(torch.float8_e4m3fn) if kind == "fp8" else t).float()
        pages.append((view(E.k_pages(0))[pg, :, at % 16], view(E.v_pages(0))[pg, :, :, at % 16]))
    step = {"f32": 2.0 ** -20, "bf16": 2.0 ** -7, "fp8": 2.0 ** -3}[kind]
    for a, b in zip(*pages):
        floor = 2.0 ** -9 if kind == "fp8" else 1e-6
        assert torch.all((a - b).abs() <= step * torch.maximum(a.abs(), b.abs()) + floor)
        assert a.abs().max() > 0
