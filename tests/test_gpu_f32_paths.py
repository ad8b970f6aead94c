"""The fp32 kernels at the edges of their tiles, against float64.

Attention: context lengths around the 16-token pages, the 64-key tiles and the
128-key items (one item: normalised in the split pass; several: merged), GQA
groups that fill a wave's rows unevenly, slots past a context's end NaN.
Projections: row counts around each form of the few-row kernel and its limit of
16, K around its 256-wide steps, columns that do not fill a wave, and inputs
that are not 16-byte aligned (the same sums).

Tolerances: a lane adds at most K/64 + 16 products (attention: dims, then keys)
in a chain of fp32 roundings, so |error| <= (n + 16) 2^-24 sum |a||b| for a
projection; attention outputs are convex sums of N(0, 1) values whose weights
carry the score's error, (dims + keys/64 + 16) 2^-24 times scores of size < 16.
"""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _attention64(q, k, v):
    """q [Hq][Dh], k and v [n][Hkv][Dh] in float64."""
    hq, dh = q.shape
    g = hq // k.shape[1]
    out = np.empty_like(q)
    for h in range(hq):
        s = k[:, h // g] @ q[h] / np.sqrt(dh)
        p = np.exp(s - s.max())
        out[h] = (p / p.sum()) @ v[:, h // g]
    return out


@pytest.mark.parametrize("hq,hkv,dh", [(4, 2, 64), (5, 1, 128), (16, 1, 64), (12, 4, 128), (2, 2, 64)])
@pytest.mark.parametrize("lens", [(1, 15, 16, 17), (63, 64, 65, 127), (128,), (129, 3, 1000, 640)])
def test_attention_tile_edges(hq, hkv, dh, lens):
    import paper_2609_36899_amd as P
    from workload import paged_attention_case
    case = paged_attention_case(len(lens), hq, hkv, dh, np.array(lens), 200, seed=7 + dh, bf16=False)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    out = torch.full((len(lens), hq, dh), np.nan, device="cuda")
    bt = dev(np.maximum(case.block_table, 0))
    P.paged_decode_attention(dev(case.q), dev(case.k_pool), dev(case.v_pool.transpose(0, 1, 3, 2)),
                             bt, lens, out)
    got = out.cpu().numpy()
    for b, n in enumerate(lens):
        pages = case.block_table[b, :(n + 15) // 16]
        flat = lambda pool: pool[pages].transpose(0, 2, 1, 3).reshape(-1, hkv, dh)[:n].astype(np.float64)
        ref = _attention64(case.q[b].astype(np.float64), flat(case.k_pool), flat(case.v_pool))
        tol = (dh + n / 64 + 16) * 2.0 ** -24 * 16
        assert np.max(np.abs(got[b] - ref)) <= tol


def test_attention_pages_of_any_alignment():
    """Pools that start at an element's own alignment: the same bits."""
    import paper_2609_36899_amd as P
    from workload import paged_attention_case
    lens = (1, 17, 130, 400)
    case = paged_attention_case(4, 4, 2, 64, np.array(lens), 60, seed=3, bf16=False)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    bt, q = dev(np.maximum(case.block_table, 0)), dev(case.q)
    k, v = dev(np.nan_to_num(case.k_pool)), dev(np.nan_to_num(case.v_pool).transpose(0, 1, 3, 2))
    res = []
    for shift in (0, 1, 2):
        at = lambda t: torch.cat([torch.zeros(shift, device="cuda"), t.flatten()])[shift:].view(t.shape)
        out = torch.empty((4, 4, 64), device="cuda")
        P.paged_decode_attention(q, at(k), at(v), bt, lens, out)
        res.append(out)
    assert torch.equal(res[1], res[0]) and torch.equal(res[2], res[0])


@pytest.mark.parametrize("M", [1, 2, 3, 4, 5, 8, 9, 16, 17])
@pytest.mark.parametrize("N,K,shift", [(4, 4, 0), (516, 252, 0), (1024, 256, 0), (260, 688, 0),
                                       (64, 1030, 0), (132, 256, 1)])
def test_projection_rows(M, N, K, shift):
    import paper_2609_36899_amd as P
    rng = np.random.default_rng(M * 1000 + K)
    x, w, w2 = (rng.standard_normal(s).astype(np.float32) for s in ((M, K), (N, K), (N, K)))
    buf = torch.empty(shift + M * K, device="cuda")
    xd = buf[shift:].view(M, K)
    xd.copy_(torch.from_numpy(x))
    wd, wd2 = (P.pack_weight(torch.from_numpy(a).cuda()) for a in (w, w2))
    x64, w64, u64 = x.astype(np.float64), w.astype(np.float64), w2.astype(np.float64)
    eps = (K / 64 + 16) * 2.0 ** -24
    out = torch.full((M, N), np.nan, device="cuda")
    P.weight_projection(xd, wd, out)
    bound = eps * (np.abs(x64) @ np.abs(w64).T)
    assert np.all(np.abs(out.cpu().numpy() - x64 @ w64.T) <= bound)
    u = torch.full((M, N), np.nan, device="cuda")
    P.swiglu_projection(xd, wd, wd2, u)
    g, up = x64 @ w64.T, x64 @ u64.T
    ref = g / (1 + np.exp(-g)) * up
    # d silu <= 1.1 per unit of g; expf and the divide add a few roundings.
    tol = 1.1 * bound * np.abs(up) + eps * (np.abs(x64) @ np.abs(u64).T) * np.abs(g) + \
        8 * 2.0 ** -24 * np.abs(ref) + 1e-30
    assert np.all(np.abs(u.cpu().numpy() - ref) <= tol)


@pytest.mark.parametrize("M", [1, 4, 8, 16])
@pytest.mark.parametrize("shift", [1, 2])
def test_projection_rows_of_any_alignment(M, shift):
    """Activations and weights that start at an element's own alignment take the same
    kernel as aligned ones: the same bits."""
    import paper_2609_36899_amd as P
    N, K = 516, 688
    gen = torch.Generator("cuda").manual_seed(M)
    x, w, w2 = (torch.randn(s, device="cuda", generator=gen) for s in ((M, K), (N, K), (N, K)))

    def off(t):  # the same values at an odd place
        buf = torch.empty(shift + t.numel(), device="cuda")
        buf[shift:].copy_(t.flatten())
        return buf[shift:].view(t.shape)

    res = []
    for f in (lambda t: t, off):
        pw = [P.PackedWeight(f(t), N, K, P.F32) for t in (w, w2)]  # fp32: row-major as it is
        out, u = torch.empty((M, N), device="cuda"), torch.empty((M, N), device="cuda")
        P.weight_projection(f(x), pw[0], out)
        P.swiglu_projection(f(x), pw[0], pw[1], u)
        res.append((out, u))
    for a, b in zip(*res):
        assert torch.equal(a, b)


@pytest.mark.parametrize("n,bad", [(20, 19), (40, 17), (200, 199), (200, 70)])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_prefill_rows_do_not_see_later_tokens(n, bad, value):
    """A token whose embedding is not finite has K and V that are not: earlier tokens,
    in its query block too, must not take anything from it.  Their layer-1 K and V,
    which depend on layer 0's attention, are compared with those of the same tokens
    with another one in its place: the same sums."""
    import paper_2609_36899_amd as P
    from workload import TINY, make_weights, random_tokens
    w = make_weights(TINY, seed=3, bf16=False)
    toks = random_tokens(n, TINY.vocab, 5)
    marked, plain = TINY.vocab - 1, TINY.vocab - 2
    toks = [t if t < plain else 0 for t in toks]
    w["embed"] = w["embed"].copy()
    w["embed"][marked] = value
    kv = []
    for tok in (plain, marked):
        E = P.Engine(TINY, P.weights_to_device(w, P.F32), P.F32,
                     16 * 16 * P.kv_bytes_per_token(TINY, P.F32), max_seqs=1, max_seq_len=256,
                     max_batch=1, max_chunk=256)
        s = E.kv_alloc(0)
        E.kv_append_prefix(s, toks[:bad] + [tok] + toks[bad + 1:], chunk_tokens=256)
        at = torch.arange(n, device="cuda")
        pg = torch.from_numpy(E.kv_block_table(s)).cuda().long()[at // 16]
        kv.append((E.k_pages(1)[pg, :, at % 16].clone(), E.v_pages(1)[pg, :, :, at % 16].clone()))
    for want, got in zip(*kv):
        assert not torch.isfinite(got[bad]).all()
        assert torch.equal(got[:bad], want[:bad]) and torch.isfinite(want).all()
