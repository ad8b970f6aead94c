"""Branches of the top-p sampler against the oracle, token for token.

The sampler orders tokens by logit and cuts its threshold bin into ranges of the
integer keys where the bin holds more tokens than its list, or lies where one key
spans several bins; top_p = 1 skips the threshold; rows that do not start 16-byte
aligned are read word by word.  Each row shape below takes one of these, at
vocabularies around the index-block edges, in the one-group form and in the split
form.  Rows of many equal logits (the ties that join the nucleus, a sample of the
row that shows one key or misleads) have a test of their own, and one of the time:
no row shape may fall far behind an ordinary one.
"""

import numpy as np
import pytest
import torch

from oracle.sampling import sample_top_p as oracle_sample

pytestmark = pytest.mark.gpu


def _rows(kind, n, vocab, rng):
    if kind == "normal":
        return rng.standard_normal((n, vocab)) * 3.0
    if kind == "narrow":    # every token within one or two bins: the list overflows
        return rng.standard_normal((n, vocab)) * 0.01
    if kind == "wide":      # thresholds among masses of a few units
        return rng.standard_normal((n, vocab)) * 7.0
    if kind == "steps":     # tie groups, ending in masses of 1 and 0
        return -rng.integers(0, 30, size=(n, vocab)).astype(np.float64)
    if kind == "close":     # pairs one float apart around every bin edge
        z = -rng.integers(0, 400, size=(n, vocab)) * (np.log(2.0) / 16.0) - np.log(2.0) / 32.0
        return z * (1.0 + rng.integers(-2, 3, size=z.shape) * 2.0 ** -23)
    z = np.full((n, vocab), -np.inf)  # "masked": few finite logits
    z[:, :: max(1, vocab // 7)] = rng.standard_normal(z[:, :: max(1, vocab // 7)].shape)
    return z


@pytest.mark.parametrize("kind,vocab,top_p,offset", [
    ("normal", 151936, 0.95, 0), ("normal", 131073, 0.9, 0), ("normal", 128256, 0.95, 1),
    ("normal", 32772, 1.0, 0), ("normal", 1, 0.5, 0), ("normal", 257, 0.999, 0),
    ("narrow", 40000, 0.6, 0), ("narrow", 140001, 0.3, 0), ("narrow", 40000, 1.0, 0),
    ("wide", 50000, 0.9999999, 0), ("wide", 50001, 1.0, 0), ("steps", 30000, 0.9999999, 0),
    ("steps", 30000, 0.75, 3), ("close", 20000, 0.8, 0), ("close", 20000, 0.99999, 0),
    ("masked", 20000, 0.9, 0),
])
def test_sampler_paths_match_oracle(kind, vocab, top_p, offset):
    import paper_2609_36899_amd as P
    rng = np.random.default_rng(vocab + len(kind))
    n = 3
    z = _rows(kind, n, vocab, rng).astype(np.float32)
    u = rng.random(n).astype(np.float32)
    buf = torch.empty(offset + n * vocab, dtype=torch.float32, device="cuda")
    zd = buf[offset:].view(n, vocab)  # offset words off the allocation's alignment
    zd.copy_(torch.from_numpy(z))
    ud = torch.from_numpy(u).cuda()
    for temperature in (1.0, 0.8):
        want = [oracle_sample(z[b], temperature, top_p, u[b]) for b in range(n)]
        for split in (True, False):
            out = torch.full((n,), -1, dtype=torch.int32, device="cuda")
            P.sample_top_p(zd, out, temperature, top_p, ud, split=split)
            np.testing.assert_array_equal(out.cpu().numpy(), want)


def _tied(kind, n, vocab, rng):
    z = np.zeros((n, vocab))
    if kind == "two":          # both in the top bin, in different ranges of it
        z[:, ::3] = 0.01
    elif kind == "coarse":     # logits as bf16 would hold them
        z = rng.standard_normal((n, vocab)).astype(np.float32) * np.float32(0.1)
        z = (z.view(np.uint32) & np.uint32(0xFFFF0000)).view(np.float32)
    elif kind == "misled":     # one range of keys; its first tokens all have the higher one
        z[:, 2000:] = -2.0 ** -16
    elif kind == "late":       # the first tokens are below the range
        z[:, :1100] = -1.0
        z[:, 1100::2] = -2.0 ** -16
    elif kind == "deep":       # ties among masses of a few units
        z[:, 1:] = -27.0 - 0.001 * rng.integers(0, 3, (n, vocab - 1))
    return z


@pytest.mark.parametrize("kind", ["equal", "two", "coarse", "misled", "late", "deep"])
@pytest.mark.parametrize("vocab,top_p", [(8192, 0.95), (8193, 0.5), (40000, 0.9), (140000, 0.7),
                                         (128257, 0.9999999)])
def test_many_equal_logits_match_oracle(kind, vocab, top_p):
    import paper_2609_36899_amd as P
    rng = np.random.default_rng(vocab)
    n = 3
    z = _tied(kind, n, vocab, rng).astype(np.float32)
    u = np.array([0.0, 0.37, 0.9999], dtype=np.float32)
    zd, ud = torch.from_numpy(z).cuda(), torch.from_numpy(u).cuda()
    want = [oracle_sample(z[b], 0.8, top_p, u[b]) for b in range(n)]
    for split in (True, False):
        out = torch.full((n,), -1, dtype=torch.int32, device="cuda")
        P.sample_top_p(zd, out, 0.8, top_p, ud, split=split)
        np.testing.assert_array_equal(out.cpu().numpy(), want)


@pytest.mark.parametrize("B", [16, 64])
@pytest.mark.parametrize("kind", ["equal", "two", "coarse", "narrow"])
@pytest.mark.parametrize("vocab", [8192, 128256])
def test_no_row_shape_is_slow(B, kind, vocab):
    """At most five times an ordinary row's time (measured: 0.9 to 3; a rank of ties by
    all pairs of them took up to 220 times it)."""
    import paper_2609_36899_amd as P
    rng = np.random.default_rng(1)
    u = torch.from_numpy(rng.random(B).astype(np.float32)).cuda()
    out = torch.empty(B, dtype=torch.int32, device="cuda")

    def us(z):
        zd = torch.from_numpy(z.astype(np.float32)).cuda()
        for _ in range(3):
            P.sample_top_p(zd, out, 0.8, 0.95, u)
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(20):
            P.sample_top_p(zd, out, 0.8, 0.95, u)
        b.record()
        b.synchronize()
        return a.elapsed_time(b) * 50.0

    z = _rows(kind, B, vocab, rng) if kind == "narrow" else _tied(kind, B, vocab, rng)
    assert us(z) <= 5.0 * us(_rows("normal", B, vocab, rng))
