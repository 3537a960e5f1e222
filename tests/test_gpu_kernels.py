"""GPU parity, stage by stage: each kernel-level entry point of the C ABI against
the oracle's definition of that stage, on seeded inputs that span several tiles
and a ragged tail."""
import numpy as np
import pytest
import torch

from oracle import dare_oracle as orc
from paper_2605_08134_amd import synth
from parity_util import assert_close, dev, host, rel_err, store

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2605_08134_amd import binding
    binding.lib()
    return binding


def _rng(seed):
    return np.random.Generator(np.random.PCG64(seed))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_pack_weight_is_exact_transpose(B, dtype):
    w = store(_rng(1).standard_normal((192, 320)), dtype)
    wt = B.dare_k_pack_weight(dev(w, dtype))
    torch.cuda.synchronize()
    assert np.array_equal(host(wt), w.T)


@pytest.mark.parametrize("dtype,m,n,k,seg", [
    ("bf16", 300, 384, 256, 128),     # 3 segments, ragged rows
    ("bf16", 128, 128, 64, 128),      # exactly one tile, one k step
    ("bf16", 1, 64, 128, 64),         # single row, narrow tile config
    ("bf16", 517, 1024, 512, 1024),   # many tiles
    ("f32", 150, 192, 64, 64),
    ("f32", 64, 64, 64, 64),
])
def test_gemm_all_rows(B, dtype, m, n, k, seg):
    r = _rng(m + n)
    a = store(r.standard_normal((m, k)), dtype)
    w = store(r.standard_normal((k, n)) * 0.05, dtype)
    wt = B.dare_k_pack_weight(dev(w, dtype))
    nseg = n // seg
    outs = [torch.zeros((m, seg), dtype=wt.dtype, device="cuda") for _ in range(nseg)]
    c32_cols = min(64, n)
    c32 = torch.zeros((m, c32_cols), dtype=torch.float32, device="cuda")
    B.dare_k_gemm(dev(a, dtype), wt, outs, seg, c32=c32)
    torch.cuda.synchronize()
    want = a.astype(np.float64) @ w.astype(np.float64)
    got = np.concatenate([host(o) for o in outs], axis=1)
    assert_close(got, want, dtype)
    assert rel_err(host(c32), want[:, :c32_cols]) <= 2e-6     # fp32 accumulators, unrounded


# (the text begins with the tile shape: tests/test_gemm_route.py checks it against the rule)
LARGE_TILES = [
    (1000, 12288, 64, 4096, "256 x 192, one k-step, ragged rows"),
    (961, 12096, 192, 12096, "256 x 192, an odd number of k-steps, one row in the last tile's last 64"),
    (1024, 12480, 128, 4160, "256 x 256, ragged columns"),
    (1793, 8192, 320, 4096, "256 x 256, five k-steps, one row in the last tile"),
    (1500, 12160, 192, 12160, "256 x 192 four waves, three k-steps, ragged both ways"),
    (1500, 12160, 320, 12160, "256 x 192 four waves, five k-steps, ragged both ways"),
    (1793, 12480, 256, 4160, "256 x 256 four waves, four k-steps, ragged columns, one row in the last tile"),
    (1793, 12480, 448, 4160, "256 x 256 four waves, seven k-steps, ragged columns, one row in the last tile"),
    (1793, 12480, 128, 4160, "256 x 256, two rounds of two k-steps"),
    (2100, 2112, 64, 2112, "256 x 128, one k-step, ragged both ways"),
    (2305, 2048, 320, 2048, "256 x 128, five k-steps, one row in the last tile"),
    (33, 24640, 64, 24640, "64 x 128, one k-step, ragged both ways"),
    (64, 24576, 448, 8192, "64 x 96, one row tile, seven k-steps, full rows"),
    (65, 8256, 64, 8256, "64 x 96, one k-step, one row in the last tile"),
    (128, 8192, 320, 4096, "64 x 64, two row tiles, five k-steps"),
]


@pytest.mark.parametrize("m,n,k,seg,tile", LARGE_TILES)
def test_gemm_all_rows_large_tiles(B, m, n, k, seg, tile):
    r = _rng(m + n + k)
    a = store(r.standard_normal((m, k), dtype=np.float32), "bf16")
    w = store(r.standard_normal((k, n), dtype=np.float32) * np.float32(0.05), "bf16")
    wt = B.dare_k_pack_weight(dev(w, "bf16"))
    outs = [torch.full((m, seg), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(n // seg)]
    c32 = torch.full((m, 68), float("nan"), dtype=torch.float32, device="cuda")    # ends inside a lane's eight columns
    B.dare_k_gemm(dev(a, "bf16"), wt, outs, seg, c32=c32)
    torch.cuda.synchronize()
    want = a.astype(np.float64) @ w.astype(np.float64)
    assert_close(np.concatenate([host(o) for o in outs], axis=1), want, "bf16")
    assert rel_err(host(c32), want[:, :68]) <= 2e-6     # fp32 accumulators, unrounded


@pytest.mark.parametrize("m,n,k,tile", [
    (17, 80, 64, "16 x 16, one step per quarter of k"),
    (150, 1296, 320, "32 x 32, five steps per quarter (a chunk of four and a rest), ragged both ways"),
    (600, 1296, 448, "64 x 64, ragged both ways"),
    (1473, 2064, 192, "64 x 64, many tiles, one row in the last row tile's last 16"),
])
def test_gemm_f32_tile_shapes_agree_bit_for_bit(B, m, n, k, tile):
    """The sum over k has one order whatever the tile shape: a row of the launch equals the
    same row projected alone, for the first 16 columns alone as well."""
    r = _rng(m + n + k)
    a = r.standard_normal((m, k), dtype=np.float32)
    w = r.standard_normal((k, n), dtype=np.float32) * np.float32(0.05)
    wt, ad = B.dare_k_pack_weight(dev(w, "f32")), dev(a, "f32")

    def project(rows, weight):
        out = torch.full((rows.shape[0], weight.shape[0]), float("nan"), device="cuda")
        B.dare_k_gemm(rows, weight, [out], weight.shape[0])
        torch.cuda.synchronize()
        return host(out)

    got = project(ad, wt)
    assert rel_err(got, a.astype(np.float64) @ w.astype(np.float64)) <= 2e-6
    assert np.array_equal(project(ad[m - 1:].contiguous(), wt)[0], got[m - 1])
    assert np.array_equal(project(ad, wt[:16].contiguous()), got[:, :16])


@pytest.mark.parametrize("seq,dh", [(1, 128), (31, 64), (33, 128), (129, 64), (161, 128)])
def test_attention_f32_edges(B, seq, dh):
    """Key-waves without a tile, ragged 32-key tiles and ragged 16-row query blocks."""
    q, k, v, _ = _attn_case(seq + dh, 2, seq, 2, dh, "f32", 1.0)
    out = torch.full((2 * seq, 2 * dh), float("nan"), device="cuda")
    B.dare_k_attention(dev(q, "f32"), dev(k, "f32"), dev(v, "f32"), out, 2, seq, 2, dh)
    torch.cuda.synchronize()
    for b in range(2):
        sl = slice(b * seq, (b + 1) * seq)
        assert rel_err(host(out)[sl], orc.attention_rows(q[sl], k[sl], v[sl], 2)) <= 1e-5


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("count", [0, 1, 16, 17, 32, 33, 129, 205])
def test_gemm_selected_rows_device_count(B, dtype, count):
    r = _rng(count + 5)
    n_tok, k, n = 400, 128, 256
    a = store(r.standard_normal((n_tok, k)), dtype)
    w = store(r.standard_normal((k, n)) * 0.05, dtype)
    wt = B.dare_k_pack_weight(dev(w, dtype))
    rows = np.sort(r.permutation(n_tok)[:count]).astype(np.int32)
    idx = np.full(n_tok, 10 ** 6, dtype=np.int32)      # entries past the count must never be used
    idx[:count] = rows
    sentinel = store(np.full((n_tok, 128), 3.0), dtype)
    outs = [dev(sentinel, dtype), dev(sentinel, dtype)]
    m_dev = torch.tensor([count], dtype=torch.int32, device="cuda")
    B.dare_k_gemm(dev(a, dtype), wt, outs, 128, idx=dev(idx), m_dev=m_dev, m_max=n_tok)
    torch.cuda.synchronize()
    got = np.concatenate([host(o) for o in outs], axis=1)
    want = np.full((n_tok, n), 3.0)
    want[rows] = a[rows].astype(np.float64) @ w.astype(np.float64)
    untouched = np.setdiff1d(np.arange(n_tok), rows)
    assert np.all(got[untouched] == 3.0)
    if count:
        assert_close(got[rows], want[rows], dtype)


@pytest.mark.parametrize("n_tok,count", [(1024, 0), (1024, 1), (1024, 7), (1024, 16), (1024, 17), (1024, 32), (1024, 33), (1024, 52), (1024, 100), (1024, 205),
                                         (1024, 700), (1024, 1024), (3072, 2900), (4096, 2561), (4096, 3266),
                                         (4096, 3500)])
def test_gemm_selected_rows_wide_output(B, n_tok, count):
    """12288 columns, the tile shape follows the device-side row count: 64 x 64, 128 x 48, 128 x 96,
    256 x 192, 256 x 256 in rounds over 256 workgroups.  2561, 2900 and 3266 rows leave a last round that
    is at most half full and is cut into 128 x 128 tiles (64, 256 and 448 of them, some
    without rows); 3500 rows walk three rounds of whole tiles."""
    r = _rng(count + 77)
    k, seg = 192, 4096
    n = 3 * seg
    a = store(r.standard_normal((n_tok, k)), "bf16")
    w = store(r.standard_normal((k, n)) * 0.05, "bf16")
    wt = B.dare_k_pack_weight(dev(w, "bf16"))
    rows = np.sort(r.permutation(n_tok)[:count]).astype(np.int32)
    idx = np.full(n_tok, 10 ** 6, dtype=np.int32)
    idx[:count] = rows
    outs = [torch.full((n_tok, seg), 3.0, dtype=torch.bfloat16, device="cuda") for _ in range(3)]
    m_dev = torch.tensor([count], dtype=torch.int32, device="cuda")
    B.dare_k_gemm(dev(a, "bf16"), wt, outs, seg, idx=dev(idx), m_dev=m_dev, m_max=n_tok)
    torch.cuda.synchronize()
    got = np.concatenate([host(o) for o in outs], axis=1)
    untouched = np.setdiff1d(np.arange(n_tok), rows)
    assert np.all(got[untouched] == 3.0)
    if count:
        want = a[rows].astype(np.float64) @ w.astype(np.float64)
        assert_close(got[rows], want, "bf16")


_LONG_K = {}


def _long_k_operands(n):
    """a [1200, 4096] and w [4096, n], drawn once per width (the wide one is 200 MB)."""
    if n not in _LONG_K:
        r = _rng(4096 + n)
        a = store(r.standard_normal((1200, 4096), dtype=np.float32), "bf16")
        w = store(r.standard_normal((4096, n), dtype=np.float32) * np.float32(0.02), "bf16")
        _LONG_K.clear()
        _LONG_K[n] = (a, w)
    return _LONG_K[n]


LONG_K_TILES = [
    (1024, 1100, "128 x 48, ragged both ways"),
    (4096, 16, "stream, one row block, full"),
    (4096, 17, "stream, two row blocks, one row in the second"),
    (4096, 24, "stream, two row blocks"),
    (4096, 32, "stream, two full row blocks"),
    (4096, 33, "64 x 64, one row tile"),
    (4096, 64, "64 x 64, one full row tile"),
    (4096, 65, "64 x 64, one row in the second row tile"),
    (4096, 205, "64 x 64, four row tiles"),
    (4096, 256, "64 x 64, 256 tiles"),
    (4096, 257, "128 x 64, one row in the third row tile"),
    (4096, 400, "128 x 64"),
    (12288, 64, "64 x 64, full row tile"),
    (12288, 65, "128 x 48, one row beyond 64"),
    (12288, 128, "128 x 48, full row tile"),
    (12288, 129, "128 x 96, one row in the second row tile"),
    (12288, 24, "64 x 64"),
    (12288, 100, "128 x 48"),
    (12288, 205, "128 x 96"),
    (12288, 257, "128 x 192, one row in the third row tile"),
    (12288, 384, "128 x 192, full row tiles"),
    (12288, 400, "256 x 128"),
    (12288, 600, "256 x 192"),
    (12288, 900, "256 x 192"),
]


@pytest.mark.parametrize("n,count,shape", LONG_K_TILES)
def test_gemm_selected_rows_long_k(B, n, count, shape):
    """The device-side tile choice at k = 4096 (64 k-steps: the operand ring of every shape
    runs in its steady state, not only its prologue), rows gathered through a list, output
    rows written at their token index."""
    a, w = _long_k_operands(n)
    n_tok, k = a.shape
    r = _rng(count)
    seg = n if n <= 4096 else 4096
    rows = np.sort(r.permutation(n_tok)[:count]).astype(np.int32)
    idx = np.full(n_tok, 10 ** 6, dtype=np.int32)
    idx[:count] = rows
    wt = B.dare_k_pack_weight(dev(w, "bf16"))
    outs = [torch.full((n_tok, seg), 3.0, dtype=torch.bfloat16, device="cuda") for _ in range(n // seg)]
    m_dev = torch.tensor([count], dtype=torch.int32, device="cuda")
    B.dare_k_gemm(dev(a, "bf16"), wt, outs, seg, idx=dev(idx), m_dev=m_dev, m_max=n_tok)
    torch.cuda.synchronize()
    got = np.concatenate([host(o) for o in outs], axis=1)
    untouched = np.setdiff1d(np.arange(n_tok), rows)
    assert np.all(got[untouched] == 3.0)
    want = a[rows].astype(np.float64) @ w.astype(np.float64)
    assert_close(got[rows], want, "bf16")


@pytest.mark.parametrize("n_tok", [1024, 1025])   # 256 tiles of 64 x 64 for all rows: a kernel of that shape alone; 272: the one of all shapes
@pytest.mark.parametrize("count", [0, 1, 16, 17, 32, 33, 1000, 1024])
def test_gemm_listed_rows_around_one_round_of_the_smallest_tiles(B, n_tok, count):
    n = k = 1024
    r = _rng(n_tok + count)
    a = store(r.standard_normal((n_tok, k), dtype=np.float32), "bf16")
    w = store(r.standard_normal((k, n), dtype=np.float32) * np.float32(0.05), "bf16")
    rows = np.sort(r.permutation(n_tok)[:count]).astype(np.int32)
    idx = np.full(n_tok, 10 ** 6, dtype=np.int32)
    idx[:count] = rows
    out = torch.full((n_tok, n), 3.0, dtype=torch.bfloat16, device="cuda")
    B.dare_k_gemm(dev(a, "bf16"), B.dare_k_pack_weight(dev(w, "bf16")), [out], n, idx=dev(idx),
                  m_dev=torch.tensor([count], dtype=torch.int32, device="cuda"), m_max=n_tok)
    torch.cuda.synchronize()
    got = host(out)
    assert np.all(got[np.setdiff1d(np.arange(n_tok), rows)] == 3.0)
    if count:
        assert_close(got[rows], a[rows].astype(np.float64) @ w.astype(np.float64), "bf16")


# every shape of best_tile: ragged last row tile, n that is no multiple of the tile's columns, odd k-steps
EVERY_TILE = {
    (False, 402, 512): "64 x 64", (False, 1000, 1536): "64 x 96", (False, 1001, 2048): "64 x 128",
    (False, 2331, 1024): "128 x 96", (False, 1001, 4096): "128 x 128", (False, 300, 12288): "128 x 192",
    (False, 1025, 6080): "256 x 128", (False, 1300, 6144): "256 x 192", (False, 1000, 9216): "256 x 192",
    (False, 2331, 6144): "256 x 256",
    (True, 33, 512): "64 x 64", (True, 400, 3072): "128 x 48", (True, 300, 4096): "128 x 64", (True, 601, 4096): "128 x 96",
    (True, 777, 4096): "128 x 128", (True, 300, 12288): "128 x 192", (True, 1300, 4096): "256 x 128",
    (True, 1000, 9216): "256 x 192", (True, 2900, 4096): "256 x 256",
    (True, 3101, 12288): "256 x 256 cut",   # the last round in 128 x 128
}


EVERY_TILE_SIZES = [
    (False, 402, 512, 192), (False, 1000, 1536, 128), (False, 1001, 2048, 64), (False, 2331, 1024, 192),
    (False, 1001, 4096, 64), (False, 1025, 6080, 128), (False, 1300, 6144, 64), (False, 1000, 9216, 128),
    (False, 2331, 6144, 64),
    (True, 33, 512, 192), (True, 400, 3072, 128), (True, 300, 4096, 64), (True, 601, 4096, 192),
    (True, 777, 4096, 128), (True, 1300, 4096, 64), (True, 1000, 9216, 128), (True, 2900, 4096, 64),
    (True, 3101, 12288, 64),
    # k-steps around the length of the ring, odd and even: the last of them load nothing
    *((False, m, n, k) for m, n in ((1000, 1536), (1001, 4096), (1300, 6144), (1000, 9216), (2331, 6144))
      for k in (256, 320, 384, 448)),
    *((True, m, n, k) for m, n in ((400, 3072), (601, 4096), (777, 4096), (1300, 4096), (1000, 9216), (2900, 4096))
      for k in (256, 320, 384, 448)),
    # 128 x 192, whose ring is the shortest: one to seven k-steps
    *((listed, 300, 12288, k) for listed in (False, True) for k in (64, 128, 192, 256, 320, 448)),
]


@pytest.mark.parametrize("listed,m,n,k", EVERY_TILE_SIZES)
def test_gemm_every_tile_shape(B, listed, m, n, k):
    assert (listed, m, n) in EVERY_TILE
    r = _rng(m + n + k)
    n_tok = m + 50 if listed else m
    a = store(r.standard_normal((n_tok, k), dtype=np.float32), "bf16")
    w = store(r.standard_normal((k, n), dtype=np.float32) * np.float32(0.05), "bf16")
    wt = B.dare_k_pack_weight(dev(w, "bf16"))
    out = torch.full((n_tok, n), 3.0, dtype=torch.bfloat16, device="cuda")
    rows = np.sort(r.permutation(n_tok)[:m]).astype(np.int32)
    if listed:
        idx = np.full(n_tok, 10 ** 6, dtype=np.int32)
        idx[:m] = rows
        B.dare_k_gemm(dev(a, "bf16"), wt, [out], n, idx=dev(idx), m_dev=torch.tensor([m], dtype=torch.int32, device="cuda"),
                      m_max=n_tok)
    else:
        B.dare_k_gemm(dev(a, "bf16"), wt, [out], n)
    torch.cuda.synchronize()
    got = host(out)
    assert np.all(got[np.setdiff1d(np.arange(n_tok), rows)] == 3.0)
    assert_close(got[rows], a[rows].astype(np.float64) @ w.astype(np.float64), "bf16")


def test_gemm_k_parts_feed_the_score(B):
    # the scored-columns projection cut along k: slabs of partial sums that the score
    # kernel adds up, against the uncut projection and the oracle's score
    r = _rng(3)
    m, k, n, parts = 1000, 2048, 128, 4
    a = store(r.standard_normal((m, k)), "bf16")
    w = store(r.standard_normal((k, n)) * 0.03, "bf16")
    wt = B.dare_k_pack_weight(dev(w, "bf16"))
    slabs = torch.full((parts, m, n), float("nan"), dtype=torch.float32, device="cuda")
    B.dare_k_gemm(dev(a, "bf16"), wt, [None], n, m_max=m, c32=slabs, k_parts=parts)
    torch.cuda.synchronize()
    want = a.astype(np.float64) @ w.astype(np.float64)
    assert rel_err(host(slabs).sum(axis=0), want) <= 2e-6
    for s in range(parts):
        ks = slice(s * k // parts, (s + 1) * k // parts)
        assert rel_err(host(slabs[s]), a[:, ks].astype(np.float64) @ w[ks].astype(np.float64)) <= 2e-6
    p = (want + 0.05 * r.standard_normal(want.shape)).astype(np.float32)
    pd = dev(p)
    scores = torch.zeros(m, dtype=torch.float32, device="cuda")
    mask = torch.zeros(m, dtype=torch.uint8, device="cuda")
    B.dare_k_score(slabs.view(parts * m, n), pd, 0.01, False, scores, mask, n_parts=parts)
    torch.cuda.synchronize()
    assert np.max(np.abs(host(scores) - orc.drift_scores(want, p))) < 5e-7
    assert rel_err(host(pd), want) <= 2e-6


@pytest.mark.parametrize("m,n,k,parts", [
    (8192, 128, 256, 2), (8193, 128, 256, 2),   # the last size in 64 x 64 tiles, the first in 128 x 128, one row in the last
    (65, 8192, 512, 8), (1025, 3072, 192, 3),   # 128 x 128: one k-step per range
    (300, 4096, 768, 4), (200, 192, 512, 4), (1, 64, 128, 2),   # 64 x 64: three k-steps, three column tiles, one row
])
def test_gemm_k_in_ranges(B, m, n, k, parts):
    r = _rng(m + n)
    a = store(r.standard_normal((m, k), dtype=np.float32), "bf16")
    w = store(r.standard_normal((k, n), dtype=np.float32) * np.float32(0.05), "bf16")
    slabs = torch.full((parts + 1, m, n), 7.0, dtype=torch.float32, device="cuda")
    B.dare_k_gemm(dev(a, "bf16"), B.dare_k_pack_weight(dev(w, "bf16")), [None], n, m_max=m, c32=slabs, k_parts=parts)
    torch.cuda.synchronize()
    got = host(slabs)
    assert np.all(got[parts] == 7.0)
    for s in range(parts):
        ks = slice(s * k // parts, (s + 1) * k // parts)
        assert rel_err(got[s], a[:, ks].astype(np.float64) @ w[ks].astype(np.float64)) <= 2e-6


def test_score_kernel(B):
    r = _rng(9)
    n, w, ld = 333, 128, 160
    q = r.standard_normal((n, ld)).astype(np.float32)
    p = r.standard_normal((n, w)).astype(np.float32)
    p[:40] = q[:40, :w]                      # unchanged tokens: score exactly 0
    p[40:60] = 2.5 * q[40:60, :w]            # rescaled: score ~ 0
    p[60:70] = -q[60:70, :w]                 # opposite: score 2
    p[70] = 0.0                              # zero norm: cosine taken as 0
    p[100:200] = q[100:200, :w] + 0.3 * r.standard_normal((100, w)).astype(np.float32)
    want = orc.drift_scores(q[:, :w], p)
    tau = 0.05
    qd, pd = dev(q), dev(p)
    scores = torch.zeros(n, dtype=torch.float32, device="cuda")
    mask = torch.full((n,), 9, dtype=torch.uint8, device="cuda")
    B.dare_k_score(qd, pd, tau, False, scores, mask)
    torch.cuda.synchronize()
    s = host(scores)
    assert np.all(s[:40] == 0.0)
    assert np.max(np.abs(s - want)) < 5e-7
    assert s[70] == 1.0
    ties = np.abs(want - np.float32(tau)) < 1e-6
    assert np.array_equal(host(mask)[~ties], orc.reuse_decision(want, tau)[~ties].astype(np.uint8))
    assert np.array_equal(host(pd), q[:, :w])                 # score cache replaced for every token
    # force_refresh: scores still reported, mask all zero
    B.dare_k_score(qd, dev(p), 2.5, True, scores, mask)
    torch.cuda.synchronize()
    assert not host(mask).any() and np.max(np.abs(host(scores) - want)) < 5e-7


@pytest.mark.parametrize("batch,seq,frac", [(1, 128, 0.2), (3, 1000, 0.5), (2, 2500, 0.07),
                                            (4, 64, 0.0), (2, 1024, 1.0), (8, 2048, 0.2),
                                            (3, 1031, 0.3), (5, 7, 0.5), (2, 4099, 0.9)])   # sequence starts off the 16-byte grid
def test_compaction_is_ordered_and_exact(B, batch, seq, frac):
    r = _rng(batch * seq)
    reuse = r.random((batch, seq)) >= frac
    mask = dev(reuse.astype(np.uint8))
    sel_idx = torch.full((batch * seq,), -1, dtype=torch.int32, device="cuda")
    sel_count = torch.full((batch,), -1, dtype=torch.int32, device="cuda")
    sel_off = torch.full((batch + 1,), -1, dtype=torch.int32, device="cuda")
    B.dare_k_compact(mask, batch, seq, sel_idx, sel_count, sel_off)
    torch.cuda.synchronize()
    idx, cnt, off = orc.selection(reuse)
    assert np.array_equal(host(sel_idx)[:len(idx)], idx)
    assert np.all(host(sel_idx)[len(idx):] == -1)
    assert np.array_equal(host(sel_count), cnt)
    assert np.array_equal(host(sel_off), off)


def _attn_case(seed, batch, seq, heads, dh, dtype, frac):
    r = _rng(seed)
    d = heads * dh
    q = store(r.standard_normal((batch * seq, d)), dtype)
    k = store(r.standard_normal((batch * seq, d)), dtype)
    v = store(r.standard_normal((batch * seq, d)), dtype)
    reuse = r.random((batch, seq)) >= frac
    return q, k, v, reuse


@pytest.mark.parametrize("dtype,batch,seq,heads,dh", [
    ("bf16", 1, 256, 2, 128), ("bf16", 2, 200, 3, 128), ("bf16", 1, 1, 1, 128),
    ("bf16", 2, 333, 2, 64), ("bf16", 1, 65, 1, 64),
    # enough rows for blocks without key-waves: 128 rows, 256 with heads of 64
    ("bf16", 8, 300, 16, 128), ("bf16", 4, 520, 32, 64),
    ("f32", 1, 128, 4, 64), ("f32", 2, 77, 2, 128), ("f32", 1, 1100, 1, 64),
])
def test_attention_all_rows(B, dtype, batch, seq, heads, dh):
    q, k, v, _ = _attn_case(seq + dh, batch, seq, heads, dh, dtype, 1.0)
    out = torch.zeros((batch * seq, heads * dh), dtype=torch.bfloat16 if dtype == "bf16" else torch.float32,
                      device="cuda")
    B.dare_k_attention(dev(q, dtype), dev(k, dtype), dev(v, dtype), out, batch, seq, heads, dh)
    torch.cuda.synchronize()
    got = host(out)
    for b in range(batch):
        sl = slice(b * seq, (b + 1) * seq)
        want = orc.attention_rows(q[sl], k[sl], v[sl], heads)
        assert_close(got[sl], want, dtype, slack=8.0)


@pytest.mark.parametrize("dtype,batch,seq,heads,dh,frac", [
    ("bf16", 2, 300, 2, 128, 0.2), ("bf16", 3, 200, 1, 128, 0.9), ("bf16", 2, 130, 2, 64, 0.5),
    ("f32", 2, 100, 2, 64, 0.3),
])
def test_attention_selected_rows(B, dtype, batch, seq, heads, dh, frac):
    q, k, v, reuse = _attn_case(seq + 3, batch, seq, heads, dh, dtype, frac)
    reuse[0] = True if batch > 2 else reuse[0]          # a sequence with nothing selected
    idx, cnt, off = orc.selection(reuse)
    idx_full = np.full(batch * seq, 10 ** 6, dtype=np.int32)
    idx_full[:len(idx)] = idx
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    out = torch.full((batch * seq, heads * dh), 5.0, dtype=tdt, device="cuda")
    B.dare_k_attention(dev(q, dtype), dev(k, dtype), dev(v, dtype), out, batch, seq, heads, dh,
                       idx=dev(idx_full), sel_off=dev(off))
    torch.cuda.synchronize()
    got = host(out)
    for b in range(batch):
        sl = slice(b * seq, (b + 1) * seq)
        rows = np.flatnonzero(~reuse[b])
        keep = np.flatnonzero(reuse[b])
        assert np.all(got[sl][keep] == 5.0)               # unselected rows untouched
        if len(rows):
            want = orc.attention_rows(q[sl][rows], k[sl], v[sl], heads)
            assert_close(got[sl][rows], want, dtype, slack=8.0)


@pytest.mark.parametrize("batch,seq,heads,dh,frac", [
    (5, 300, 32, 64, 0.6),        # more than 256 blocks of 64 rows: blocks of 128
    (70, 40, 1, 64, 0.5),         # many short sequences: a workgroup per possible block
    (2, 300, 32, 128, 0.9),       # 64 x 5 blocks: 128 rows, ragged
    (130, 2100, 1, 64, 0.02),     # more sequences than lanes, twice over: 64 rows
    (66, 1153, 8, 64, 0.08),      # the same, two blocks of 64 rows per (sequence, head) or one of 128
    (65, 1100, 4, 128, 0.001),    # the same, half of the sequences without a refreshed row
    (2, 650, 32, 128, 0.9),       # 320 blocks of 128 rows: the last 64 as blocks of 64 rows
    (2, 650, 32, 128, 0.81),      # the same, 12 and 18 rows in the last blocks: the second half of it is empty
])
def test_attention_block_layout_from_the_counts(B, batch, seq, heads, dh, frac):
    """Per element: a probability p_i rounded to bf16 is off by at most 2^-9 p_i, in the sum over
    p_i v_i and in the row sum alike, and the output is rounded once more:
    |error| <= 2^-9 (sum_i p_i |v_i| + 2 |out|), and 1e-5 for the fp32 arithmetic.  (A bound on the
    output's rms, as above, does not hold for the few rows that one key dominates.)"""
    q, k, v, reuse = _attn_case(seq + dh, batch, seq, heads, dh, "bf16", frac)
    idx, _, off = orc.selection(reuse)
    idx_full = np.full(batch * seq, 10 ** 6, dtype=np.int32)
    idx_full[:len(idx)] = idx
    out = torch.full((batch * seq, heads * dh), 5.0, dtype=torch.bfloat16, device="cuda")
    B.dare_k_attention(dev(q, "bf16"), dev(k, "bf16"), dev(v, "bf16"), out, batch, seq, heads, dh,
                       idx=dev(idx_full), sel_off=dev(off))
    torch.cuda.synchronize()
    got = host(out).astype(np.float64).reshape(batch, seq, heads, dh)
    assert np.all(got[reuse] == 5.0)
    for b in range(batch):
        rows = np.flatnonzero(~reuse[b])
        sl = slice(b * seq, (b + 1) * seq)
        Q, K, V = (a[sl].astype(np.float64).reshape(seq, heads, dh).transpose(1, 0, 2) for a in (q, k, v))
        z = Q[:, rows] @ K.transpose(0, 2, 1) / np.sqrt(dh)
        pr = np.exp(z - z.max(-1, keepdims=True))
        pr /= pr.sum(-1, keepdims=True)
        want = pr @ V
        bound = 2.0 ** -9 * (pr @ np.abs(V) + 2 * np.abs(want)) + 1e-5
        assert np.all(np.abs(got[b, rows].transpose(1, 0, 2) - want) <= bound)


@pytest.mark.parametrize("batch,seq,heads,dh,frac", [
    (1, 257, 4, 128, 0.01), (3, 300, 2, 64, 0.2), (2, 1000, 3, 128, 0.004),  # a few blocks with rows, the others read ahead
    (2, 515, 3, 64, 0.001),       # a sequence without a refreshed row
    (1, 1025, 32, 128, 0.2), (1, 513, 32, 64, 0.99),                        # as many blocks as CUs, nearly
    (20, 160, 5, 64, 0.6), (33, 300, 3, 128, 0.9),   # more pairs per XCD than take a turn, the last turn short
])
def test_attention_blocks_without_rows_read_ahead(B, batch, seq, heads, dh, frac):
    test_attention_block_layout_from_the_counts(B, batch, seq, heads, dh, frac)


@pytest.mark.parametrize("batch,heads", [(1, 2), (9, 32)])       # two key-waves per block, none
@pytest.mark.parametrize("seq", [1, 31, 32, 33, 63, 64, 65, 96, 97, 127, 128, 129, 160, 193, 257])
def test_attention_blocks_of_128_rows_at_tile_edges(B, batch, heads, seq):
    """Key counts around a subtile, a tile and a step; logits that grow along the keys, so that the reference
    exponent moves in the middle (and in the last, ragged tile).  Per element as above, but with the whole rounding
    error of bf16, whose 8 significant bits leave up to 2^-8 of a value just above a power of two: with one or two keys per
    row nothing averages it out.  |error| <= 2^-8 (sum_i p_i |v_i| + 2 |out|), and the fp32 arithmetic."""
    r = _rng(seq + heads)
    d = heads * 128
    q, k, v = (r.standard_normal((batch * seq, d)) for _ in range(3))
    k = (k.reshape(batch, seq, d) * (0.2 + 8.0 * np.arange(seq)[None, :, None] / seq)).reshape(-1, d)
    q, k, v = (store(a, "bf16") for a in (q, k, v))
    out = torch.zeros((batch * seq, d), dtype=torch.bfloat16, device="cuda")
    B.dare_k_attention(dev(q, "bf16"), dev(k, "bf16"), dev(v, "bf16"), out, batch, seq, heads, 128)
    torch.cuda.synchronize()
    got = host(out).astype(np.float64).reshape(batch, seq, heads, 128)
    for b in range(batch):
        Q, K, V = (a.reshape(batch, seq, heads, 128)[b].astype(np.float64).transpose(1, 0, 2) for a in (q, k, v))
        z = Q @ K.transpose(0, 2, 1) / np.sqrt(128)
        pr = np.exp(z - z.max(-1, keepdims=True))
        pr /= pr.sum(-1, keepdims=True)
        want = pr @ V
        # fp32 logits: 128 products each, off by up to 2^-24 of the sum of their magnitudes, a relative error of p
        fp32 = 2.0 ** -23 * (np.abs(Q) @ np.abs(K).transpose(0, 2, 1)).max(-1, keepdims=True) / np.sqrt(128)
        bound = (2.0 ** -8 + fp32) * (pr @ np.abs(V) + 2 * np.abs(want)) + 1e-5
        assert np.all(np.abs(got[b].transpose(1, 0, 2) - want) <= bound)


def _attention_of_rounded_probabilities(q, k, v, batch, seq, heads, refs):
    """float64, but probabilities rounded to bf16 relative to the maximum of a tile of 64 keys and the output rounded
    once: [sequence, head, row, channel].  refs: the tile whose maximum it is, per tile."""
    Q, K, V = (a.reshape(batch, seq, heads, 128).astype(np.float64).transpose(0, 2, 1, 3) for a in (q, k, v))
    z = Q @ K.transpose(0, 1, 3, 2) / np.sqrt(128)
    num, den = 0.0, 0.0
    for t in range(0, seq, 64):
        of = refs[t // 64] * 64
        top = z[..., of:of + 64].max(-1, keepdims=True)
        pr = synth.round_to_bf16(np.exp(z[..., t:t + 64] - top).astype(np.float32)).astype(np.float64) * np.exp(top)
        num, den = num + pr @ V[..., t:t + 64, :], den + pr.sum(-1, keepdims=True)
    return synth.round_to_bf16((num / den).astype(np.float32))


@pytest.mark.parametrize("batch,heads,refs", [
    (1, 8, (0, 1, 0)),      # two key-waves per block, each with the maximum of its first tile
    (130, 1, (0, 1, 1)),    # the same up to 128 keys; then none, and the reference moves to the second tile's maximum
    (9, 32, (0, 0, 0)),     # none; it does not
])
@pytest.mark.parametrize("seq", [32, 50, 64, 65, 100, 128, 129, 150, 192])
def test_attention_largest_probability_of_a_tile_is_not_rounded(B, batch, heads, refs, seq):
    """refs: the tile whose maximum is the reference exponent of each tile.  fp32 sums and exponentials, off by some 2^-22, give
    another bf16 value than float64 where the result is that close to the middle of two, 2^-8 apart: about one in 10^4
    for the output and for a probability, of which up to 192 are in each."""
    r = _rng(seq + heads)
    q, k, v = (store(a * r.standard_normal((batch * seq, heads * 128)), "bf16") for a in (1.13, 1.13, 1.0))
    out = torch.zeros((batch * seq, heads * 128), dtype=torch.bfloat16, device="cuda")
    B.dare_k_attention(dev(q, "bf16"), dev(k, "bf16"), dev(v, "bf16"), out, batch, seq, heads, 128)
    torch.cuda.synchronize()
    got = host(out).reshape(batch, seq, heads, 128).transpose(0, 2, 1, 3)
    assert np.mean(got != _attention_of_rounded_probabilities(q, k, v, batch, seq, heads, refs)) <= 0.02


def test_attention_reference_moves_by_its_own_rows_growth(B):
    """Logits that grow by 5 (even rows) and by 12 (odd rows) in base 2 from the first tile to the second: only the odd
    rows' reference exponents move, whatever their neighbours in the block do.  Bound as above."""
    batch, heads, seq = 9, 32, 128
    r = _rng(3)
    q, k, v = (0.6 * r.standard_normal((batch, seq, heads, 128)) for _ in range(3))
    q[..., 0] = np.where(np.arange(seq) % 2, 12.0, 5.0)[None, :, None]
    k[..., 0] = np.where(np.arange(seq) < 64, 0.0, np.sqrt(128) / np.log2(np.e))[None, :, None]
    q, k, v = (store(a.reshape(batch * seq, heads * 128), "bf16") for a in (q, k, v))
    out = torch.zeros((batch * seq, heads * 128), dtype=torch.bfloat16, device="cuda")
    B.dare_k_attention(dev(q, "bf16"), dev(k, "bf16"), dev(v, "bf16"), out, batch, seq, heads, 128)
    torch.cuda.synchronize()
    got = host(out).reshape(batch, seq, heads, 128).transpose(0, 2, 1, 3)
    for first, refs in ((0, (0, 0)), (1, (0, 1))):
        want = _attention_of_rounded_probabilities(q, k, v, batch, seq, heads, refs)
        assert np.mean(got[:, :, first::2] != want[:, :, first::2]) <= 0.02


def _one_dominant_key(B, batch, heads, seq, at, log2_logit):
    """Logits 0 but for key `at`, whose logit is log2_logit in base 2 for every second row (0 for the others); one-hot
    values.  The output of those rows is the value of that key, of the others the mean of all."""
    q = torch.zeros((batch * seq, heads, 128), dtype=torch.bfloat16, device="cuda")
    k, v = torch.zeros_like(q), torch.zeros_like(q)
    q[::2, :, 0] = 16.0
    k.view(batch, seq, heads, 128)[:, at, :, 0] = log2_logit / np.log2(np.e) * np.sqrt(128) / 16.0
    tok = torch.arange(seq, device="cuda")
    v.view(batch, seq, heads, 128)[:, tok, :, tok % 128] = 1.0
    out = torch.zeros_like(q)
    B.dare_k_attention(q, k, v, out, batch, seq, heads, 128)
    torch.cuda.synchronize()
    got = out.double().cpu().reshape(batch * seq, heads, 128)
    want = torch.zeros((128,), dtype=torch.float64)
    want[at % 128] = 1.0
    assert torch.equal(got[::2], want.expand_as(got[::2]))                # all of the weight: exact
    mean = torch.bincount(tok.cpu() % 128, minlength=128).double() / seq  # a probability of 1 each: rounded once
    assert bool(((got[1::2] - mean).abs() <= 2.0 ** -8 * mean).all())


@pytest.mark.parametrize("batch,heads", [(1, 2), (9, 32)])       # two key-waves per block, none
@pytest.mark.parametrize("seq", [32, 64, 150, 257])
def test_attention_one_key_far_above_the_others(B, batch, heads, seq):
    """A logit 250 above the reference exponent in base 2 (its probability overflows unless the reference moves), at
    every key of the first tile, where each lane holds four of 16, and of the last subtile."""
    for at in sorted(set(range(0, min(seq, 64), 3)) | set(range(max(0, seq - 33), seq, 4)) | {seq - 1}):
        _one_dominant_key(B, batch, heads, seq, at, 250.0)


@pytest.mark.parametrize("batch,heads", [(1, 2), (9, 32)])       # two key-waves per block, none
@pytest.mark.parametrize("seq,at", [(20, 7), (64, 40), (150, 100), (150, 149)])
def test_attention_rows_of_logits_near_the_lowest_finite(B, batch, heads, seq, at):
    """Every logit is -2^105, but -2^104 for one key (powers of two: times the scale exact to fp32's rounding): all of the
    weight is that key's."""
    q = torch.full((batch * seq, heads, 128), 0.0, dtype=torch.bfloat16, device="cuda")
    q[:, :, 3] = 2.0 ** 52
    k, v = torch.zeros_like(q), torch.randn(q.shape, device="cuda").to(torch.bfloat16)
    k[:, :, 3] = -2.0 ** 53
    k.view(batch, seq, heads, 128)[:, at, :, 3] = -2.0 ** 52
    out = torch.zeros_like(q)
    B.dare_k_attention(q, k, v, out, batch, seq, heads, 128)
    torch.cuda.synchronize()
    assert torch.equal(out.view(batch, seq, heads, 128), v.view(batch, seq, heads, 128)[:, at:at + 1].expand(batch, seq, heads, 128))


@pytest.mark.parametrize("batch,heads", [(1, 2), (9, 32)])       # two key-waves per block, none
@pytest.mark.parametrize("growth", [7.5, 11.5])                  # in base 2, over the keys of the first two tiles
def test_attention_of_values_near_the_largest(B, batch, heads, growth):
    """Values of 1e36 times a probability of more than 340 are not finite, their weighted mean is.  |error| as above:
    2^-8 for each of probability, row sum and output; fp32 logits of 10 and exponentials add less than 2^-18."""
    seq = 150
    q = torch.zeros((batch * seq, heads, 128), dtype=torch.bfloat16, device="cuda")
    q[:, :, 0] = 1.0
    k, v = torch.zeros_like(q), torch.zeros_like(q)
    k.view(batch, seq, heads, 128)[:, 130, :, 0] = growth / np.log2(np.e) * np.sqrt(128)
    v.view(batch, seq, heads, 128)[:, 130] = 1e36
    out = torch.zeros_like(q)
    B.dare_k_attention(q, k, v, out, batch, seq, heads, 128)
    torch.cuda.synchronize()
    weight = float(torch.exp(k.double().max() / np.sqrt(128)))
    want = float(v.double().max()) * weight / (weight + seq - 1)
    assert bool(((out.double() - want).abs() <= 3 * 2.0 ** -8 * want).all())


def test_attention_large_logits_are_stable(B):
    q, k, v, _ = _attn_case(77, 1, 192, 1, 128, "bf16", 1.0)
    q = store(q * 30.0, "bf16")
    out = torch.zeros((192, 128), dtype=torch.bfloat16, device="cuda")
    B.dare_k_attention(dev(q, "bf16"), dev(k, "bf16"), dev(v, "bf16"), out, 1, 192, 1, 128)
    torch.cuda.synchronize()
    got = host(out)
    assert np.all(np.isfinite(got))
    assert rel_err(got, orc.attention_rows(q, k, v, 1)) <= 2e-2


def test_copy_rows(B):
    r = _rng(4)
    src = r.standard_normal((100, 256)).astype(np.float32)
    dst = torch.zeros((100, 256), dtype=torch.float32, device="cuda")
    B.dare_k_copy_rows(dev(src), dst)
    torch.cuda.synchronize()
    assert np.array_equal(host(dst), src)
    dst.zero_()
    rows = np.array([3, 4, 50, 99], dtype=np.int32)
    idx = np.full(100, 10 ** 6, dtype=np.int32)
    idx[:4] = rows
    B.dare_k_copy_rows(dev(src), dst, idx=dev(idx), m_dev=torch.tensor([4], dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    want = np.zeros_like(src)
    want[rows] = src[rows]
    assert np.array_equal(host(dst), want)
