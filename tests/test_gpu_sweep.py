"""Seeded sweeps of random small shapes through the attention, Q-projection
and K/V-refresh entry points, each checked against the CPU oracle.

The shapes are drawn so that every launch plan gets exercised: per-head and
grouped-head attention (4 or 8 waves, idle waves, one or many key splits,
ragged key tiles and query groups; the ring kernel for long key ranges), and
the GEMM plans (small-M kernel, DMA kernel, row kernel, and the tile kernel's
64- to 256-row by 128- to 256-column tiles) with ragged row tiles and refresh
row counts.  Tolerances as in
test_gpu_parity: fp32 1e-4, bf16 2e-2 relative per (row, head); rows the
refresh does not touch byte-identical.
"""

import ctypes

import numpy as np
import pytest

from oracle import polestar_ref as ref
from paper_2607_14107_amd import inputs
from tests._util import RTOL, assert_rows_close, ensure_built, from_dev, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    ensure_built()
    from paper_2607_14107_amd import polestar
    return polestar


def _plan(P, m, N, K):
    """The bf16 product's kernel (0 small, 1 DMA, 2 tile, 3 rows), tile rows and columns, splits of K."""
    info = (ctypes.c_int * 4)()
    P.lib().ps_gemm_plan_info(1, ctypes.c_long(m), N, K, info)
    return tuple(info)


def _i32(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()


def _attend_case(i):
    g = np.random.default_rng(7000 + i)
    dtype = "bf16" if i % 3 else "fp32"
    hkv = int(g.choice([1, 2, 4]))
    group = int(g.choice([1, 2, 3, 4, 7, 8]))
    hd = int(g.choice([64, 128]))
    batch = int(g.integers(1, 4))
    nq = int(g.integers(1, 97))
    seq = int(g.integers(nq, 700))
    bs = int(g.integers(0, seq - nq + 1))
    return dtype, batch, seq, bs, nq, hkv * group, hkv, hd


@pytest.mark.parametrize("case", range(24))
def test_attend_random_shapes(P, case):
    dtype, batch, seq, bs, nq, H, Hkv, hd = _attend_case(case)
    g = np.random.default_rng(9000 + case)
    q = inputs.store(g.standard_normal((batch, nq, H, hd), dtype=np.float32), dtype)
    kc = inputs.store(g.standard_normal((batch, seq, Hkv, hd), dtype=np.float32), dtype)
    vc = inputs.store(g.standard_normal((batch, seq, Hkv, hd), dtype=np.float32), dtype)
    torch = pytest.importorskip("torch")
    lse = torch.empty((batch, H, nq), dtype=torch.float32, device="cuda")
    out, _ = P.attend(None, None, to_dev(kc, dtype), to_dev(vc, dtype), bs, nq, H,
                      q_buf=to_dev(q, dtype), lse=lse)
    o_want, lse_want = ref.attend(ref.decode(q, dtype), ref.decode(kc, dtype), ref.decode(vc, dtype))
    shape = f"{dtype} b{batch} seq{seq} nq{nq} H{H}/{Hkv} hd{hd}"
    assert_rows_close(ref.decode(from_dev(out), dtype), o_want, RTOL[dtype], "output " + shape)
    np.testing.assert_allclose(from_dev(lse), lse_want, rtol=RTOL[dtype], atol=RTOL[dtype], err_msg=shape)


@pytest.mark.parametrize("batch,seq,nq,H,Hkv,hd", [
    (4, 2100, 32, 16, 16, 64),     # 66 key tiles (the last ragged) in 4 splits of 17: head_dim 64
    (4, 1600, 20, 24, 12, 128),    # two query heads per KV head, 20 queries, 2 splits of 25 tiles
    (1, 4200, 32, 64, 64, 128),    # 132 key tiles in 4 splits of 33: long walks per wave
])
def test_attend_ring_kernel_shapes(P, batch, seq, nq, H, Hkv, hd):
    """bf16 shapes whose plan takes the ring kernel (one workgroup per CU,
    at least four key tiles per wave), against the oracle."""
    dtype = "bf16"
    g = np.random.default_rng(seq + nq + H)
    bs = seq // 3
    q = inputs.store(g.standard_normal((batch, nq, H, hd), dtype=np.float32), dtype)
    kc = inputs.store(g.standard_normal((batch, seq, Hkv, hd), dtype=np.float32), dtype)
    vc = inputs.store(g.standard_normal((batch, seq, Hkv, hd), dtype=np.float32), dtype)
    torch = pytest.importorskip("torch")
    lse = torch.empty((batch, H, nq), dtype=torch.float32, device="cuda")
    out, _ = P.attend(None, None, to_dev(kc, dtype), to_dev(vc, dtype), bs, nq, H,
                      q_buf=to_dev(q, dtype), lse=lse)
    o_want, lse_want = ref.attend(ref.decode(q, dtype), ref.decode(kc, dtype), ref.decode(vc, dtype))
    shape = f"b{batch} seq{seq} nq{nq} H{H}/{Hkv} hd{hd}"
    assert_rows_close(ref.decode(from_dev(out), dtype), o_want, RTOL[dtype], "output " + shape)
    np.testing.assert_allclose(from_dev(lse), lse_want, rtol=RTOL[dtype], atol=RTOL[dtype], err_msg=shape)


def _gemm_dims(g, dtype):
    # d: K split into 8..16 stages per split for the DMA kernel at several of these
    d = int(g.choice([128, 256, 640, 1280, 1536, 1792, 2048])) if dtype == "bf16" else int(g.choice([128, 256, 512]))
    hd = int(g.choice([64, 128]))
    return d, hd


@pytest.mark.parametrize("case", range(18))
def test_linear_random_tile_shapes(P, case):
    """Row counts and widths where the tile kernel's plans compete (64- to
    256-row by 128-column tiles, unsplit; the last six few rows of a long K,
    which plans split), ragged in both directions, bf16."""
    torch = pytest.importorskip("torch")
    g = np.random.default_rng(17000 + case)
    batch = int(g.integers(1, 4))
    n = int(g.integers(200, 1600)) // batch
    rs = int(g.integers(0, 40))
    seq = n + rs + int(g.integers(0, 30))
    K = int(g.choice([1024, 2048, 3072, 4096]))
    N = 16 * int(g.integers(16, 376))                      # 256 .. 6000 columns
    if case >= 12:
        n = int(g.integers(66, 300)) // batch
        seq = n + rs + int(g.integers(0, 30))
        K = 128 * int(g.integers(20, 64))
        N = 16 * int(g.integers(4, 120))                   # 64 .. 1900 columns
    kernel, _, _, splits = _plan(P, batch * n, N, K)
    assert kernel == 2 and (splits > 1) == (case >= 12)
    x = inputs.store(g.standard_normal((batch, seq, K)).astype(np.float32), "bf16")
    w = inputs.store((g.standard_normal((N, K)) * 0.05).astype(np.float32), "bf16")
    y = torch.empty((batch, n, N), dtype=torch.bfloat16, device="cuda")
    P.linear(to_dev(x, "bf16"), rs, n, to_dev(w, "bf16"), y)
    want = ref.decode(x, "bf16")[:, rs:rs + n] @ ref.decode(w, "bf16").T
    assert_rows_close(ref.decode(from_dev(y), "bf16"), want, RTOL["bf16"],
                      f"linear {batch}x{n} rows x {N} x K {K}")


@pytest.mark.parametrize("m,N,K,rows,cols,splits", [
    # each tile shape (rows x columns) of the tile kernel, unsplit and split where plans take both, K tiles
    # per split whole and not whole multiples of its LDS slots, ragged last tiles in both directions
    (66, 80, 256, 64, 128, 1), (70, 64, 384, 64, 128, 1), (257, 4288, 3200, 64, 128, 1),
    (98, 64, 1536, 64, 128, 3), (71, 96, 1664, 64, 128, 4), (69, 64, 4352, 64, 128, 7),
    (385, 4656, 256, 128, 128, 1), (262, 6544, 384, 128, 128, 1),
    (68, 4288, 2048, 64, 128, 3), (66, 2432, 3968, 64, 128, 6), (66, 4448, 2816, 128, 128, 6), (2713, 64, 3968, 128, 128, 8),
    (771, 6624, 256, 128, 192, 1), (775, 6576, 512, 128, 192, 1), (74, 6768, 5376, 128, 192, 7),
    (71, 8352, 3200, 128, 192, 5),
    (1055, 6576, 384, 128, 256, 1), (1032, 6672, 512, 128, 256, 1), (69, 12400, 5120, 128, 256, 5),
    (523, 6624, 384, 192, 128, 1), (527, 6624, 256, 192, 128, 1), (133, 5456, 3328, 192, 128, 5),
    (130, 4112, 3584, 192, 128, 7),
    (1031, 7232, 384, 192, 192, 1), (1032, 7312, 256, 192, 192, 1), (142, 11408, 4096, 192, 192, 4),
    (1156, 6976, 256, 192, 256, 1), (2305, 7696, 384, 192, 256, 1), (259, 6288, 11520, 192, 256, 5),
    (772, 7104, 384, 256, 128, 1), (774, 6928, 256, 256, 128, 1), (195, 8240, 4096, 256, 128, 3),
    (2048, 6144, 1024, 256, 192, 1), (1737, 6608, 128, 256, 192, 1), (195, 10992, 11648, 256, 192, 4),
    (1537, 8192, 512, 256, 256, 1), (1546, 7344, 128, 256, 256, 1), (405, 4112, 11648, 256, 256, 7),
])
def test_linear_tile_kernel_edges(P, m, N, K, rows, cols, splits):
    """The tile kernel's shapes at their edges against an fp32 product of the
    same bf16 operands: both sum exact products in fp32 in some order and
    round once, so a row's largest difference is one bf16 step (2^-8) of the
    row's largest value plus fp32 noise, well under the 2e-2 of the sweep.  The
    plan is named, so that a change of the plan's rule cannot move a case to
    another kernel unseen."""
    assert _plan(P, m, N, K) == (2, rows, cols, splits)
    torch = pytest.importorskip("torch")
    gen = torch.Generator(device="cuda").manual_seed(m * 7 + N)
    x = torch.randn((1, m + 3, K), generator=gen, device="cuda").to(torch.bfloat16)
    w = (torch.randn((N, K), generator=gen, device="cuda") * 0.05).to(torch.bfloat16)
    y = torch.full((1, m, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    P.linear(x, 2, m, w, y)
    want = x[0, 2:2 + m].float() @ w.float().t()
    err = (y[0].float() - want).abs().amax(1) / want.abs().amax(1)
    assert float(err.max()) <= 5e-3, (m, N, K, float(err.max()))


@pytest.mark.parametrize("case", range(16))
def test_project_q_random_shapes(P, case):
    g = np.random.default_rng(11000 + case)
    dtype = "bf16" if case % 4 else "fp32"
    d, hd = _gemm_dims(g, dtype)
    H = int(g.integers(1, 9))
    batch = int(g.integers(1, 6))
    bl = int(g.integers(1, 70))
    seq = int(g.integers(bl, bl + 60))
    bs = int(g.integers(0, seq - bl + 1))
    h = inputs.store(g.standard_normal((batch, seq, d), dtype=np.float32), dtype)
    wq = inputs.store(0.05 * g.standard_normal((H * hd, d), dtype=np.float32), dtype)
    q = P.project_q(to_dev(h, dtype), to_dev(wq, dtype), bs, bl, H)
    want = ref.q_project(ref.decode(h, dtype), ref.decode(wq, dtype), bs, bl, H, hd)
    assert_rows_close(ref.decode(from_dev(q), dtype), want, RTOL[dtype],
                      f"Q {dtype} b{batch} rows {batch * bl} d{d} H{H} hd{hd}")


@pytest.mark.parametrize("case", range(16))
def test_refresh_random_shapes(P, case):
    g = np.random.default_rng(13000 + case)
    dtype = "bf16" if case % 4 else "fp32"
    d, hd = _gemm_dims(g, dtype)
    kvh = int(g.integers(1, 5))
    batch = int(g.integers(1, 4))
    seq = int(g.integers(40, 400))
    bl = int(g.integers(1, 40))
    bs = int(g.integers(0, seq - bl + 1))
    k_max = int(g.integers(0, min(seq, 120)))
    if case == 5:
        batch, bl, k_max = 1, 8, 6                         # at most 16 rows: the small-M kernel
        bs = min(bs, seq - bl)
    cached = np.setdiff1d(np.arange(seq), np.arange(bs, bs + bl))
    idx = np.full((batch, max(k_max, 1)), -1, dtype=np.int32)
    cnt = np.zeros(batch, dtype=np.int32)
    for b in range(batch):
        c = int(g.integers(0, min(k_max, cached.size) + 1))
        idx[b, :c] = np.sort(g.choice(cached, size=c, replace=False))
        cnt[b] = c
    h = inputs.store(g.standard_normal((batch, seq, d), dtype=np.float32), dtype)
    wk = inputs.store(0.05 * g.standard_normal((kvh * hd, d), dtype=np.float32), dtype)
    wv = inputs.store(0.05 * g.standard_normal((kvh * hd, d), dtype=np.float32), dtype)
    kc0 = inputs.store(g.standard_normal((batch, seq, kvh, hd), dtype=np.float32), dtype)
    vc0 = inputs.store(g.standard_normal((batch, seq, kvh, hd), dtype=np.float32), dtype)
    kc, vc = to_dev(kc0, dtype), to_dev(vc0, dtype)
    if k_max > 0:
        P.refresh_kv(to_dev(h, dtype), _i32(idx[:, :k_max]), _i32(cnt), bs, bl,
                     to_dev(wk, dtype), to_dev(wv, dtype), kc, vc)
    else:
        P.refresh_kv(to_dev(h, dtype), None, None, bs, bl, to_dev(wk, dtype), to_dev(wv, dtype), kc, vc)
    kg, vg = from_dev(kc), from_dev(vc)
    hdec, wkd, wvd = ref.decode(h, dtype), ref.decode(wk, dtype), ref.decode(wv, dtype)
    shape = f"{dtype} b{batch} seq{seq} k_max{k_max} bl{bl} d{d} kv{kvh}x{hd}"
    for b in range(batch):
        rows = np.asarray(sorted(set(idx[b, :cnt[b]].tolist()) | set(range(bs, bs + bl))), dtype=np.int64)
        keep = np.setdiff1d(np.arange(seq), rows)
        assert np.array_equal(kg[b, keep], kc0[b, keep]) and np.array_equal(vg[b, keep], vc0[b, keep]), \
            "untouched rows changed " + shape
        kw = ref.project_rows(hdec[b], wkd, rows).reshape(rows.size, kvh, hd)
        vw = ref.project_rows(hdec[b], wvd, rows).reshape(rows.size, kvh, hd)
        assert_rows_close(ref.decode(kg[b, rows], dtype), kw, RTOL[dtype], f"K rows b{b} " + shape)
        assert_rows_close(ref.decode(vg[b, rows], dtype), vw, RTOL[dtype], f"V rows b{b} " + shape)


@pytest.mark.parametrize("batch,seq,bs,bl,d,kvh,hd,k_max", [
    (2, 700, 600, 32, 3584, 4, 128, 603),   # 1270 rows x 1024 columns: eight 159-row DMA tiles, four K splits
    (1, 800, 400, 20, 640, 4, 128, 680),    # 700 rows x 1024 columns: five DMA tiles, K unsplit (5 steps)
])
def test_refresh_narrow_output_many_row_tiles(P, batch, seq, bs, bl, d, kvh, hd, k_max):
    """Outputs of at most 1024 columns keep the DMA kernel up to eight row
    tiles; every stale slot is filled, every refreshed row compared."""
    g = np.random.default_rng(d + k_max)
    dtype = "bf16"
    cached = np.setdiff1d(np.arange(seq), np.arange(bs, bs + bl))
    idx = np.stack([np.sort(g.choice(cached, size=k_max, replace=False)) for _ in range(batch)]).astype(np.int32)
    cnt = np.full(batch, k_max, dtype=np.int32)
    h = inputs.store(g.standard_normal((batch, seq, d), dtype=np.float32), dtype)
    wk = inputs.store(0.05 * g.standard_normal((kvh * hd, d), dtype=np.float32), dtype)
    wv = inputs.store(0.05 * g.standard_normal((kvh * hd, d), dtype=np.float32), dtype)
    kc0 = inputs.store(g.standard_normal((batch, seq, kvh, hd), dtype=np.float32), dtype)
    vc0 = inputs.store(g.standard_normal((batch, seq, kvh, hd), dtype=np.float32), dtype)
    kc, vc = to_dev(kc0, dtype), to_dev(vc0, dtype)
    P.refresh_kv(to_dev(h, dtype), _i32(idx), _i32(cnt), bs, bl, to_dev(wk, dtype), to_dev(wv, dtype), kc, vc)
    kg, vg = from_dev(kc), from_dev(vc)
    hdec, wkd, wvd = ref.decode(h, dtype), ref.decode(wk, dtype), ref.decode(wv, dtype)
    for b in range(batch):
        rows = np.asarray(sorted(set(idx[b].tolist()) | set(range(bs, bs + bl))), dtype=np.int64)
        keep = np.setdiff1d(np.arange(seq), rows)
        assert np.array_equal(kg[b, keep], kc0[b, keep]) and np.array_equal(vg[b, keep], vc0[b, keep])
        kw = ref.project_rows(hdec[b], wkd, rows).reshape(rows.size, kvh, hd)
        vw = ref.project_rows(hdec[b], wvd, rows).reshape(rows.size, kvh, hd)
        assert_rows_close(ref.decode(kg[b, rows], dtype), kw, RTOL[dtype], f"K rows b{b}")
        assert_rows_close(ref.decode(vg[b, rows], dtype), vw, RTOL[dtype], f"V rows b{b}")


@pytest.mark.parametrize("batch,k_max,counts", [
    (3, 500, "half"), (3, 500, "exactly half"), (3, 500, "one more"), (3, 500, "full"), (3, 500, "none"),
    (16, 96, "half"), (16, 96, "uneven"),
])
def test_refresh_packed_lists(P, batch, k_max, counts):
    """Lists without a block that are not full: their used rows are packed and
    run in the smaller of the plan's two tile shapes when they are few enough,
    in the other one when not.  Entries outside the sequence are skipped, rows
    no entry names stay byte-identical, the rest are within a bf16 step of an
    fp32 product."""
    g = np.random.default_rng(batch + k_max)
    half = (batch * k_max + 1) // 2
    cnt = np.zeros(batch, dtype=np.int64)
    if counts == "half":
        cnt[:] = int(0.45 * k_max)
    elif counts == "full":
        cnt[:] = k_max
    elif counts == "uneven":
        cnt[:] = g.integers(0, k_max, size=batch)
        cnt[3], cnt[7] = 0, k_max
    elif counts != "none":
        left = half + (counts == "one more")
        for b in range(batch):
            cnt[b] = min(k_max, left)
            left -= cnt[b]
    _check_packed(P, g, batch, k_max, cnt, 512, 32, 128)


def _check_packed(P, g, batch, k_max, cnt, d, kvh, hd):
    torch = pytest.importorskip("torch")
    seq = k_max + 37
    idx = np.stack([g.permutation(seq)[:k_max] for _ in range(batch)]).astype(np.int32)
    idx[0, 5], idx[batch // 2, 0], idx[batch - 1, 7] = -1, seq, -7
    gen = torch.Generator(device="cuda").manual_seed(k_max)
    rnd = lambda *sh: torch.randn(sh, generator=gen, device="cuda").to(torch.bfloat16)  # noqa: E731
    h, wk, wv = rnd(batch, seq, d), rnd(kvh * hd, d) * 0.05, rnd(kvh * hd, d) * 0.05
    kc0, vc0 = rnd(batch, seq, kvh, hd), rnd(batch, seq, kvh, hd)
    kc, vc = kc0.clone(), vc0.clone()
    P.refresh_kv(h, _i32(idx), _i32(cnt), 0, 0, wk, wv, kc, vc)
    for b in range(batch):
        rows = [int(p) for p in idx[b, :cnt[b]] if 0 <= p < seq]
        keep = torch.ones(seq, dtype=torch.bool, device="cuda")
        keep[rows] = False
        for got, was, w in ((kc, kc0, wk), (vc, vc0, wv)):
            assert torch.equal(got[b][keep], was[b][keep]), b
            if rows:
                want = h[b, rows].float() @ w.float().t()
                err = (got[b, rows].reshape(len(rows), -1).float() - want).abs().amax(1) / want.abs().amax(1)
                assert float(err.max()) <= 5e-3, (b, float(err.max()))


@pytest.mark.parametrize("batch,k_max,d,kvh,pair", [
    (3, 259, 256, 39, (192, 256, 192, 128)), (10, 365, 896, 39, (256, 128, 192, 128)),
    (2, 322, 512, 33, (256, 128, 128, 128)), (2, 200, 1408, 33, (192, 128, 128, 128)),
    (8, 459, 896, 26, (128, 256, 128, 128)), (70, 11, 512, 30, (256, 128, 128, 128)),
])
@pytest.mark.parametrize("where", ["line", "past it", "full"])
def test_refresh_packed_shapes(P, batch, k_max, d, kvh, pair, where):
    """Every pair of tile shapes that packed lists run in, at the number of rows
    that is the last one for the smaller shape, one row more, and full lists;
    more sequences than a wave has lanes."""
    info = (ctypes.c_int * 5)()
    assert P.lib().ps_packed_plan_info(ctypes.c_long(batch * k_max), 2 * kvh * 128, d, info)
    assert tuple(info)[:4] == pair
    line = min(info[4], batch * k_max - 1)
    left = {"line": line, "past it": line + 1, "full": batch * k_max}[where]
    g = np.random.default_rng(batch * k_max)
    cnt = np.zeros(batch, dtype=np.int64)
    while left > 0:                                        # uneven lists
        b = int(g.integers(0, batch))
        more = min(left, int(g.integers(1, 30)), k_max - int(cnt[b]))
        cnt[b] += more
        left -= more
    _check_packed(P, g, batch, k_max, cnt, d, kvh, 128)


@pytest.mark.parametrize("batch,n,d,ffn", [
    (16, 32, 1024, 3072), (1, 300, 512, 1040), (3, 111, 3584, 4736), (2, 700, 384, 2064), (1, 1500, 256, 4096),
    (4, 8, 512, 768), (1, 2400, 512, 3088),
])
def test_linear_swiglu_against_its_calls(P, batch, n, d, ffn):
    """One launch (unsplit plans of the tile kernel) or the two calls: either
    way within a bf16 step (2^-8, and one for the gate's and up's own rounding
    landing apart) of silu(gate) * up on the rounded fp32 products."""
    torch = pytest.importorskip("torch")
    gen = torch.Generator(device="cuda").manual_seed(n + ffn)
    x = torch.randn((batch, n + 5, d), generator=gen, device="cuda").to(torch.bfloat16)
    w = (torch.randn((2 * ffn, d), generator=gen, device="cuda") * 2 / d ** 0.5).to(torch.bfloat16)
    gu = torch.empty((batch, n, 2 * ffn), dtype=torch.bfloat16, device="cuda")
    a = torch.full((batch, n, ffn), float("nan"), dtype=torch.bfloat16, device="cuda")
    P.linear_swiglu(x, 3, n, w, gu, a)
    p = (x[:, 3:3 + n].reshape(-1, d).float() @ w.float().t()).to(torch.bfloat16).float()
    want = (p[:, :ffn] * torch.sigmoid(p[:, :ffn]) * p[:, ffn:]).view(batch, n, ffn)
    err = (a.float() - want).abs().amax(2) / want.abs().amax(2)
    assert float(err.max()) <= 2 * 2 ** -8, (batch, n, d, ffn, float(err.max()))


@pytest.mark.parametrize("n,d,ffn,tile", [
    (65, 128, 144, (128, 128)), (529, 128, 3280, (192, 128)), (771, 128, 3280, (256, 128)),
    (1044, 128, 3280, (128, 256)), (1041, 128, 3600, (192, 256)), (1546, 128, 3616, (256, 256)),
    (65, 2688, 8368, (128, 128)),   # unsplit, where the plain product's plan splits K
    (529, 128, 3288, None),    # 2 ffn no multiple of 32: two calls
    (200, 1536, 384, None),    # no tile kernel: two calls
])
def test_linear_swiglu_has_its_calls_values(P, n, d, ffn, tile):
    """Every tile shape of the one-launch form (and the calls that take two)
    has the values of polestar_linear and polestar_swiglu, bit for bit, over
    gates that a shorter formula would treat differently: to +-120 in steps of a
    quarter (the quotient's denominator passes 2^126 at -87.4 and overflows at
    -88.7), zero, the largest finite values, and rows whose products are
    infinite or NaN."""
    info = (ctypes.c_int * 4)()
    one_launch = P.lib().ps_swiglu_plan_info(ctypes.c_long(n), 2 * ffn, d, info)
    assert (tuple(info)[1:3] if one_launch else None) == tile
    torch = pytest.importorskip("torch")
    x = torch.zeros((1, n, d), device="cuda")
    x[0, :, 0] = torch.tensor([1.0, -1.0, 0.5, 4.0, 0.0, float("inf"), float("nan")], device="cuda")[
        torch.arange(n, device="cuda") % 7]
    w = torch.zeros((2 * ffn, d), device="cuda")
    f = torch.arange(ffn, device="cuda")
    w[:ffn, 0] = (f % 960 - 480) / 4.0
    w[:ffn:97, 0], w[5:ffn:97, 0] = 3e38, -3e38
    w[ffn:, 0] = torch.where(f % 2 == 0, 1.0, -3.0) * 2.0 ** (f % 5)
    x, w = x.to(torch.bfloat16), w.to(torch.bfloat16)
    gu = torch.empty((1, n, 2 * ffn), dtype=torch.bfloat16, device="cuda")
    one, two = torch.empty((1, n, ffn), dtype=torch.bfloat16, device="cuda"), torch.empty(
        (1, n, ffn), dtype=torch.bfloat16, device="cuda")
    P.linear_swiglu(x, 0, n, w, gu, one)
    P.linear(x, 0, n, w, gu)
    P.swiglu(gu, two)
    a, b = one.view(torch.int16), two.view(torch.int16)
    assert torch.equal(a, b), (n, d, ffn, int((a != b).sum()))


@pytest.mark.parametrize("m,N,K,kernel", [
    (9, 256, 256, (0, 0, 0, 1)), (40, 4096, 4096, (1, 0, 0, 8)),
    (529, 6560, 128, (2, 192, 128, 1)), (1546, 7232, 128, (2, 256, 256, 1)), (68, 4288, 2048, (2, 64, 128, 3)),
])
def test_linear_nan_bits(P, m, N, K, kernel):
    """A NaN output is the quiet NaN 0x7fc0 from every kernel, whatever the
    sign and payload of the operands', and reaches its own row only."""
    torch = pytest.importorskip("torch")
    assert _plan(P, m, N, K) == kernel
    gen = torch.Generator(device="cuda").manual_seed(m)
    x = torch.randn((1, m, K), generator=gen, device="cuda").to(torch.bfloat16)
    w = torch.randn((N, K), generator=gen, device="cuda").to(torch.bfloat16)
    clean = P.linear(x, 0, m, w, torch.empty((1, m, N), dtype=torch.bfloat16, device="cuda"))
    rows = list(range(3, m, 5))
    x.view(torch.int16)[0, rows, K // 3] = -63          # 0xffc1
    y = P.linear(x, 0, m, w, torch.empty((1, m, N), dtype=torch.bfloat16, device="cuda"))
    want = clean.view(torch.int16).clone()
    want[0, rows] = 0x7fc0
    assert torch.equal(y.view(torch.int16), want)


@pytest.mark.parametrize("dtype,batch,n,d,H,kv,hd,kernel,splits", [
    ("bf16", 16, 32, 512, 8, 8, 64, 2, 1), ("bf16", 1, 32, 1024, 8, 2, 128, 0, 1), ("bf16", 3, 50, 512, 4, 4, 128, 2, 1),
    ("bf16", 2, 400, 256, 16, 4, 64, 2, 1), ("bf16", 1, 9, 256, 4, 1, 64, 0, 1), ("fp32", 2, 60, 128, 4, 2, 64, 3, 2),
    ("bf16", 2, 20, 4096, 32, 16, 64, 1, 8), ("bf16", 6, 32, 1536, 8, 8, 64, 1, 3), ("bf16", 2, 50, 2048, 4, 2, 64, 2, 4),
    ("bf16", 5, 28, 4096, 32, 16, 128, 1, 4),
])
def test_project_qkv_against_its_calls(P, dtype, batch, n, d, H, kv, hd, kernel, splits):
    """Each kernel that a product of three weight matrices runs on (0 small, 1
    DMA with one and two row tiles, 2 tile, 3 rows), unsplit and split."""
    torch = pytest.importorskip("torch")
    info = (ctypes.c_int * 4)()
    P.lib().ps_gemm_plan_info(int(dtype == "bf16"), ctypes.c_long(batch * n), (H + 2 * kv) * hd, d, info)
    assert (info[0], info[3]) == (kernel, splits)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(n + d)
    rnd = lambda *sh: torch.randn(sh, generator=gen, device="cuda").to(td)  # noqa: E731
    seq, lo = n + 20, 7
    h = rnd(batch, seq, d)
    wq, wk, wv = rnd(H * hd, d) * 0.05, rnd(kv * hd, d) * 0.05, rnd(kv * hd, d) * 0.05
    k0, v0 = rnd(batch, seq, kv, hd), rnd(batch, seq, kv, hd)
    k, v, q = k0.clone(), v0.clone(), torch.full((batch, n, H, hd), float("nan"), dtype=td, device="cuda")
    P.project_qkv(h, lo, n, wq, wk, wv, q, k, v)
    rows = h[:, lo:lo + n].double()
    tol = 5e-3 if dtype == "bf16" else 1e-5            # one rounding to bf16 / fp32 sums
    for got, w in ((q, wq), (k[:, lo:lo + n], wk), (v[:, lo:lo + n], wv)):
        want = rows @ w.double().t()
        err = (got.reshape(batch, n, -1).double() - want).abs().amax(2) / want.abs().amax(2)
        assert float(err.max()) <= tol, (dtype, n, float(err.max()))
    for got, was in ((k, k0), (v, v0)):
        assert torch.equal(got[:, :lo], was[:, :lo]) and torch.equal(got[:, lo + n:], was[:, lo + n:])


@pytest.mark.parametrize("dtype,d", [("bf16", 4096), ("bf16", 260), ("fp32", 1028), ("fp32", 9000)])
def test_residual_rmsnorm_is_its_two_calls(P, dtype, d):
    torch = pytest.importorskip("torch")
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(d)
    x = torch.randn((3, 37, d), generator=gen, device="cuda")
    t = torch.randn((3, 37, d), generator=gen, device="cuda").to(td)
    x2, out = x.clone(), torch.zeros((3, 50, d), dtype=td, device="cuda")
    out2 = out.clone()
    P.residual_add(x, t)
    P.rmsnorm(x, 0, 37, out, 11)
    P.residual_rmsnorm(x2, t, out2, 11)
    assert torch.equal(x, x2) and torch.equal(out, out2)
