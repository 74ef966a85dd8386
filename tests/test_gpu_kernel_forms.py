"""Two kernel forms of the same step against each other, at the sizes where a form's
own indexing can go wrong.  The forms do the same arithmetic in fp32 from the same
bf16 products, so they differ by the rounding of bf16 probabilities and outputs."""

import numpy as np
import pytest

from _helpers import ensure_built, host64, max_abs_rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ensure_built()
    return torch.device("cuda:0")


def _lists(rng, rows, nC, k, holes):
    """Random retrieval lists of `rows` x nC landmark rows (row t among chunks < t), with
    pads in the middle, rows that are all pads and an out-of-range index when `holes`."""
    idx = np.full((rows, nC, k), -1, np.int32)
    sel = np.full((rows, nC, k), -np.inf, np.float32)
    for r in range(rows):
        for t in range(1, nC):
            n = min(t, k)
            js = np.sort(rng.choice(t, size=n, replace=False))
            if holes and t % 5 == 0:
                js[rng.integers(n)] = -1
            if holes and t % 7 == 0:
                js[:] = -1
            idx[r, t, :n] = js
            sel[r, t, :n] = np.where(js >= 0, rng.standard_normal(n), -np.inf)
    if holes and nC > 9:
        idx[0, 9, 0] = nC + 3
    return idx, sel


@pytest.mark.parametrize("B,H,Hr,nC,k,holes,obo", [
    (1, 1, 1, 1, 3, False, False),        # one chunk, nothing retrieved
    (1, 2, 1, 11, 1, True, False),        # one slot per chunk: a chunk switch every tile
    (2, 3, 3, 13, 5, True, True),
    (1, 3, 1, 700, 8, True, False),       # more items than resident streams
    (1, 1, 1, 2100, 8, False, False),     # window order
])
def test_forward_wave_form_equals_pair_form(dev, B, H, Hr, nC, k, holes, obo):
    """bf16 lists of up to 8 run on one wave per chunk; the same lists padded to 9 slots
    run on a pair of waves per chunk."""
    import torch
    from paper_2410_01651_amd import gca
    rng = np.random.default_rng(nC + k)
    idx, sel = _lists(rng, B * Hr, nC, k, holes)
    g = torch.Generator(device=dev).manual_seed(nC)
    q, kk, v = (torch.randn(B, H, nC * 64, 64, generator=g, device=dev, dtype=torch.bfloat16) for _ in range(3))
    got = []
    for K in (k, 9):
        p = gca.problem(B, H, nC, K, Hr=Hr, D=64, off_by_one=obo)
        i = np.full((B, Hr, nC, K), -1, np.int32)
        s = np.full((B, Hr, nC, K), -np.inf, np.float32)
        i[..., :k] = idx.reshape(B, Hr, nC, k)
        s[..., :k] = sel.reshape(B, Hr, nC, k)
        out, lse, w = gca.grouped_xattn_fwd(p, q, kk, v, torch.from_numpy(i).to(dev), torch.from_numpy(s).to(dev))
        got.append((host64(out), host64(lse)[..., :k], host64(w)[..., :k]))
    (o0, l0, w0), (o1, l1, w1) = got
    assert max_abs_rel(o0, o1) <= 2.0 ** -7    # two bf16 roundings of sums that differ in bf16 probabilities
    assert max_abs_rel(l0, l1) <= 1e-6
    assert max_abs_rel(w0, w1) <= 1e-6


@pytest.mark.parametrize("B,H,nC,first_empty", [
    (1, 1000, 3, 3),      # streams that end with a sequence's chunks 0 and 1
    (1, 3, 1400, 500),    # lists that are all pads from a row on: streams with empty chunks at their end
    (2, 1, 1500, 2),      # one chunk that retrieves anything per sequence
    (1, 1, 2300, 900),    # the same in window order
])
def test_forward_streams_ending_in_empty_chunks(dev, B, H, nC, first_empty):
    """A persistent stream whose last chunks retrieve nothing: their zeros are written, and the
    last chunk before them is as on the pair form."""
    import torch
    from paper_2410_01651_amd import gca
    k = 4
    rng = np.random.default_rng(nC)
    idx = np.full((B, 1, nC, 9), -1, np.int32)
    sel = np.full((B, 1, nC, 9), -np.inf, np.float32)
    for t in range(1, min(first_empty, nC)):
        n = min(t, k)
        idx[:, 0, t, :n] = np.sort(rng.choice(t, size=n, replace=False))
        sel[:, 0, t, :n] = rng.standard_normal((B, n))
    g = torch.Generator(device=dev).manual_seed(nC)
    q, kk, v = (torch.randn(B, H, nC * 64, 64, generator=g, device=dev, dtype=torch.bfloat16) for _ in range(3))
    got = []
    for K in (k, 9):
        i, s = (torch.from_numpy(np.ascontiguousarray(x[..., :K])).to(dev) for x in (idx, sel))
        out, lse, w = gca.grouped_xattn_fwd(gca.problem(B, H, nC, K, D=64), q, kk, v, i, s)
        got.append((host64(out), host64(lse)[..., :k], host64(w)[..., :k]))
    for a, b, tol in zip(*got, (2.0 ** -7, 1e-6, 1e-6)):   # as above
        assert max_abs_rel(a, b) <= tol
    empty = got[0][0].reshape(B, H, nC, 64 * 64)[:, :, min(first_empty, nC) + 1:]
    assert not empty.any()


@pytest.mark.parametrize("dtype,D,nC,k,gumbel", [
    ("bf16", 576, 1, 3, False),
    ("bf16", 1024, 129, 8, False),       # few chunks: one pass with and without room for the lists
    ("bf16", 640, 1100, 16, True),
    ("bf16", 576, 9100, 5, False),       # several parts per class
    ("fp32", 320, 700, 8, True),
    ("bf16", 1024, 257, 8, False),       # a third row block of one row and a ragged third key tile
    ("bf16", 576, 255, 8, False),        # the most chunks of few rows that stay with the one-pass form
])
def test_wide_select_equals_score_matrix(dev, dtype, D, nC, k, gumbel):
    """Selection without the matrix for landmarks too wide for registers (its lists in the
    output buffer), against the same selection from the score matrix and, with the output
    in the query buffer, against the one-pass form that needs no scratch."""
    import torch
    from paper_2410_01651_amd import gca
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device=dev).manual_seed(D + nC)
    lq, lk = (torch.randn(1, 2, nC, D, generator=g, device=dev, dtype=dt) for _ in range(2))
    q, kk, v = (torch.randn(1, 2, nC * 64, 64, generator=g, device=dev, dtype=dt) for _ in range(3))
    seed = 77 if gumbel else None
    got = {}
    for name, flags, out in (("split", gca.FLAG_FUSED_TOPK, None), ("matrix", gca.FLAG_MATERIALIZE, None),
                             ("one pass", gca.FLAG_FUSED_TOPK, q)):
        p = gca.problem(1, 2, nC, k, D=D, Hr=2, dtype=dtype, flags=flags, gumbel_seed=seed)
        assert name == "matrix" or gca.workspace_size(p, gca.OP_FORWARD) == 0
        f = gca.forward(p, lq, lk, q, kk, v, out=out)
        got[name] = f["idx"].cpu().numpy(), host64(f["sel"])
    for name in ("matrix", "one pass"):
        # the scores are the same products summed in the same order
        np.testing.assert_array_equal(got["split"][0], got[name][0])
        assert max_abs_rel(got["split"][1], got[name][1]) <= 1e-5


@pytest.mark.parametrize("dtype,D,nC,k,gumbel", [
    ("bf16", 64, 300, 8, False), ("bf16", 512, 150, 16, True), ("fp32", 256, 200, 5, False),   # queries in registers
    ("bf16", 576, 300, 8, False), ("bf16", 1024, 150, 16, True), ("fp32", 320, 200, 5, False),  # both through LDS,
    ("bf16", 1024, 290, 16, True), ("fp32", 320, 260, 5, False),                                # from 256 chunks
])
def test_select_without_matrix_takes_finite_scores_only(dev, dtype, D, nC, k, gumbel):
    """Scores that overflow to +inf and -inf are no candidates, in rows with and without k finite
    ones, for every form of the selection.  (Wide landmarks run one pass when the output overlaps
    an input or the chunks are few; narrow ones only for k > 16.)"""
    import torch
    from paper_2410_01651_amd import gca
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    rng = np.random.default_rng(D + nC)
    lk = np.zeros((1, 2, nC, D), np.float32)
    lq = np.zeros((1, 2, nC, D), np.float32)
    big = rng.random((1, 2, nC)) < np.where(np.arange(nC) < 40, 0.9, 0.2)
    # distinct whole numbers, and values that 16 overflows and 1/2 does not
    whole = np.stack([rng.permutation(nC) - nC // 2 for _ in range(2)])[None]
    lk[..., 3] = np.where(big, rng.choice([-3e38, 3e38], big.shape), whole)
    lq[..., 3] = rng.choice([16.0, 16.0, 0.5, 0.0], (1, 2, nC))
    g = torch.Generator(device=dev).manual_seed(D)
    q, kk, v = (torch.randn(1, 2, nC * 64, 64, generator=g, device=dev, dtype=dt) for _ in range(3))
    tq, tk = (torch.from_numpy(a).to(dev).to(dt) for a in (lq, lk))
    seed = 5 if gumbel else None
    got = {}
    for name, flags, out in (("split", gca.FLAG_FUSED_TOPK, None), ("matrix", gca.FLAG_MATERIALIZE, None),
                             ("overlap", gca.FLAG_FUSED_TOPK, q)):
        p = gca.problem(1, 2, nC, k, D=D, Hr=2, dtype=dtype, flags=flags, gumbel_seed=seed)
        f = gca.forward(p, tq, tk, q, kk, v, out=out)
        got[name] = f["idx"].cpu().numpy(), host64(f["sel"])
    with np.errstate(over="ignore"):
        sc = (host64(tq)[..., 3][..., :, None] * host64(tk)[..., 3][..., None, :]).astype(np.float32)
    cand = np.isfinite(sc) & np.tri(nC, k=-1, dtype=bool)
    for name, (i, s) in got.items():
        assert np.array_equal((i >= 0).sum(-1), np.minimum(cand.sum(-1), k)), name
        assert np.isfinite(s[i >= 0]).all(), name
        np.testing.assert_array_equal(i, got["matrix"][0])
        np.testing.assert_array_equal(s, got["matrix"][1])


def _kernels(fn):
    """Names of the kernels that fn launches, in order."""
    import ctypes
    import torch
    from paper_2410_01651_amd import gca
    hip = ctypes.CDLL("libamdhip64.so")
    ev = (ctypes.c_void_p * 32)()
    for i in range(32):
        assert hip.hipEventCreate(ctypes.byref(ev, i * ctypes.sizeof(ctypes.c_void_p))) == 0
    try:
        torch.cuda.synchronize()
        gca.profile_arm(ev, 32)
        fn()
        torch.cuda.synchronize()
        return gca.profile_record()
    finally:
        gca.profile_arm(None, 0)
        for i in range(32):
            hip.hipEventDestroy(ctypes.c_void_p(ev[i]))


@pytest.mark.parametrize("B,nC,split", [(1, 64, False), (1, 255, False), (1, 256, True), (8, 128, False),
                                        (7, 146, False), (8, 129, True)])
def test_wide_select_splits_many_chunks_only(dev, B, nC, split):
    """Few chunks are too few tiles for the split selection to pay for its two extra launches."""
    import torch
    from paper_2410_01651_amd import gca
    p = gca.problem(B, 1, nC, 4, D=1024, flags=gca.FLAG_FUSED_TOPK)
    lq, lk = (torch.zeros(B, 1, nC, 1024, device=dev, dtype=torch.bfloat16) for _ in range(2))
    q, kk, v = (torch.zeros(B, 1, nC * 64, 64, device=dev, dtype=torch.bfloat16) for _ in range(3))
    names = _kernels(lambda: gca.forward(p, lq, lk, q, kk, v))
    assert ("select_wide_kernel" in names) == split
    assert ("fused_select_kernel" in names) != split


@pytest.mark.parametrize("B,H,nC,k,obo", [(65, 4, 40, 8, False), (20, 13, 9, 12, True), (130, 2, 33, 32, False),
                                          (300, 1, 3, 5, False)])
def test_decode_large_batch_equals_small(dev, B, H, nC, k, obo):
    """Batches of more (batch, head) items than compute units keep one slot per wave pair
    resident; the same items in batches of a few keep two."""
    import torch
    from paper_2410_01651_amd import gca
    g = torch.Generator(device=dev).manual_seed(B)
    D = 192
    t = {n: torch.randn(s, generator=g, device=dev, dtype=torch.bfloat16)
         for n, s in (("lmk_q", (B, 1, 1, D)), ("lmk_k", (B, 1, nC, D)), ("q", (B, H, 64, 64)),
                      ("k", (B, H, nC * 64, 64)), ("v", (B, H, nC * 64, 64)))}
    run = lambda b0, n: gca.forward(gca.problem(n, H, nC, k, D=D, mode="decode", off_by_one=obo),  # noqa: E731
                                    *(t[x][b0:b0 + n].contiguous() for x in ("lmk_q", "lmk_k", "q", "k", "v")))
    whole = run(0, B)
    for b0 in range(0, B, 16):
        part = run(b0, min(16, B - b0))
        for n, tol in (("idx", 0.0), ("sel", 1e-6), ("w", 1e-6), ("lse", 1e-6), ("out", 2.0 ** -7)):
            a, b = whole[n][b0:b0 + 16], part[n]
            if n == "idx":
                assert torch.equal(a, b)
            else:
                assert max_abs_rel(host64(a), host64(b)) <= tol, n


@pytest.mark.parametrize("B,nC,k,pw", [(4, 8192, 14, 32), (4, 16384, 18, 64), (4, 16384, 27, 64), (4, 16000, 32, 64),
                                       (18, 896, 10, 16), (11, 5888, 22, 64), (2, 1000, 9, 8)])
def test_decode_winners_in_one_scan_list(dev, B, nC, k, pw):
    """Most of a row's best k in the scan's first list (chunks c < 4 pw with c mod 32 < 8, pw
    chunks per list), and list counts whose entries leave the merge's last step of 64 lanes
    partial.  Scores are small whole numbers, so the selection is exact."""
    import torch
    from oracle import gca as og
    from paper_2410_01651_amd import gca
    rng = np.random.default_rng(nC + k)
    D = 256
    val = -rng.integers(1, 256, (B, nC)).astype(np.float32)
    first = np.arange(nC)[(np.arange(nC) < 4 * pw) & (np.arange(nC) % 32 < 8)]
    for b in range(B):
        n = min(len(first), k + 2)
        val[b, rng.choice(first, n, replace=False)] = 1 + rng.permutation(n)
        val[b, rng.integers(nC)] = 40
    lk = np.zeros((B, 1, nC, D), np.float32)
    lk[:, 0, :, 3] = val
    lq = np.zeros((B, 1, 1, D), np.float32)
    lq[..., 3] = 16.0
    g = torch.Generator(device=dev).manual_seed(nC)
    q = torch.randn(B, 1, 64, 64, generator=g, device=dev, dtype=torch.bfloat16)
    kk, v = (torch.randn(B, 1, nC * 64, 64, generator=g, device=dev, dtype=torch.bfloat16) for _ in range(2))
    p = gca.problem(B, 1, nC, k, D=D, mode="decode")  # score scale 1/16
    up = lambda a: torch.from_numpy(a).to(dev).bfloat16()  # noqa: E731
    f = gca.forward(p, up(lq), up(lk), q, kk, v)
    ref_i, ref_s = og.topk(val[:, None, None, :].astype(np.float64), k)
    np.testing.assert_array_equal(f["idx"].cpu().numpy(), ref_i)
    np.testing.assert_array_equal(host64(f["sel"]), ref_s)


@pytest.mark.parametrize("mode,Hr,nC,k,D,hot", [
    ("causal", 1, 2, 1, 64, False),
    ("causal", 1, 17, 3, 64, False),       # a second group of one chunk
    ("causal", 2, 300, 8, 512, True),      # one group collects more entries than fit in LDS
    ("causal", 1, 4200, 2, 1024, False),   # 32 chunks per group; landmark rows of two waves
    ("decode", 1, 70000, 9, 192, False),   # 512 chunks per group, one landmark row
    ("causal", 1, 1024, 32, 64, False),    # 8 chunks per group; as many entries as one launch takes
    ("causal", 1, 1025, 32, 64, False),    # more: a launch per step
    ("causal", 2, 4200, 8, 64, False),
    ("causal", 1, 4200, 8, 192, True),     # the same with lists of 4,199 entries
    ("causal", 1, 16400, 3, 64, False),
])
def test_backward_preparation(dev, mode, Hr, nC, k, D, hot):
    """Fusion weights, inverse lists and landmark gradients against fp64 torch: with dV and
    the landmark gradients linear in them, a missing, doubled or misplaced list entry is
    an error of the size of the result (tolerance: the bf16 rounding of dV, fp32 sums)."""
    import torch
    from paper_2410_01651_amd import gca
    B, H = 1, 2
    nQ = nC if mode == "causal" else 1
    rng = np.random.default_rng(nC)
    idx = np.full((B, Hr, nQ, k), -1, np.int32)
    sel = np.full((B, Hr, nQ, k), -np.inf, np.float32)
    for r in range(Hr):
        for t in range(nQ):
            past = t if mode == "causal" else nC
            n = min(past, k)
            idx[0, r, t, :n] = np.arange(n) if hot else np.sort(rng.choice(past, size=n, replace=False))
            sel[0, r, t, :n] = rng.standard_normal(n)
    ti, ts = torch.from_numpy(idx).to(dev), torch.from_numpy(sel).to(dev)
    g = torch.Generator(device=dev).manual_seed(nC)
    rnd = lambda *s: torch.randn(*s, generator=g, device=dev, dtype=torch.bfloat16)  # noqa: E731
    q, do = rnd(B, H, nQ * 64, 64), rnd(B, H, nQ * 64, 64)
    kk, v = rnd(B, H, nC * 64, 64), rnd(B, H, nC * 64, 64)
    lq, lk = rnd(B, Hr, nQ, D), rnd(B, Hr, nC, D)
    p = gca.problem(B, H, nC, k, D=D, Hr=Hr, mode=mode)
    _, lse, w = gca.grouped_xattn_fwd(p, q, kk, v, ti, ts)
    d = gca.grouped_xattn_bwd(p, q, kk, v, ti, ts, lse, do, lq, lk)
    w64 = torch.softmax(ts.double(), dim=-1).nan_to_num(0.0)
    dv = torch.zeros(H, nC, 64, 64, dtype=torch.float64, device=dev)
    shift = 1 if mode == "causal" else 0
    for h in range(H):
        r = h if Hr > 1 else 0
        for s in range(k):
            j = ti[0, r, :nQ - shift, s].long()
            t = torch.nonzero(j >= 0)[:, 0]
            if not len(t):
                continue
            j, c = j[t], t + shift
            a = torch.bmm(q[0, h].view(nQ, 64, 64)[c].double(),
                          kk[0, h].view(nC, 64, 64)[j].double().transpose(1, 2).contiguous()) / 8
            pw = torch.softmax(a, dim=2) * w64[0, r, t, s][:, None, None]
            dv[h].index_add_(0, j, torch.bmm(pw.transpose(1, 2).contiguous(), do[0, h].view(nQ, 64, 64)[c].double()))
    assert max_abs_rel(host64(d["dv"]), dv.view(1, H, nC * 64, 64).cpu().numpy()) <= 2.0 ** -7
    # landmark gradients from the kernel's own dsel
    glq, glk = torch.zeros(Hr, nQ, D, dtype=torch.float64, device=dev), torch.zeros(Hr, nC, D, dtype=torch.float64,
                                                                                    device=dev)
    for r in range(Hr):
        for s in range(k):
            j = ti[0, r, :, s].long()
            t = torch.nonzero(j >= 0)[:, 0]
            c = d["dsel"][0, r, t, s].double()[:, None] / D ** 0.5
            glq[r, t] += c * lk[0, r, j[t]].double()
            glk[r].index_add_(0, j[t], c * lq[0, r, t].double())
    assert max_abs_rel(host64(d["dlmk_q"]), glq[None].cpu().numpy()) <= 1e-5
    assert max_abs_rel(host64(d["dlmk_k"]), glk[None].cpu().numpy()) <= 1e-5


@pytest.mark.parametrize("dtype,B,nC,k,D,hot", [
    ("bf16", 2, 511, 3, 64, False),     # 1,022 rows: a workgroup each
    ("bf16", 3, 343, 3, 64, False),     # 1,029: a wave each, the last workgroup with one row
    ("bf16", 1, 2000, 32, 192, False),  # two groups per wave, idle lanes; first chunks' lists on four waves
    ("bf16", 7, 450, 8, 512, True),     # one group; hot chunks of several slices
    ("fp32", 9, 347, 4, 256, False),
    ("fp32", 4, 300, 32, 64, True),
])
def test_landmark_gradients_of_many_rows(dev, dtype, B, nC, k, D, hot):
    """dlmk_q and dlmk_k against fp64 torch from the kernel's own dsel (tolerance: fp32 sums)."""
    import torch
    from paper_2410_01651_amd import gca
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device=dev).manual_seed(nC)
    t = torch.arange(nC, device=dev).view(1, 1, nC, 1)
    s = torch.arange(k, device=dev).view(1, 1, 1, k)
    j = s.expand(B, 1, nC, k) if hot else (t * (s + torch.rand(B, 1, nC, k, generator=g, device=dev)) / k).long()
    ok = (j < t) if hot else (t > s)
    idx = torch.where(ok, j, -1).to(torch.int32).contiguous()
    sel = torch.randn(B, 1, nC, k, generator=g, device=dev).masked_fill(idx < 0, float("-inf"))
    rnd = lambda *a: torch.randn(*a, generator=g, device=dev, dtype=dt)  # noqa: E731
    q, kk, v, do = (rnd(B, 1, nC * 64, 64) for _ in range(4))
    lq, lk = rnd(B, 1, nC, D), rnd(B, 1, nC, D)
    p = gca.problem(B, 1, nC, k, D=D, dtype=dtype)
    _, lse, _ = gca.grouped_xattn_fwd(p, q, kk, v, idx, sel)
    d = gca.grouped_xattn_bwd(p, q, kk, v, idx, sel, lse, do, lq, lk)
    at = idx.long().clamp(min=0) + nC * torch.arange(B, device=dev).view(B, 1, 1, 1)   # rows of [B * nC, D]
    c = (d["dsel"].double() * (idx >= 0) / D ** 0.5).view(B * nC, k)
    lq64, lk64 = lq.double().view(B * nC, D), lk.double().view(B * nC, D)
    glq, glk = torch.zeros_like(lq64), torch.zeros_like(lk64)
    for e in range(k):
        a = at.view(B * nC, k)[:, e]
        glq += c[:, e:e + 1] * lk64[a]
        glk.index_add_(0, a, c[:, e:e + 1] * lq64)
    assert max_abs_rel(host64(d["dlmk_q"]), glq.view(B, 1, nC, D).cpu().numpy()) <= 1e-5
    assert max_abs_rel(host64(d["dlmk_k"]), glk.view(B, 1, nC, D).cpu().numpy()) <= 1e-5


@pytest.mark.parametrize("dtype,H,Hr,nC,k,holes,obo,copies", [
    ("bf16", 1, 1, 2, 1, False, False, 300),
    ("bf16", 4, 1, 16, 8, True, True, 9),       # alone: four wave pairs per item
    ("bf16", 12, 12, 37, 5, True, False, 3),    # two
    ("bf16", 3, 1, 30, 12, False, False, 12),
    ("fp32", 1, 1, 16, 2, True, False, 40),
    ("fp32", 4, 4, 60, 11, True, True, 5),
    ("fp32", 8, 1, 63, 8, True, False, 7),      # 504 and 3,528 items: two ring slots and one in the forward
    ("fp32", 12, 1, 90, 3, True, True, 4),      # 1,080 (two slots) and 4,320
    ("fp32", 4, 1, 60, 1, True, False, 30),     # one slot per chunk: nothing to share out
    ("bf16", 12, 12, 42, 1, False, True, 4),
])
def test_few_items_equal_many(dev, dtype, H, Hr, nC, k, holes, obo, copies):
    """A problem of few items (several wave pairs per query or key chunk) against the same
    sequence repeated in a batch of many (one pair or wave per chunk)."""
    import torch
    from paper_2410_01651_amd import gca
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    idx, sel = _lists(np.random.default_rng(nC), Hr, nC, k, holes)
    ti, ts = (torch.from_numpy(x.reshape(1, Hr, nC, k)).to(dev) for x in (idx, sel))
    g = torch.Generator(device=dev).manual_seed(nC + k)
    q, kk, v, do = (torch.randn(1, H, nC * 64, 64, generator=g, device=dev, dtype=dt) for _ in range(4))
    got = []
    for B in (1, copies):
        rep = lambda x: x.expand(B, *x.shape[1:]).contiguous()  # noqa: E731
        p = gca.problem(B, H, nC, k, D=64, Hr=Hr, dtype=dtype, off_by_one=obo)
        a = [rep(x) for x in (q, kk, v, ti, ts)]
        out, lse, w = gca.grouped_xattn_fwd(p, *a)
        d = gca.grouped_xattn_bwd(p, *a, lse, rep(do), landmark_grads=False)
        got.append(dict(out=out, lse=lse, w=w, dq=d["dq"], dk=d["dk"], dv=d["dv"], dsel=d["dsel"]))
    few, many = got
    for n in few:
        # fp32 sums in another order; bf16 results and probabilities rounded from them
        tol = 1e-6 if n in ("lse", "w") else (2.0 ** -7 if dtype == "bf16" and n != "dsel" else 1e-5)
        ref = host64(few[n])
        for b in (0, copies - 1):
            assert max_abs_rel(host64(many[n][b:b + 1]), ref) <= tol, (n, b)


def test_one_slot_takes_the_per_chunk_forward(dev):
    """k = 1 leaves nothing for several wave pairs to take side by side."""
    import torch
    from paper_2410_01651_amd import gca
    for dtype, dt in (("bf16", torch.bfloat16), ("fp32", torch.float32)):
        q, kk, v = (torch.zeros(1, 4, 40 * 64, 64, device=dev, dtype=dt) for _ in range(3))
        for k, name in ((1, "xattn_fwd_kernel"), (2, "xattn_decode_kernel")):
            idx = torch.zeros(1, 1, 40, k, device=dev, dtype=torch.int32)
            sel = torch.zeros(1, 1, 40, k, device=dev)
            p = gca.problem(1, 4, 40, k, dtype=dtype)
            assert _kernels(lambda: gca.grouped_xattn_fwd(p, q, kk, v, idx, sel)) == [name]


def _best_ms(fn):
    """The shortest of five runs of 20 calls in a graph."""
    import torch
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        fn()
    s.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        for _ in range(20):
            fn()
    a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    t = []
    for _ in range(6):
        a.record()
        graph.replay()
        b.record()
        torch.cuda.synchronize()
        t.append(a.elapsed_time(b))
    return min(t[1:])


def _cus():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count


def _fp32_step(dev, items, k, bwd):
    """Time of the attention forward or the backward of `items` fp32 chunks in 12 heads."""
    import torch
    from paper_2410_01651_amd import gca
    g = torch.Generator(device=dev).manual_seed(items)
    H, nC = 12, items // 12
    # every row retrieves the k chunks before it: no long lists, whose length would be the time
    ti = (torch.arange(nC, device=dev)[:, None] - k + torch.arange(k, device=dev)).clamp(min=-1)
    ti = ti.to(torch.int32)[None, None].contiguous()
    ts = torch.where(ti >= 0, 0.0, float("-inf"))
    q, kk, v, do = (torch.randn(1, H, nC * 64, 64, generator=g, device=dev) for _ in range(4))
    p = gca.problem(1, H, nC, k, D=64, dtype="fp32")
    out, lse, w = gca.grouped_xattn_fwd(p, q, kk, v, ti, ts)
    if not bwd:
        return _best_ms(lambda: gca.grouped_xattn_fwd(p, q, kk, v, ti, ts, out=out, lse=lse, w=w))
    ws = gca.workspace(p, gca.OP_BACKWARD)[0]
    d = gca.grouped_xattn_bwd(p, q, kk, v, ti, ts, lse, do, landmark_grads=False, ws=ws)
    return _best_ms(lambda: gca.grouped_xattn_bwd(p, q, kk, v, ti, ts, lse, do, landmark_grads=False, ws=ws, grads=d))


def test_fp32_forward_time_of_two_items_per_cu(dev):
    """Two fp32 items per CU take 0.59 of the time of four (with one ring slot 0.89)."""
    cus = _cus()
    assert _fp32_step(dev, 2 * cus // 12 * 12, 8, False) <= 0.75 * _fp32_step(dev, 4 * cus // 12 * 12, 8, False)


def test_fp32_backward_time_of_one_slot(dev):
    """Lists of one entry give four wave pairs per chunk nothing to share: two chunks per CU
    take 0.64 of the time of three (0.83 with four pairs per chunk)."""
    cus = _cus()
    assert _fp32_step(dev, 2 * cus // 12 * 12, 1, True) <= 0.75 * _fp32_step(dev, 3 * cus // 12 * 12, 1, True)


@pytest.mark.parametrize("mode", ["causal", "decode"])
@pytest.mark.parametrize("nC,k", [(1, 1), (64, 32), (65, 8), (1024, 31), (1100, 1), (3000, 32)])
def test_topk_adversarial_rows(dev, mode, nC, k):
    """Rows that ascend (every column beats the ones before), descend, are constant (ties to
    the lower chunk), mix signs and zeros, or hold infinities and NaN (no candidates)."""
    import torch
    from oracle import gca as og
    from paper_2410_01651_amd import gca
    rng = np.random.default_rng(nC)
    nQ = nC if mode == "causal" else 1
    B = 1 if mode == "causal" else 6
    r = np.empty((B, 1, nQ, nC), np.float32)
    for i in range(B * nQ):
        x = rng.standard_normal(nC)
        row = [np.sort(x), -np.sort(x), np.full(nC, -1.5), np.sign(x) * rng.integers(0, 3, nC),
               np.where(x > 0.3, np.inf, np.where(x < -0.5, np.nan, x)), x][i % 6]
        r.reshape(-1, nC)[i] = row
    if mode == "causal":
        r[0, 0][np.triu_indices(nC)] = -np.inf
    p = gca.problem(B, 1, nC, k, D=64, mode=mode)
    idx, sel = gca.topk(p, torch.from_numpy(r).to(dev))
    ref_i, ref_s = og.topk(r.astype(np.float64), k)
    np.testing.assert_array_equal(idx.cpu().numpy(), ref_i)
    np.testing.assert_array_equal(host64(sel), ref_s)


@pytest.mark.parametrize("nC,k", [(1023, 8), (5000, 1), (5000, 8), (5000, 31), (5000, 32)])
def test_topk_rows_in_batches(dev, nC, k):
    """Rows whose batches of 1,024 columns each hold more survivors than fit, none, or ties with
    what earlier batches hold: stairs up and down, saw teeth, plateaus of the lowest and highest
    finite value, a rise among infinities."""
    import torch
    from oracle import gca as og
    from paper_2410_01651_amd import gca
    j = np.arange(nC)
    big = np.finfo(np.float32).max
    rows = [j, -j, j // 100, -(j // 100), j % 1024, -(j % 1000), np.full(nC, -big), np.where(j % 3 == 0, big, 0.0),
            np.where(j % 2 == 0, np.inf, j), np.where(j < nC - 3, -np.inf, -1.0), np.where(j % 5 == 0, np.nan, j // 7),
            np.where(j % 64 == 5, -0.0, 0.0)]
    r = np.stack(rows).astype(np.float32).reshape(len(rows), 1, 1, nC)
    idx, sel = gca.topk(gca.problem(len(rows), 1, nC, k, D=64, mode="decode"), torch.from_numpy(r).to(dev))
    ref_i, ref_s = og.topk(r.astype(np.float64), k)
    np.testing.assert_array_equal(idx.cpu().numpy(), ref_i)
    np.testing.assert_array_equal(host64(sel), ref_s)


def test_topk_time_does_not_depend_on_the_order_of_scores(dev):
    """Rising rows (recency) cost about what random ones do (a floor for a row's first batch
    alone made them 4.8 times as long)."""
    import torch
    from paper_2410_01651_amd import gca
    nC = 8192
    x = torch.randn(64, 1, 1, nC, generator=torch.Generator(device=dev).manual_seed(1), device=dev)
    p = gca.problem(64, 1, nC, 8, D=64, mode="decode")
    a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))

    def best(s):
        idx, sel = gca.topk(p, s)
        t = []
        for _ in range(5):
            a.record()
            for _ in range(50):
                gca.topk(p, s, idx=idx, sel=sel)
            b.record()
            torch.cuda.synchronize()
            t.append(a.elapsed_time(b))
        return min(t)
    assert best(x.sort(-1).values.contiguous()) <= 2.0 * best(x)
