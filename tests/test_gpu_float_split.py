"""Float inputs on the bf16 matrix instruction (values split into three bf16 terms): the Gram matrix and the
attention at the edges of their blocks, against double precision.

Tolerances: a Gram entry is a float sum of N terms, each off by at most 2^-24 of the product of the column
norms' shares: 2^-21 of |x_i| |x_j|, which the float instruction meets as well.  Attention 1e-5 of the largest output:
scores of magnitude up to 30 in float (2^-24 * 30 each way) move a weight by 4e-6 at most."""
import numpy as np
import pytest

from paper_2603_02561_amd import synth

pytestmark = pytest.mark.gpu


def _binding():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("needs the GPU")
    from paper_2603_02561_amd import binding
    return torch, binding


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("N", [1, 31, 32, 33, 127, 129, 513, 1100])
def test_gram_float(d, N):
    torch, sb = _binding()
    B = 3
    rng = np.random.default_rng(7 * N + d)
    X = rng.standard_normal((B, N, d)).astype(np.float32) * (1 + 100 * rng.random((1, 1, d))).astype(np.float32)
    lengths = np.array([N, max(1, N // 2), max(1, N - 1)], dtype=np.int32)
    Xd = torch.from_numpy(X).cuda()
    for b in range(B):
        Xd[b, lengths[b]:] = float("nan")
    G = torch.empty((B, d, d), device="cuda")
    ws = torch.empty(sb.solar_workspace_bytes(B, N, d, 1, 1, sb.SOLAR_F32), dtype=torch.uint8, device="cuda")
    sb.solar_gram(Xd, torch.from_numpy(lengths).cuda(), G, ws)
    got = G.double().cpu().numpy()
    for b in range(B):
        x = X[b, :lengths[b]].astype(np.float64)
        want = x.T @ x
        nrm = np.sqrt(np.diag(want))
        assert (np.abs(got[b] - want) / np.outer(nrm, nrm)).max() < 2.0**-21


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("N", [40, 700])
@pytest.mark.parametrize("value", [-3.4028235e38, 3.4e38, float("inf"), -float("inf"), 1e25, float("nan")])
def test_gram_float_extreme(d, N, value):
    """One entry of a user at the end of the float range, infinite or NaN, in the first and the last valid row: entries of
    G are what the sum of float products is (N 2^-24 of the sum of their sizes where that is finite, an infinity of the
    right sign where it overflows), and the columns and users beside it are not touched."""
    torch, sb = _binding()
    print(f"[case] extreme Gram d={d} N={N} {value}", flush=True)
    rng = np.random.default_rng(N + d)
    X = (rng.standard_normal((3, N, d)) / 16).astype(np.float32)
    X[0, 0, d - 3] = value
    X[1, N - 1, 5] = value
    G = torch.empty((3, d, d), device="cuda")
    ws = torch.empty(sb.solar_workspace_bytes(3, N, d, 1, 1, sb.SOLAR_F32), dtype=torch.uint8, device="cuda")
    sb.solar_gram(torch.from_numpy(X).cuda(), None, G, ws)
    got = G.double().cpu().numpy()
    x = X.astype(np.float64)
    big = float(np.finfo(np.float32).max)
    for b in range(3):
        with np.errstate(invalid="ignore"):
            want, size = x[b].T @ x[b], np.abs(x[b]).T @ np.abs(x[b])
            error = np.abs(got[b] - want)
        assert np.array_equal(np.isnan(got[b]), np.isnan(want))
        small = size < 0.5 * big
        assert small.sum() >= (d - 1) ** 2
        assert (error[small] <= N * 2.0**-24 * size[small]).all()
        over = np.abs(want) > 1.01 * big
        assert np.array_equal(got[b][over], np.sign(want[over]) * np.inf)


@pytest.mark.parametrize("d,r", [(64, 1), (64, 7), (64, 16), (128, 17), (128, 32), (128, 47), (128, 48), (64, 64), (256, 20),
                                 (256, 32)])
@pytest.mark.parametrize("B,N,M", [(1, 64, 1), (2, 65, 17), (3, 257, 130), (40, 130, 700)])
def test_attention_float(d, r, B, N, M):
    torch, sb = _binding()
    rng = np.random.default_rng(r + N)
    V = np.stack([np.linalg.qr(rng.standard_normal((d, r)))[0] for _ in range(B)]).astype(np.float32)
    P = rng.standard_normal((B, N, r)).astype(np.float32)
    Q = rng.standard_normal((B, M, d)).astype(np.float32)
    lengths = rng.integers(max(1, r if N >= r else 1), N + 1, size=B).astype(np.int32)
    Pd = torch.from_numpy(P).cuda()
    for b in range(B):
        Pd[b, lengths[b]:] = float("nan")
    S = torch.ones((B, r), device="cuda")
    O = torch.empty((B, M, d), device="cuda")
    scale = 30.0 / (4 * np.sqrt(r) + 8)
    if r > N:
        pytest.skip("rank above the sequence length is refused")
    sb.solar_svd_attention(torch.from_numpy(Q).cuda(), S, torch.from_numpy(V).cuda(), Pd,
                           torch.from_numpy(lengths).cuda(), N, float(scale), sb.SOLAR_ATTN_SEQ_SOFTMAX, O)
    got = O.double().cpu().numpy()
    for b in range(B):
        p, v = P[b, :lengths[b]].astype(np.float64), V[b].astype(np.float64)
        s = np.float64(np.float32(scale)) * (Q[b].astype(np.float64) @ v) @ p.T
        w = np.exp(s - s.max(1, keepdims=True))
        want = (w / w.sum(1, keepdims=True)) @ p @ v.T
        assert np.abs(got[b] - want).max() / np.abs(want).max() < 1e-5


@pytest.mark.parametrize("d,r", [(64, 16), (128, 30), (128, 48), (64, 64), (256, 32)])
@pytest.mark.parametrize("B,N,M", [(1, 300, 20), (9, 700, 130), (44, 300, 700), (8, 300, 8200)])
@pytest.mark.parametrize("value,query", [(-3.4028235e38, 1.0), (-1e30, 1e12)])
def test_attention_float_extreme(d, r, B, N, M, value, query):
    """A row of P with a value that has no bf16 terms, or with a score that overflows, far below the other scores of
    its user: its weight is zero and the rest of the softmax is not disturbed.  In the first user early in
    the sequence, in the last in its last valid row.  The shapes reach every form of the kernel."""
    torch, sb = _binding()
    print(f"[case] extreme attention d={d} r={r} B={B} N={N} M={M} {value}", flush=True)
    rng = np.random.default_rng(r + N + M)
    V = np.stack([np.abs(np.linalg.qr(rng.standard_normal((d, r)))[0]) for _ in range(B)]).astype(np.float32)
    P = rng.standard_normal((B, N, r)).astype(np.float32)
    Q = (np.abs(rng.standard_normal((B, M, d))) * query / 4).astype(np.float32)
    lengths = rng.integers(N - 40, N + 1, size=B).astype(np.int32)
    P[0, 11, r // 2] = value
    P[B - 1, lengths[B - 1] - 1, r - 1] = value
    O = torch.full((B, M, d), 7.0, device="cuda")
    sb.solar_svd_attention(torch.from_numpy(Q).cuda(), torch.ones((B, r), device="cuda"), torch.from_numpy(V).cuda(),
                           torch.from_numpy(P).cuda(), torch.from_numpy(lengths).cuda(), N, 0.5,
                           sb.SOLAR_ATTN_SEQ_SOFTMAX, O)
    got = O.cpu().numpy()
    assert np.isfinite(got).all()
    for b in sorted({0, B // 2, B - 1}):
        p, v = P[b, :lengths[b]].astype(np.float64), V[b].astype(np.float64)
        s = 0.5 * (Q[b].astype(np.float64) @ v) @ p.T
        w = np.exp(s - s.max(1, keepdims=True))
        want = (w / w.sum(1, keepdims=True)) @ p @ v.T
        # scores of magnitude up to 60 in float move a weight by 2^-24 * 60 each way
        assert np.abs(got[b] - want).max() / np.abs(want).max() < 1e-5


@pytest.mark.parametrize("d,r", [(64, 12), (128, 20), (128, 32), (128, 40), (64, 48), (128, 64), (256, 30)])
@pytest.mark.parametrize("B,N,M", [(44, 700, 700), (64, 520, 1030), (128, 330, 1024)])
def test_attention_float_two_query_blocks(d, r, B, N, M):
    """Batches of 256 and more workgroups of 128 queries, where a wave takes two blocks of sixteen queries (with the
    sequence shared between two groups of waves, and not from 1024 workgroups on): full chunks of 32 ranks, an odd last
    block, both, ragged, at least three steps of the loop.  A few users against double precision."""
    torch, sb = _binding()
    print(f"[case] two query blocks d={d} r={r} B={B} N={N} M={M}", flush=True)
    rng = np.random.default_rng(r + N)
    V = np.stack([np.linalg.qr(rng.standard_normal((d, r)))[0] for _ in range(B)]).astype(np.float32)
    P = rng.standard_normal((B, N, r), dtype=np.float32)
    Q = rng.standard_normal((B, M, d), dtype=np.float32)
    lengths = rng.integers(N // 2, N + 1, size=B).astype(np.int32)
    lengths[0], lengths[1] = N, r
    for b in range(B):
        P[b, lengths[b]:] = np.nan
    scale = 30.0 / (4 * np.sqrt(r) + 8)
    O = torch.empty((B, M, d), device="cuda")
    sb.solar_svd_attention(torch.from_numpy(Q).cuda(), torch.ones((B, r), device="cuda"), torch.from_numpy(V).cuda(),
                           torch.from_numpy(P).cuda(), torch.from_numpy(lengths).cuda(), N, float(scale),
                           sb.SOLAR_ATTN_SEQ_SOFTMAX, O)
    got = O.cpu().numpy()
    assert np.isfinite(got).all()
    for b in (0, 1, 2, B // 2, B - 1):
        p, v = P[b, :lengths[b]].astype(np.float64), V[b].astype(np.float64)
        s = np.float64(np.float32(scale)) * (Q[b].astype(np.float64) @ v) @ p.T
        w = np.exp(s - s.max(1, keepdims=True))
        want = (w / w.sum(1, keepdims=True)) @ p @ v.T
        assert np.abs(got[b] - want).max() / np.abs(want).max() < 1e-5
