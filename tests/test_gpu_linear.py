"""GPU parity of linear attention (Query (Key^T Value) with Key = Value = X) and of the folded
projections against the oracle.  Tolerances: products accumulate in float over <= N terms twice;
1e-4 for float inputs; 1e-3 for bf16 inputs (the inputs are exact, the only 16-bit rounding is the
optional bf16 output of the folding step, 2^-9 relative, tested at 5e-3)."""
import numpy as np
import pytest

from paper_2603_02561_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("these tests need the GPU")
    from paper_2603_02561_amd import binding
    return binding


@pytest.fixture(scope="module")
def oracle():
    from oracle import oracle as o
    return o


CASES = [
    ("f32_d64", synth.make_workload("t", 2, 333, 64, 8, 70, synth.F32, "gauss_lowrank", seed=201)),
    ("bf16_d128_varlen", synth.make_workload("t", 3, 900, 128, 32, 130, synth.BF16, "spectrum", 0.5, 0.02,
                                             var_len=(300, 900), seed=202)),
    ("f32_d256", synth.make_workload("t", 2, 300, 256, 16, 41, synth.F32, "gauss_lowrank", seed=203)),
]


def rel_err(got, want):
    return max(np.abs(got[b] - want[b]).max() / np.abs(want[b]).max() for b in range(want.shape[0]))


@pytest.mark.parametrize("name,w", CASES, ids=[c[0] for c in CASES])
def test_linear_attention(lib, oracle, name, w):
    import torch
    print(f"[case] linear attention {name}", flush=True)
    db = lib.DeviceBatch(w.X, w.Q, w.lengths, w.r, w.dtype == synth.BF16)
    db.linear(0.37)
    torch.cuda.synchronize()
    want = oracle.linear_attention(w.Q, w.X, 0.37, w.lengths)
    err = rel_err(db.O.cpu().numpy().astype(np.float64), want)
    print(f"  err {err:.3e}", flush=True)
    assert err < (1e-4 if w.dtype == synth.F32 else 1e-3)


@pytest.mark.parametrize("name,w", CASES, ids=[c[0] for c in CASES])
def test_folded_projections(lib, oracle, name, w):
    """C (W_Q W_K^T) -> SVD-attention (mode 0) -> W_V on the GPU against the oracle doing the same
    steps in double on the same folded candidates."""
    import torch
    print(f"[case] folded projections {name}", flush=True)
    g = np.random.default_rng(7)
    d = w.d
    Wf = (np.eye(d) + 0.1 * g.standard_normal((d, d)) / np.sqrt(d)).astype(np.float32)
    Wv = (np.eye(d) + 0.1 * g.standard_normal((d, d)) / np.sqrt(d)).astype(np.float32)
    bf16 = w.dtype == synth.BF16
    db = lib.DeviceBatch(w.X, w.Q, w.lengths, w.r, bf16)
    Wf_d, Wv_d = torch.from_numpy(Wf).cuda(), torch.from_numpy(Wv).cuda()
    Qf = torch.empty_like(db.Q)
    lib.solar_apply_weights(db.Q, Wf_d, Qf)
    torch.cuda.synchronize()
    want_qf = oracle.apply_weights(w.Q, Wf)
    got_qf = Qf.float().cpu().numpy().astype(np.float64)
    e1 = rel_err(got_qf, want_qf)
    print(f"  folded candidates err {e1:.3e}", flush=True)
    assert e1 < (1e-5 if not bf16 else 5e-3)
    # the operator on the folded candidates (the GPU's own, rounded if bf16), then W_V
    db.Q = Qf
    db.factorize()
    db.attention(1.0, 0)
    Of = torch.empty_like(db.O)
    lib.solar_apply_weights(db.O, Wv_d, Of)
    torch.cuda.synchronize()
    f = oracle.svd_factorize(w.X, w.r, w.lengths)
    want = oracle.apply_weights(oracle.svd_attention(got_qf, w.X, f["S"], f["V"], 1.0, 0, w.lengths), Wv)
    e2 = rel_err(Of.cpu().numpy().astype(np.float64), want)
    print(f"  output err {e2:.3e}", flush=True)
    assert e2 < (1e-4 if not bf16 else 2e-2)


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("rows", [1, 31, 33, 255, 257, 8225])
@pytest.mark.parametrize("in_bf16,out_bf16", [(True, True), (True, False), (False, True), (False, False)])
def test_row_blocks(lib, d, rows, in_bf16, out_bf16):
    """Rows at the edges of the 32-row blocks, of a workgroup's eight and of the second round of workgroups,
    against the product in double precision.  Float outputs: the operands are exact sums of bf16 terms, so
    what is left is the rounding of a float sum of d products, d 2^-24 at worst (1.6e-5 of the norm of a row
    times that of a column; measured 3e-7); a bf16 output adds 2^-9 of its own size (2^-7 allowed)."""
    import torch
    print(f"[case] row blocks d={d} rows={rows} {in_bf16} {out_bf16}", flush=True)
    g = torch.Generator().manual_seed(1000 * d + rows)
    In = torch.randn(rows, d, generator=g).to(torch.bfloat16 if in_bf16 else torch.float32).cuda()
    W = torch.randn(d, d, generator=g).cuda()
    Out = torch.full((rows, d), 7.0, dtype=torch.bfloat16 if out_bf16 else torch.float32, device="cuda")
    lib.solar_apply_weights(In, W, Out)
    torch.cuda.synchronize()
    want = In.double() @ W.double()
    size = In.double().norm(dim=1, keepdim=True) * W.double().norm(dim=0, keepdim=True)
    err = ((Out.double() - want).abs() / (size + (want.abs() * 2.0 ** 8 if out_bf16 else 0))).max().item()
    assert err < (2.0 ** -16 if not out_bf16 else 2.0 ** -15)


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("in_bf16", [False, True])
def test_extreme_rows(lib, d, in_bf16):
    """Rows with a value at the end of the float range (a mask value), an infinity or a NaN, and a matrix with such
    values: what comes out is what the sum of float products is, finite where that is finite, and rows
    beside them are not touched.  Finite outputs to d 2^-24 of the sum of the absolute products."""
    import torch
    print(f"[case] extreme rows d={d} {in_bf16}", flush=True)
    big = torch.finfo(torch.float32).max
    g = torch.Generator().manual_seed(d)
    In = torch.randn(70, d, generator=g)
    W = torch.randn(d, d, generator=g) / (4 * d)
    W[5] = torch.where(torch.arange(d) % 3 == 0, torch.full((d,), 2.0 ** -9), W[5])   # fewer than three terms
    In[:, 6] /= 16
    In[3, 5], In[8, 5], In[9, 5], In[40, 5] = -big, float("inf"), -float("inf"), float("nan")
    In[41, 5], In[41, 6] = float("inf"), -float("inf")
    In[69, 5] = 3.4e38
    In = In.to(torch.bfloat16 if in_bf16 else torch.float32).cuda()
    W = W.cuda()
    for matrix in (W, W.clone().index_fill_(0, torch.tensor([6], device="cuda"), -big)):
        Out = torch.full((70, d), 7.0, device="cuda")
        lib.solar_apply_weights(In, matrix, Out)
        torch.cuda.synchronize()
        want = In.double() @ matrix.double()
        size = In.double().abs() @ matrix.double().abs()
        finite = size < 0.5 * big                       # no partial sum overflows
        assert torch.equal(torch.isnan(want), torch.isnan(Out))
        assert torch.equal(want[torch.isinf(want)].float(), Out[torch.isinf(want)])
        assert finite.sum() > 60 * d
        assert ((Out.double() - want).abs()[finite] <= d * 2.0 ** -24 * size[finite]).all()


def test_linear_attention_extreme_query(lib):
    """A query row with a mask value in linear attention: finite where the float products are."""
    import torch
    g = torch.Generator().manual_seed(5)
    for d in (64, 128, 256):
        X = torch.randn(2, 50, d, generator=g).cuda() / 64
        Q = torch.randn(2, 40, d, generator=g).cuda()
        Q[0, 7, 3] = -torch.finfo(torch.float32).max
        O = torch.empty(2, 40, d, device="cuda")
        ws = torch.empty(lib.solar_workspace_bytes(2, 50, d, 1, 40, 0), dtype=torch.uint8, device="cuda")
        lib.solar_linear_attention(Q, X, None, 1.0, O, ws)
        torch.cuda.synchronize()
        G = X.double().transpose(1, 2).contiguous() @ X.double()
        want, size = Q.double() @ G, Q.double().abs() @ G.abs()
        assert torch.isfinite(O).all()
        assert ((O.double() - want).abs() <= (50 + d) * 2.0 ** -24 * size).all()


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("rows", [1, 40, 257, 20011, 70000])
@pytest.mark.parametrize("bf16", [True, False])
def test_in_place(lib, d, rows, bf16):
    """Out is In: the same bits as with an output of its own, at one and at several rounds of rows per workgroup, with a
    row that is taken a second time on the float instruction."""
    import torch
    print(f"[case] in place d={d} rows={rows} {bf16}", flush=True)
    g = torch.Generator().manual_seed(d + rows)
    In = torch.randn(rows, d, generator=g).to(torch.bfloat16 if bf16 else torch.float32).cuda()
    In[rows // 2, 3] = float("inf")
    W = torch.randn(d, d, generator=g).cuda()
    want = torch.empty_like(In)
    lib.solar_apply_weights(In, W, want)
    lib.solar_apply_weights(In, W, In)
    torch.cuda.synchronize()
    assert torch.equal(In.isnan(), want.isnan())
    assert torch.equal(In.nan_to_num(nan=0.0), want.nan_to_num(nan=0.0))


def test_linear_attention_in_place(lib):
    """O is Q (float), several users."""
    import torch
    g = torch.Generator().manual_seed(9)
    for d in (64, 128, 256):
        X, Q = torch.randn(3, 200, d, generator=g).cuda(), torch.randn(3, 333, d, generator=g).cuda()
        O = torch.empty_like(Q)
        ws = torch.empty(lib.solar_workspace_bytes(3, 200, d, 1, 333, 0), dtype=torch.uint8, device="cuda")
        lib.solar_linear_attention(Q, X, None, 0.5, O, ws)
        lib.solar_linear_attention(Q, X, None, 0.5, Q, ws)
        torch.cuda.synchronize()
        assert torch.equal(O, Q)
