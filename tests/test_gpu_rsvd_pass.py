"""The one-pass power step of Algorithm 1 on bf16 inputs (W = H^T (H Omega) and Y^T Y without Y in memory) at
the sizes where it can go wrong: every block width of both embeddings, sequences around its 32-row blocks and
its chunks, ragged batches with NaN past the valid rows; against the oracle of the printed algorithm.

Tolerance: float sums leave W = H^T H Omega off by about 2^-21 of its norm (measured 2^-20.6 at worst), which turns the
range of the block by that times cond(W) (up to 1e3 here: rank r above a noise floor, Gaussian Omega), and V V^T
and S with it.  S and P = H V see the factors at 1e-5 beside that."""
import numpy as np
import pytest

from paper_2603_02561_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,r", [(64, 16), (64, 32), (64, 48), (64, 64), (128, 16), (128, 32), (128, 48), (128, 64)])
@pytest.mark.parametrize("N,low", [(131, 0), (511, 200), (1024, 0), (2085, 300)])
def test_power_pass(d, r, N, low):
    import torch
    from oracle import oracle
    from paper_2603_02561_amd import binding
    if not torch.cuda.is_available():
        pytest.fail("needs the GPU")
    w = synth.make_workload("t", 3, N, d, r, 8, synth.BF16, "spectrum", 0.3, 0.02,
                            var_len=(low, N) if low else None, seed=900 + d + r + N)
    db = binding.DeviceBatch(w.X, w.Q, w.lengths, w.r, True)
    for b in range(w.B):
        db.X[b, int(w.lengths[b]):] = float("nan")
    Om = synth.make_omega(w.B, d, r)
    Omd = torch.from_numpy(Om).cuda()
    for q in (0, 1):
        print(f"[case] power pass d={d} r={r} N={N} n_iter={q}", flush=True)
        db.factorize_rsvd(Omd, q)
        torch.cuda.synchronize()
        S, V, info = db.S.cpu().numpy().astype(np.float64), db.V.cpu().numpy().astype(np.float64), db.info.cpu().numpy()
        f = oracle.rsvd_alg1(w.X, Om, q, w.lengths)
        for b in range(w.B):
            assert info[b] == 0
            H = w.X[b, :int(w.lengths[b])].astype(np.float64)
            block = Om[b].astype(np.float64)
            cond = np.linalg.cond(H @ block) if q == 0 else np.linalg.cond(H.T @ (H @ block))
            s_err = np.abs(S[b] - f["S"][b]).max() / f["S"][b][0]
            p_err = np.abs(V[b] @ V[b].T - f["V"][b] @ f["V"][b].T).max()
            print(f"  user {b}: cond {cond:.0f} S {s_err:.2e} proj {p_err:.2e}", flush=True)
            assert s_err < 1e-5 + 2.0**-20 * cond and p_err < 1e-5 + 2.0**-20 * cond
            assert np.abs(V[b].T @ V[b] - np.eye(r)).max() < 2e-6


def test_equal_singular_values():
    """All singular values equal (rows of the identity over and over): the dense solver of the last step cannot
    separate its vectors and leaves them to the Jacobi sweeps.  S to 1e-5, V orthonormal."""
    import torch
    from paper_2603_02561_amd import binding
    if not torch.cuda.is_available():
        pytest.fail("needs the GPU")
    for d, r in ((64, 32), (128, 64)):
        X = np.tile(np.eye(d, dtype=np.float32), (1, 6, 1))
        db = binding.DeviceBatch(X, X[:, :8].copy(), None, r, True)
        for q in (0, 1):
            print(f"[case] equal singular values d={d} r={r} n_iter={q}", flush=True)
            db.factorize_rsvd(torch.from_numpy(synth.make_omega(1, d, r)).cuda(), q)
            torch.cuda.synchronize()
            V = db.V[0].double().cpu().numpy()
            assert int(db.info[0]) == 0
            assert np.abs(db.S[0].cpu().numpy() / np.sqrt(6.0) - 1).max() < 1e-5
            assert np.abs(V.T @ V - np.eye(r)).max() < 1e-5
