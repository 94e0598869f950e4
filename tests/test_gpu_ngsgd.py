"""GPU parity of ngsgd_precondition and of the NG-SGD training step against the float64 oracle.

Eigenvector signs (and rotations inside near-degenerate eigenvalue clusters) are free, so the state is
compared through what is unique: the row space of R (principal angles), d, rho, t, and above all the
preconditioned output of every following minibatch."""
import numpy as np
import pytest

import gen
from oracle import dnn, ngsgd
from oracle import averaging
from tests.util import check_close, dev, host, rel_err, workspace

pytestmark = pytest.mark.gpu


def read_state(buf, dim, rank):
    raw = host(buf).tobytes()
    ld = (dim + 3) // 4 * 4
    R = np.frombuffer(raw, np.float32, rank * ld).reshape(rank, ld)
    off = rank * ld * 4
    d = np.frombuffer(raw, np.float64, rank, off)
    rho = np.frombuffer(raw, np.float64, 1, off + rank * 8)[0]
    t = np.frombuffer(raw, np.int64, 1, off + rank * 8 + 8)[0]
    sweeps, unconverged = np.frombuffer(raw, np.int32, 2, off + rank * 8 + 16)
    assert unconverged == 0 and 0 <= sweeps <= 14          # no fold so far ran out of Jacobi sweeps
    assert np.all(R[:, dim:] == 0)
    return R[:, :dim].astype(np.float64), d.copy(), float(rho), int(t)


def check_state(buf, dim, rank, ref, tol=2e-3, subspace_tol=None):
    R, d, rho, t = read_state(buf, dim, rank)
    assert t == ref.t
    np.testing.assert_allclose(R @ R.T, np.eye(rank), atol=2e-5)          # orthonormal rows
    sv = np.linalg.svd(R @ ref.R.T, compute_uv=False)                     # cosines of the principal angles
    # the least significant tracked direction is ill-conditioned when its eigenvalue is close to those of the
    # untracked directions (it may turn inside that cluster without changing the Fisher estimate): callers
    # with such spectra pass a looser subspace tolerance and rely on the Fisher probe below
    assert sv.min() > 1 - (tol if subspace_tol is None else subspace_tol)
    assert rel_err(d, ref.d) < tol and abs(rho - ref.rho) <= tol * max(abs(ref.rho), 1e-9)
    # the Fisher estimate itself, probed on random vectors (unique whatever basis R uses)
    rng = np.random.default_rng(0)
    V = rng.standard_normal((dim, 4))
    Fg = R.T @ (d[:, None] * (R @ V)) + rho * V
    Fo = ref.R.T @ (ref.d[:, None] * (ref.R @ V)) + ref.rho * V
    assert rel_err(Fg, Fo) < tol


def _data(n, dim, seed, t, lowrank=8):
    rng = np.random.default_rng([seed, t])
    scales = np.linspace(3.0, 0.3, dim)
    mix = np.random.default_rng(seed).standard_normal((lowrank, dim))
    return (rng.standard_normal((n, dim)) * scales[None, :] * 0.3 + rng.standard_normal((n, lowrank)) @ mix).astype(np.float32)


@pytest.mark.parametrize("n,dim,rank", [(37, 45, 5), (64, 130, 30), (100, 51, 7), (512, 441, 30), (512, 2049, 30), (512, 8000, 30),
                                        (96, 150, 33), (128, 200, 64)])    # odd rank above 32; the largest rank
def test_precondition_sequence_matches_oracle(n, dim, rank):
    import torch
    from paper_1507_01239_amd import binding as B
    eta = ngsgd.default_eta(n) if n >= 256 else 0.2
    st = torch.zeros(B.ngsgd_state_bytes(dim, rank), dtype=torch.uint8, device="cuda")
    B.ngsgd_state_init(st, dim, rank)
    ref = ngsgd.init_state(dim, rank)
    torch.cuda.synchronize()
    R0, d0, rho0, t0 = read_state(st, dim, rank)
    assert np.array_equal(R0, ref.R) and np.all(d0 == ngsgd.EPS) and rho0 == ngsgd.EPS and t0 == 0
    ws = workspace(B.ngsgd_workspace_bytes(dim, rank, n))
    ldx = (dim + 3) // 4 * 4 + 4                 # a padded leading dimension
    for t in range(4):
        X = _data(n, dim, 11, t)
        xb = torch.zeros(n, ldx, device="cuda")
        xb[:, :dim] = dev(X)
        B.ngsgd_precondition(st, dim, rank, xb, ldx, n, 4.0, eta, B.NG_INIT_UPDATE if t == 0 else B.NG_UPDATE, ws)
        torch.cuda.synchronize()
        out_ref, ref = ngsgd.precondition(ref, X, 4.0, eta, update=True)
        got = host(xb)
        assert np.all(got[:, dim:] == 0)
        assert rel_err(got[:, :dim], out_ref) < 1e-4, t
        assert abs(np.linalg.norm(got[:, :dim].astype(np.float64)) / np.linalg.norm(X.astype(np.float64)) - 1) < 1e-5
        check_state(st, dim, rank, ref)
    # apply-only leaves the state untouched
    before = host(st).copy()
    X = _data(n, dim, 11, 9)
    xb = dev(np.ascontiguousarray(np.pad(X, ((0, 0), (0, ldx - dim)))))
    B.ngsgd_precondition(st, dim, rank, xb, ldx, n, 4.0, eta, B.NG_APPLY, ws)
    torch.cuda.synchronize()
    out_ref, _ = ngsgd.precondition(ref, X, 4.0, eta, update=False)
    assert rel_err(host(xb)[:, :dim], out_ref) < 1e-4
    assert np.array_equal(host(st), before)


# one index, one pair, the last odd and the full group of 32 lanes, the first rank of the 64-lane groups, an odd one there
@pytest.mark.parametrize("n,dim,rank", [(64, 41, 1), (64, 41, 2), (64, 100, 31), (64, 100, 32), (128, 200, 63)])
def test_eigen_solver_at_the_edges_of_its_groups(n, dim, rank):
    test_precondition_sequence_matches_oracle(n, dim, rank)


# One launch decomposes and finishes the apply in slabs of 32 rows and blocks of 32 columns: edges of both, rows that no vector load
# may touch (ldx not a multiple of 4), both sizes of the rank
@pytest.mark.parametrize("n,dim,rank,pad", [(1, 20, 3, 0), (31, 33, 8, 0), (32, 32, 5, 4), (33, 65, 30, 1), (65, 130, 31, 2), (97, 257, 32, 3), (70, 99, 40, 1), (256, 300, 64, 0)])
def test_updating_call_applies_as_the_other_one_does(n, dim, rank, pad):
    import torch
    from paper_1507_01239_amd import binding as B
    st = torch.zeros(B.ngsgd_state_bytes(dim, rank), dtype=torch.uint8, device="cuda")
    B.ngsgd_state_init(st, dim, rank)
    ws = workspace(B.ngsgd_workspace_bytes(dim, rank, max(n, 128)))
    x0 = torch.zeros(128, dim, device="cuda")
    x0[:] = dev(_data(128, dim, 5, 0))
    B.ngsgd_precondition(st, dim, rank, x0, dim, 128, 4.0, 0.2, B.NG_INIT_UPDATE, ws)
    outs = []
    for mode in (B.NG_APPLY, B.NG_UPDATE):
        x = torch.full((n, dim + pad), 7.0, device="cuda")
        x[:, :dim] = dev(_data(n, dim, 5, 1))
        B.ngsgd_precondition(st, dim, rank, x, dim + pad, n, 4.0, 0.2, mode, ws)
        torch.cuda.synchronize()
        assert (x[:, dim:] == 7.0).all()
        outs.append(host(x)[:, :dim].astype(np.float64))
    # float32 products in another order; what is left after two projections is amplified by ||X|| / ||Xh||
    X = _data(n, dim, 5, 1).astype(np.float64)
    assert np.abs(outs[1] - outs[0]).max() <= 1e-4 * np.abs(outs[0]).max()
    assert abs(np.linalg.norm(outs[1]) / np.linalg.norm(X) - 1) < 1e-5


def test_ngsgd_validation_on_device_side_arguments():
    from paper_1507_01239_amd import binding as B
    A = 1 << 20
    rc = lambda *a, **k: B.lib.ngsgd_precondition(*a)
    assert B.lib.ngsgd_state_bytes(30, 30) == B.E_DIM
    assert B.lib.ngsgd_state_bytes(31, 65) == B.E_DIM
    assert B.lib.ngsgd_precondition(None, 40, 4, A, 40, 8, 4.0, 0.1, 1, A, 1 << 30, None) == B.E_NULL
    assert B.lib.ngsgd_precondition(A, 40, 4, A, 39, 8, 4.0, 0.1, 1, A, 1 << 30, None) == B.E_ALIGN
    assert B.lib.ngsgd_precondition(A, 40, 4, A, 40, 8, 4.0, 0.1, 3, A, 1 << 30, None) == B.E_FLAG
    assert B.lib.ngsgd_precondition(A, 40, 4, A, 40, 8, 4.0, 1.5, 1, A, 1 << 30, None) == B.E_DIM
    assert B.lib.ngsgd_precondition(A, 40, 4, A, 40, 8, 4.0, 0.1, 1, A, 16, None) == B.E_WORKSPACE


class NgGpu:
    def __init__(self, dims, k, n, theta0, rank):
        import torch
        from paper_1507_01239_amd import binding as B
        self.B, self.torch, self.dims, self.k, self.n, self.rank = B, torch, dims, k, n, rank
        self.shape = B.Shape(dims)
        self.P = B.mavg_param_count(self.shape)
        self.stride = (self.P + 63) // 64 * 64
        self.act_stride = (B.mavg_act_count(self.shape, n) + 63) // 64 * 64
        self.theta = torch.zeros(k, self.stride, device="cuda")
        self.theta[:, :self.P] = dev(theta0)[None, :]
        self.acts = torch.empty(k, self.act_stride, device="cuda")
        self.flags = B.MEAN_GRAD | B.USE_NGSGD
        self.ws = workspace(B.mavg_workspace_bytes(self.shape, n, k, self.flags, rank))
        self.loss = torch.zeros(k, device="cuda")
        L = len(dims) - 1
        self.sb = B.ngsgd_state_bytes(max(max(dims[:-1]) + 1, max(dims[1:])) + 1, rank)
        self.states = torch.zeros(k * 2 * L, self.sb, dtype=torch.uint8, device="cuda")
        for r in range(k):
            for l in range(1, L + 1):
                B.ngsgd_state_init(self.states[(r * 2 * L) + 2 * (l - 1)], dims[l - 1] + 1, rank)
                B.ngsgd_state_init(self.states[(r * 2 * L) + 2 * (l - 1) + 1], dims[l], rank)
        self.first = True

    def step(self, X, Y, lr, eta, fold=True):
        B = self.B
        x = dev(X.reshape(self.k, -1))
        y = dev(Y.reshape(self.k, -1).astype(np.int32))
        B.dnn_forward(self.shape, self.k, self.theta, self.stride, x, x.shape[1], self.n, self.acts, self.act_stride, self.ws)
        B.dnn_backward_update(self.shape, self.k, self.theta, self.stride, x, x.shape[1], y, y.shape[1], self.n, self.acts,
                              self.act_stride, lr,
                              self.flags | (B.NG_FIRST if self.first else 0) | (0 if (fold or self.first) else B.NG_APPLY_ONLY),
                              self.loss, self.ws,
                              ng_state=self.states, ng_state_stride=self.sb, ng_rank=self.rank, ng_alpha=4.0, ng_eta=eta)
        self.first = False

    def params(self):
        self.torch.cuda.synchronize()
        return host(self.theta[:, :self.P])

    def probe_update(self, X, Y, lr_big, eta, fold=True):
        """The update lr_big * (preconditioned gradient) this step would make, without making it: float32
        parameters resolve a step of the trajectory's own small learning rate only to about 1e-3 of its
        norm, so the step is taken once with a large power-of-two learning rate on a copy and undone."""
        theta, states, first = self.theta.clone(), self.states.clone(), self.first
        self.step(X, Y, lr_big, eta, fold)
        upd = self.params().astype(np.float64) - host(theta[:, :self.P]).astype(np.float64)
        self.theta.copy_(theta)
        self.states.copy_(states)
        self.first = first
        return upd

    def average(self):
        self.B.replicas_average(self.theta, self.stride, self.P, self.k)

    def state_blob(self, st, dim):
        """Bytes of a device state holding the oracle state st (R rounded to float32)."""
        ld = (dim + 3) // 4 * 4
        R = np.zeros((self.rank, ld), np.float32)
        R[:, :dim] = st.R
        raw = R.tobytes() + np.asarray(st.d, np.float64).tobytes() + np.float64(st.rho).tobytes() + np.int64(st.t).tobytes()
        raw += np.zeros(2, np.int32).tobytes()
        return np.frombuffer(raw + bytes(self.sb - len(raw)), np.uint8)

    def probe_update_from(self, thetas, states, X, Y, lr_big, eta):
        """As probe_update, but teacher-forced: the step starts from the given parameters (K x P) and oracle states
        (states[k] = (input-side list, output-side list)) instead of the device's own; those are restored afterwards.
        Returns the update and the float32 parameters it started from."""
        L = len(self.dims) - 1
        keep_theta, keep_states, keep_first = self.theta.clone(), self.states.clone(), self.first
        blobs = np.zeros((self.k * 2 * L, self.sb), np.uint8)
        for k in range(self.k):
            for l in range(1, L + 1):
                blobs[k * 2 * L + 2 * (l - 1)] = self.state_blob(states[k][0][l - 1], self.dims[l - 1] + 1)
                blobs[k * 2 * L + 2 * (l - 1) + 1] = self.state_blob(states[k][1][l - 1], self.dims[l])
        self.states.copy_(dev(blobs))
        start = np.asarray(thetas, np.float32)
        self.theta[:, :self.P] = dev(start)
        self.first = False
        self.step(X, Y, lr_big, eta)
        upd = self.params().astype(np.float64) - start.astype(np.float64)
        self.theta.copy_(keep_theta)
        self.states.copy_(keep_states)
        self.first = keep_first
        return upd, start


def _oracle_states(dims, rank):
    return ([ngsgd.init_state(dims[l - 1] + 1, rank) for l in range(1, len(dims))],
            [ngsgd.init_state(dims[l], rank) for l in range(1, len(dims))])


def _oracle_probe(dims, theta, batch, lr_big, eta, s_in, s_out, fold=True):
    """Oracle counterpart of NgGpu.probe_update for one replica: the step from (theta, states) on copies of the states."""
    pre = ngsgd.make_layer_preconditioner([s.copy() for s in s_in], [s.copy() for s in s_out], 4.0, eta, update=fold)
    new, _, _ = dnn.sgd_step(theta, dims, batch[0], batch[1], lr_big, precondition=pre)
    return new - theta


def check_update_tensors(upd_gpu, upd_ref, dims, tol, what):
    worst = 0.0
    for l, ((Wg, bg), (Wr, br)) in enumerate(zip(dnn.unpack(upd_gpu, dims), dnn.unpack(upd_ref, dims)), start=1):
        worst = max(worst, check_close(Wg, Wr, tol, f"{what} W{l}")[0], check_close(bg, br, tol, f"{what} b{l}")[0])
    return worst


def _run_small_ng_case(dims, K, n, lr, rank, eta, seed, fold):
    """Trajectory of len(fold) minibatches on K replicas against the oracle: before every step the preconditioned
    update itself within 1e-4 per tensor (probe at learning rate 64), after it the parameters within 1e-5."""
    T = len(fold)
    theta0 = gen.init_theta(dims, seed, 0.1)
    shards = [[(gen.features_iid(n, dims[0], seed, k, t), gen.labels_uniform(n, dims[-1], seed, k, t)) for t in range(T)]
              for k in range(K)]
    g = NgGpu(dims, K, n, theta0, rank)
    L = len(dims) - 1
    th = [theta0.astype(np.float64) for _ in range(K)]
    st = [_oracle_states(dims, rank) for _ in range(K)]
    worst = 0.0
    for t in range(T):
        X = np.stack([shards[k][t][0] for k in range(K)])
        Y = np.stack([shards[k][t][1] for k in range(K)])
        upd = g.probe_update(X, Y, 64.0, eta, fold[t])
        for k in range(K):
            ref = _oracle_probe(dims, th[k], shards[k][t], 64.0, eta, st[k][0], st[k][1], fold[t])
            worst = max(worst, check_update_tensors(upd[k], ref, dims, 1e-4, f"minibatch {t}, replica {k}, update"))
        before = host(g.states).copy() if not fold[t] else None
        g.step(X, Y, lr, eta, fold=fold[t])
        got = g.params()
        if not fold[t]:
            assert np.array_equal(host(g.states), before)          # apply-only leaves every state bit for bit
        for k in range(K):
            pre = ngsgd.make_layer_preconditioner(st[k][0], st[k][1], 4.0, eta, update=fold[t])
            th[k], _, _ = dnn.sgd_step(th[k], dims, shards[k][t][0], shards[k][t][1], lr, precondition=pre)
            assert rel_err(got[k], th[k]) < 1e-5
    for k in range(K):
        for l in range(1, L + 1):
            check_state(g.states[k * 2 * L + 2 * (l - 1)], dims[l - 1] + 1, rank, st[k][0][l - 1], tol=5e-3)
            check_state(g.states[k * 2 * L + 2 * (l - 1) + 1], dims[l], rank, st[k][1][l - 1], tol=5e-3)
    print(f"worst per-tensor relative error of a preconditioned update: {worst:.2e}")


def _oracle_ng_run(dims, theta0, shards, lr, rank, eta, fold=None):
    # fold[t] False: minibatch t is preconditioned with the states as they are and not folded into them
    K, T = len(shards), len(shards[0])
    out = []
    for k in range(K):
        s_in = [ngsgd.init_state(dims[l - 1] + 1, rank) for l in range(1, len(dims))]
        s_out = [ngsgd.init_state(dims[l], rank) for l in range(1, len(dims))]
        pre = ngsgd.make_layer_preconditioner(s_in, s_out, 4.0, eta)
        pre_apply = ngsgd.make_layer_preconditioner(s_in, s_out, 4.0, eta, update=False)      # same state lists
        th = theta0.astype(np.float64)
        traj = []
        for t in range(T):
            p_t = pre if (fold is None or fold[t]) else pre_apply
            th, _, _ = dnn.sgd_step(th, dims, shards[k][t][0], shards[k][t][1], lr, precondition=p_t)
            traj.append(th.copy())
        out.append((traj, s_in, s_out))
    return out


def test_ng_training_step_tiny_two_replicas():
    _run_small_ng_case(gen.CONFIG_TINY_DIMS, 2, 32, 0.1, 8, 0.2, 5, [True] * 4)


def test_ng_training_step_mixed_widths_rank_above_32():
    # Layer sides of very different widths in the same launches: 1601 (its thin product cut into two chunks of the
    # contraction), 91 / 200 / 201 / 1600 (one chunk, ragged tails), 48 (too short for the in-workgroup split: launched
    # by itself); rank 36 takes the two-half path of the rank update and 64-lane groups in the eigen-solver;
    # 96 rows = 3 row tiles; two replicas.
    _run_small_ng_case([90, 200, 1600, 48], 2, 96, 0.05, 36, 0.2, 9, [True] * 3)


def test_ng_training_with_folds_on_some_minibatches_only():
    # the states are folded on minibatches 0, 1 and 4 only; 2, 3 and 5 are preconditioned with the states as they are
    _run_small_ng_case([70, 130, 96, 40], 2, 64, 0.05, 12, 0.2, 13, [True, True, False, False, True, False])


def test_ng_training_step_ragged_row_tiles():
    # 45 rows = one whole tile of 32 rows and a ragged one, in the rank update that also takes H^T X for the fold;
    # widths 53 / 68 / 69 / 36 leave ragged column blocks as well
    _run_small_ng_case([52, 68, 36], 2, 45, 0.05, 7, 0.2, 21, [True] * 3)


def test_ng_training_step_ragged_row_tiles_rank_above_32():
    # the same with rank 34: two MFMA halves per operand in the rank updates and in the product H^T X
    _run_small_ng_case([52, 100, 44], 1, 45, 0.05, 34, 0.2, 27, [True] * 2)


def test_ng_training_step_on_the_split_operand_update():
    # 263 rows (a partial k-tile) and layers wide enough for the split-operand kernel of the grouped update, whose row sums
    # are then weighted by the preconditioned "ones" column: the biases of the second step
    from paper_1507_01239_amd import binding as B
    dims, n = [520, 4100, 4100], 263
    A = 1 << 20
    probs = [B.gemm_problem(A, dims[l], A, (dims[l - 1] + 32) // 32 * 32, A, dims[l - 1], dims[l], dims[l - 1], n, epi=4) for l in (1, 2)]
    assert [B.mavg_gemm_grouped_kernel(probs, 0, 0, i) for i in (0, 1)] == [0, 0]
    _run_small_ng_case(dims, 1, n, 0.05, 8, 0.2, 31, [True] * 2)


def test_ng_training_step_many_row_blocks():
    # 1100 rows: more blocks of rows than a backward pass keeps partial products H^T X for, so Y is formed by the
    # pass of its own over X (and its last tile of rows is ragged)
    _run_small_ng_case([30, 44, 20], 1, 1100, 0.05, 6, 0.2, 23, [True] * 2)


def test_config5_ng_full_size_two_steps():
    # 440-6x2048-8000, minibatch 512, rank 30, one replica, two minibatches
    dims, n, lr, rank, seed = gen.CONFIG_FULL_DIMS, 512, 0.008, 30, 41
    eta = ngsgd.default_eta(n)
    theta0 = gen.init_theta(dims, seed, 0.05)
    shards = [[(gen.features_speech_like(n, dims[0], seed, 0, t), gen.labels_zipf(n, dims[-1], seed, 0, t)) for t in range(2)]]
    ref = _oracle_ng_run(dims, theta0, shards, lr, rank, eta)
    g = NgGpu(dims, 1, n, theta0, rank)
    for t in range(2):
        g.step(shards[0][t][0][None], shards[0][t][1][None], lr, eta)
        assert rel_err(g.params()[0], ref[0][0][t]) < 1e-5
    L = len(dims) - 1
    for l in range(1, L + 1):
        check_state(g.states[2 * (l - 1)], dims[l - 1] + 1, rank, ref[0][1][l - 1], tol=5e-3, subspace_tol=0.05)
        check_state(g.states[2 * (l - 1) + 1], dims[l], rank, ref[0][2][l - 1], tol=5e-3, subspace_tol=0.05)
    # the preconditioned update itself, resolved with a learning rate large enough for float32 parameters
    big = 8.0
    ref1 = _oracle_ng_run(dims, theta0, [shards[0][:1]], big, rank, eta)
    g1 = NgGpu(dims, 1, n, theta0, rank)
    g1.step(shards[0][0][0][None], shards[0][0][1][None], big, eta)
    upd_gpu = g1.params()[0].astype(np.float64) - theta0
    upd_ref = ref1[0][0][0] - theta0
    # per-step gradients within 1e-4 relative, per tensor (measured worst: 6e-5).  This needs the folds that
    # start from the initial state in float64 and the tracked subspace projected out twice: the hidden
    # activations lie almost entirely along one direction (||X||/||Xh|| is about 120).
    worst = 0.0
    for (Wg, bg), (Wr, br) in zip(dnn.unpack(upd_gpu, dims), dnn.unpack(upd_ref, dims)):
        worst = max(worst, rel_err(Wg, Wr), rel_err(bg, br))
    print(f"NG-SGD full-size update, worst per-tensor relative error {worst:.2e}")
    assert worst < 1e-4


def test_config5_eight_replicas_ng_sgd_averaged_every_five():
    # Sec. 4 (eq. 4) together with Sec. 3 (eq. 2), the combination of Sec. 5.7: 8 replicas of the full-size
    # network, NG-SGD of rank 30 at minibatch 512, parameters averaged every 5 minibatches, two averaging periods.
    # The parameters are averaged; the 14 Fisher states of each replica are NOT (eq. 2 averages theta only) and
    # keep following their own replica's data.  The oracle side is the loop of oracle.averaging.train_with_averaging
    # written out, so that the states of the moment are at hand for the probe of a single update.
    dims, K, n, lr, rank, seed, T, n_avg = gen.CONFIG_FULL_DIMS, 8, 512, 0.008, 30, 61, 10, 5
    eta = ngsgd.default_eta(n)
    L = len(dims) - 1
    theta0 = gen.init_theta(dims, seed, 0.05)
    st = [_oracle_states(dims, rank) for _ in range(K)]
    pre = [ngsgd.make_layer_preconditioner(st[k][0], st[k][1], 4.0, eta) for k in range(K)]
    th = np.tile(theta0.astype(np.float64), (K, 1))
    g = NgGpu(dims, K, n, theta0, rank)
    for t in range(T):
        batch = [(gen.features_speech_like(n, dims[0], seed, k, t), gen.labels_zipf(n, dims[-1], seed, k, t)) for k in range(K)]
        X = np.stack([b[0] for b in batch])
        Y = np.stack([b[1] for b in batch])
        if t == n_avg:
            # First step after an averaging: the preconditioned update by itself, per tensor (first and last replica).
            # (i) Teacher-forced, the per-step bar of 1e-4: device and oracle start from the same parameters and the
            #     same Fisher states (the oracle's, R rounded to float32).
            upd, start = g.probe_update_from(th, st, X, Y, 8.0, eta)
            for k in (0, K - 1):
                s32 = tuple([ngsgd.NGState(s.R.astype(np.float32).astype(np.float64), s.d, s.rho, s.t) for s in side] for side in st[k])
                want = _oracle_probe(dims, start[k].astype(np.float64), batch[k], 8.0, eta, s32[0], s32[1])
                worst = check_update_tensors(upd[k], want, dims, 1e-4, f"replica {k}, minibatch {t}, teacher-forced update")
                print(f"replica {k}: teacher-forced update after the first averaging, worst tensor {worst:.2e}")
            # (ii) Free-running: each side from its own parameters and its own states after five folds (which agree
            #      to the tolerance of check_state, not bit for bit), so this is held to the several-steps bar.
            upd = g.probe_update(X, Y, 8.0, eta)
            for k in (0, K - 1):
                want = _oracle_probe(dims, th[k], batch[k], 8.0, eta, st[k][0], st[k][1])
                worst = check_update_tensors(upd[k], want, dims, 1e-3, f"replica {k}, minibatch {t}, free-running update")
                print(f"replica {k}: free-running update after the first averaging, worst tensor {worst:.2e}")
        g.step(X, Y, lr, eta)
        losses = np.zeros(K)
        for k in range(K):
            th[k], losses[k], _ = dnn.sgd_step(th[k], dims, batch[k][0], batch[k][1], lr, precondition=pre[k])
        assert np.allclose(host(g.loss), losses, rtol=1e-3), t
        if (t + 1) % n_avg == 0:
            th = averaging.average_replicas(th)
            g.average()
            got = g.params()
            assert all(np.array_equal(got[0], got[r]) for r in range(1, K))      # every replica holds the mean
            for l, ((Wg, bg), (Wr, br)) in enumerate(zip(dnn.unpack(got[0].astype(np.float64), dims), dnn.unpack(th[0], dims)), start=1):
                check_close(Wg, Wr, 1e-3, f"W{l} after minibatch {t}")
                check_close(bg, br, 1e-3, f"b{l} after minibatch {t}")
    # the states: each replica's own, compared with the oracle's for that replica, and different between replicas
    for k in range(K):
        for l in range(1, L + 1):
            check_state(g.states[k * 2 * L + 2 * (l - 1)], dims[l - 1] + 1, rank, st[k][0][l - 1], tol=5e-3, subspace_tol=0.05)
            check_state(g.states[k * 2 * L + 2 * (l - 1) + 1], dims[l], rank, st[k][1][l - 1], tol=5e-3, subspace_tol=0.05)
    raw = host(g.states)
    for k in range(1, K):
        for j in range(2 * L):
            assert not np.array_equal(raw[k * 2 * L + j], raw[j]), (k, j)          # not averaged, not shared
