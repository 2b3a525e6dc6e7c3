"""Dense SVM gradients where a row is one segment of 16384 columns (the margins leave the coefficients) and just beyond it (the
gradient kernel works them out from partial products): stand-alone and in a run, against 64 bits."""
import pytest
import torch

from paper_1902_01064_amd import hop, inputs
from paper_1902_01064_amd.session import Session

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1, 255, 16383, 16384, 16385])
@pytest.mark.parametrize("B", [1, 65, 1024])
@pytest.mark.parametrize("loss", [hop.HOP_LOSS_HINGE, hop.HOP_LOSS_LOG])
def test_gradient_and_coefficients(d, B, loss):
    gen = torch.Generator(device="cuda").manual_seed(d + B)
    X = torch.randn(80, d, generator=gen, device="cuda")
    y = torch.sign(torch.randn(80, generator=gen, device="cuda"))
    w = 1.5 * torch.randn(d, generator=gen, device="cuda") / d ** 0.5
    rows = torch.randint(0, 80, (B,), generator=gen, device="cuda", dtype=torch.int32)
    x, yy, lam = X[rows.long()].double(), y[rows.long()].double(), 0.25
    m = yy * (x @ w.double())
    want = yy / (B * (1 + torch.exp(m))) if loss == hop.HOP_LOSS_LOG else torch.where(m < 1, yy, 0.0) / B
    # a sum of d products of fp32 numbers is within (d + 1) 2^-24 of the sum of their magnitudes; a hinge that close may turn over
    off = (d + 1) * 2.0 ** -24 * (x.abs() @ w.double().abs())
    for alloc in (True, False):
        g, coef = torch.empty(d, device="cuda"), torch.full((B,), 7.0, device="cuda")
        args = (X.data_ptr(), y.data_ptr(), w.data_ptr(), rows.data_ptr(), B, d, lam, g.data_ptr(), coef.data_ptr())
        if alloc:
            scratch = torch.empty(hop.hop_grad_scratch_floats(d, B), device="cuda")
            hop.hop_svm_grad_dense(*args, scratch.data_ptr(), torch.cuda.current_stream().cuda_stream, loss)
        else:
            hop.hop_svm_grad_dense_static(*args, torch.cuda.current_stream().cuda_stream, loss)
        c = coef.double()
        if loss == hop.HOP_LOSS_LOG:                       # the slope of the coefficient in the margin is at most 1 / 4 B
            assert bool(((c - want).abs() <= (0.25 * off + 1e-6) / B).all())
        else:
            assert bool(((c - want).abs() <= 2.0 ** -24 / B)[(m - 1).abs() > off].all())
        ref = lam * w.double() - c @ x
        room = (B + 3) * 2.0 ** -24 * (lam * w.double().abs() + c.abs() @ x.abs())
        assert bool(((g.double() - ref).abs() <= room + 1e-30).all())


@pytest.mark.parametrize("d", [16384, 16385])
@pytest.mark.parametrize("momentum", [0.0, 0.9])
def test_coefficients_of_a_run(d, momentum):
    """Both ways a wave runs its gradients: margins beside the Reduce (8 rows) and ahead of it (64 rows)."""
    nb = inputs.ring(4)
    for B in (8, 64):
        c = dict(inputs.config(1, d=d, rows=96, K=3), in_nbrs=nb, W=inputs.uniform_weights(nb), N=4, batch=B, loss=1, momentum=momentum)
        ws = inputs.hidden_w(5, d, "cuda")
        data = [inputs.dense_svm_data(5, i, 96, d, ws, "cuda") for i in range(4)]
        p0 = 0.01 * torch.randn(d, generator=torch.Generator().manual_seed(1))
        sess = Session(c)
        try:
            sess.set_dense([x for x, _ in data], [y for _, y in data])
            sess.set_params(p0)
            s = sess.simulate()
            sess.step()
            for e in range(s.n_records):
                if int(s.iter[e]) == 0:                    # at p0, whatever came after
                    i, ids = int(s.worker[e]), torch.from_numpy(s.batch_rows[e].copy()).cuda().long()
                    X, y = data[i][0][ids].double(), data[i][1][ids].double()
                    want = y / (B * (1 + torch.exp(y * (X @ p0.cuda().double()))))
                    got = torch.from_numpy(sess.coef(e)).cuda().double()
                    assert float((got - want).abs().max()) <= 1e-5 / B
        finally:
            sess.close()


# one wave of all workers.  752, 1024 and 2304 chunks of 256 columns: 8 or 4 wavefronts share a chunk's rows, or chunks of 1024
# columns with the rows whole; 208, 512 and 900 workgroups of four rows: one row each in the first, four in the others
@pytest.mark.parametrize("side,d,B", [(4, 12001, 50), (4, 16384, 128), (6, 16383, 100)])
@pytest.mark.parametrize("momentum", [0.0, 0.9])
def test_large_waves_of_one_segment(side, d, B, momentum):
    """Coefficients and results of a wave against 64 bits, from them the gradient (log loss: no sample leaves the sum)."""
    N, nb = side * side, inputs.torus(side, side)
    c = dict(inputs.config(1, d=d, rows=160, K=1), in_nbrs=nb, W=inputs.uniform_weights(nb), N=N, s=0, b=0, batch=B, loss=1, lam=0.25,
             lr=0.5, momentum=momentum, skip_on=False, mult=None, delay_kind=inputs.DELAY_NONE)
    ws = inputs.hidden_w(6, d, "cuda")
    data = [inputs.dense_svm_data(6, i, 160, d, ws, "cuda") for i in range(N)]
    p0 = torch.randn(N, d, generator=torch.Generator(device="cuda").manual_seed(4), device="cuda") / d ** 0.5
    sess = Session(c)
    try:
        sess.set_dense([x for x, _ in data], [y for _, y in data])
        sess.set_params(p0)
        s = sess.simulate()
        assert s.n_waves == 1 and s.n_records == N
        sess.step()
        sess.sync()
        for e in range(N):
            i, ids = int(s.worker[e]), torch.from_numpy(s.batch_rows[e].copy()).cuda().long()
            X, y = data[i][0][ids].double(), data[i][1][ids].double()
            coef = torch.from_numpy(sess.coef(e)).cuda().double()
            # the slope of a coefficient in its margin is at most 1 / 4 B; a sum of d products is off by (d + 1) 2^-24 of their magnitudes
            off = (d + 1) * 2.0 ** -24 * (X.abs() @ p0[i].double().abs())
            want = y / (B * (1 + torch.exp(y * (X @ p0[i].double()))))
            assert bool(((coef - want).abs() <= (0.25 * off + 1e-6) / B).all())
            g = 0.25 * p0[i].double() - coef @ X
            mag = 0.25 * p0[i].double().abs() + coef.abs() @ X.abs()
            acc, size = torch.zeros_like(g), torch.zeros_like(g)
            for a in range(int(s.src_begin[e]), int(s.src_begin[e + 1])):
                x = float(s.src_weight[a]) * p0[int(s.src_worker[a])].double()
                acc, size = acc + x, size + x.abs()
            got = sess.slot(i, int(s.out_slot[e])).double()
            room = 2.0 ** -24 * (0.5 * (B + 4) * mag + 8 * size)        # B + 1 products, five sources and the step
            assert bool(((got - (acc - 0.5 * g)).abs() <= room).all())
    finally:
        sess.close()
