"""Runs over wide sparse data: what a session asks of the GPU's memory, and whole passes against the same pass in parts."""
import numpy as np
import pytest
import torch

from paper_1902_01064_amd import hop, inputs
from paper_1902_01064_amd.session import Session

pytestmark = pytest.mark.gpu


def _config(d, **over):
    nb = inputs.torus(4, 4)
    return dict(inputs.config(3, d=d, rows=256), in_nbrs=nb, W=inputs.uniform_weights(nb), N=16, s=3, b=1, batch=32, K=12, mult=None,
                loss=1, **over)


def test_one_gradient_buffer_per_worker():
    """The sparse part of a gradient is scattered into the result: a session asks for no more than the least."""
    c = _config(1 << 20)
    sess = Session(c)
    try:
        assert sess.arena.numel() * 4 == hop.hop_arena_bytes(16, c["d"], c["s"], c["b"], hop.make_opts(batch=c["batch"], max_ig=c["max_ig"]))
    finally:
        sess.close()


def _data(seed, rows, d):
    """Rows of no, one, 64, 65 and 130 non-zeros, columns ascending."""
    r = np.random.default_rng(seed)
    n = r.choice([0, 1, 64, 65, 130], size=rows)
    col = np.concatenate([np.sort(r.choice(d, size=k, replace=False)) for k in n] + [np.zeros(0)])
    rowptr = np.concatenate([[0], np.cumsum(n)])
    t = lambda a, k: torch.from_numpy(a.astype(k)).cuda()  # noqa: E731
    return t(rowptr, np.int64), t(col, np.int32), t(r.standard_normal(len(col)), np.float32), t(r.choice([-1.0, 1.0], size=rows), np.float32)


@pytest.mark.parametrize("graphed", [False, True])
@pytest.mark.parametrize("ahead", [1, 6])
def test_whole_pass_as_in_parts(graphed, ahead):
    """Columns that no row of the pass holds are the same bits, on the others the scatter's atomics leave rounding, and nothing is
    kept in the gradient buffers, however many the caller lends.  Two passes: the second over other columns in the same arrays."""
    d = (1 << 18) + 65
    c = _config(d, grad_ahead=ahead)
    data = [_data(i, 256, d) for i in range(16)]
    p0 = 0.1 * torch.randn(16, d, generator=torch.Generator(device="cuda").manual_seed(2), device="cuda")
    both = [Session(c) for _ in range(2)]
    try:
        for sess in both:
            sess.set_csr(data)
            sess.set_params(p0)
            sess.simulate()
        whole, parts = both
        hop.hop_use_graph(whole.ctx, int(graphed))
        held = torch.zeros(d, dtype=torch.bool, device="cuda")
        n = parts.sched.n_waves
        for rep in range(2):
            whole.step()
            parts.step(0, n // 2)
            parts.step(n // 2, n)
            whole.sync()
            for rowptr, col, _, _ in data:
                held[col.long()] = True
            a, b = [s.arena[:16 * s.D * s.stride].view(16, s.D, s.stride)[:, :, :d] for s in both]
            assert torch.equal(a[:, :, ~held], b[:, :, ~held])
            a, b = a[:, :, held].double(), b[:, :, held].double()
            # an atomic sum of up to 32 batch terms in another order, over up to 40 records: far below 1e-5 of the largest entry
            assert float((a - b).abs().max()) <= 1e-5 * float(b.abs().max())
            buffers = whole.arena[16 * whole.D * whole.stride:16 * (whole.D + ahead) * whole.stride]
            assert not bool(buffers.any())
            for _, col, _, _ in data:
                col.copy_(d - 1 - col)
    finally:
        for sess in both:
            sess.close()


# Rows of a workgroup of the scatter (16), its four blocks of margins (4 rows), and their number over a wave's records around the
# multiples of the XCDs: every coefficient is that of its own row, and the results are the records' sums
@pytest.mark.parametrize("N,B", [(1, 1), (1, 129), (3, 5), (7, 16), (8, 17), (9, 32), (16, 4), (16, 33), (64, 1), (64, 8), (64, 15)])
@pytest.mark.parametrize("momentum", [0.0, 0.9])
def test_margins_of_small_minibatches(N, B, momentum):
    d = 3001
    nb = [[]] if N == 1 else inputs.ring(N)
    c = dict(inputs.config(3, d=d, rows=300, K=1), in_nbrs=nb, W=inputs.uniform_weights(nb), N=N, s=0, b=0, batch=B, loss=1, lam=0.25,
             lr=0.5, momentum=momentum, skip_on=False, mult=None, delay_kind=inputs.DELAY_NONE)
    data = [_data(100 + i, 300, d) for i in range(N)]
    p0 = torch.randn(N, d, generator=torch.Generator(device="cuda").manual_seed(8), device="cuda") / 8
    print("small minibatches", N, B, momentum, flush=True)
    sess = Session(c)
    try:
        sess.set_csr(data)
        sess.set_params(p0)
        s = sess.simulate()
        assert s.n_waves == 1 and s.n_records == N
        sess.step()
        sess.sync()
        for e in range(N):
            i, ids = int(s.worker[e]), s.batch_rows[e]
            rowptr, col, val, y = data[i]
            w, X = p0[i].double(), torch.zeros(B, d, dtype=torch.float64, device="cuda")
            ends = rowptr.cpu().numpy()
            for m, r in enumerate(ids):
                X[m, col[ends[r]:ends[r + 1]].long()] = val[ends[r]:ends[r + 1]].double()
            t = y[torch.from_numpy(ids.copy()).cuda().long()].double()
            coef = torch.from_numpy(sess.coef(e)).cuda().double()
            # the slope of a coefficient in its margin is at most 1 / 4 B; a sum of up to 130 products is off by 131 * 2^-24 of them
            off = 131 * 2.0 ** -24 * (X.abs() @ w.abs())
            want = t / (B * (1 + torch.exp(t * (X @ w))))
            assert bool(((coef - want).abs() <= (0.25 * off + 1e-6) / B).all())
            mag = 0.25 * w.abs() + coef.abs() @ X.abs()
            acc = -0.5 * (0.25 * w - coef @ X)
            size = torch.zeros_like(acc)
            for a in range(int(s.src_begin[e]), int(s.src_begin[e + 1])):
                x = float(s.src_weight[a]) * p0[int(s.src_worker[a])].double()
                acc, size = acc + x, size + x.abs()
            got = sess.slot(i, int(s.out_slot[e])).double()
            assert bool(((got - acc).abs() <= 2.0 ** -24 * (0.5 * (B + 4) * mag + 8 * size)).all())
    finally:
        sess.close()


# A call by itself: edges of the margins' blocks (4 rows) and of the scatter's (16), and of the columns that it adds up first (1024)
@pytest.mark.parametrize("d", [600, 1024, 1025, 70001])
@pytest.mark.parametrize("B", [1, 4, 5, 16, 17, 33, 129, 1024])
def test_gradient_by_itself(d, B):
    """Every row's coefficient and every column against 64 bits.  A margin is off by at most (n + 5) 2^-24 sum |x w| with n = 130 terms, a
    coefficient by a quarter of that and 8 roundings, a column by the rounding of its terms and by its rows' coefficients."""
    rows, lam, eps = 300, 1e-3, 2.0 ** -24
    rowptr, col, val, y = _data(d + B, rows, d)
    gen = torch.Generator().manual_seed(B)
    w = (0.1 * torch.randn(d, generator=gen)).cuda()
    ids = torch.randint(0, rows, (B,), generator=gen).int().cuda()
    g, coef = torch.full((d,), 7.0, device="cuda"), torch.full((B,), 7.0, device="cuda")
    hop.hop_svm_grad_csr(rowptr.data_ptr(), col.data_ptr(), val.data_ptr(), y.data_ptr(), w.data_ptr(), ids.data_ptr(), B, d, lam, g.data_ptr(),
                         coef.data_ptr(), torch.cuda.current_stream().cuda_stream, hop.HOP_LOSS_LOG)
    torch.cuda.synchronize()
    x = torch.zeros(rows, d, dtype=torch.float64, device="cuda")
    of_row = torch.repeat_interleave(torch.arange(rows, device="cuda"), rowptr[1:] - rowptr[:-1])
    x[of_row, col.long()] = val.double()
    x, yd, wd = x[ids.long()], y[ids.long()].double(), w.double()
    want = yd / (B * (1 + torch.exp(yd * (x @ wd))))
    off = ((130 + 5) * eps * (x.abs() @ wd.abs()) / 4 + 8 * eps) / B
    assert bool(((coef.double() - want).abs() <= off).all())
    lam = float(np.float32(lam))
    terms = (x != 0).sum(0) + 1
    mag = lam * wd.abs() + want.abs() @ x.abs()
    assert bool(((g.double() - (lam * wd - want @ x)).abs() <= (terms + 3) * eps * mag + off @ x.abs()).all())
