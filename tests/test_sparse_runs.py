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
