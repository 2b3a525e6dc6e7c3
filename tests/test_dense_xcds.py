"""Waves of dense minibatches with each record on one XCD, or a slice of the columns on each, and just beyond those rules:
coefficients and results against 64 bits."""
import pytest
import torch

from paper_1902_01064_amd import hop, inputs
from paper_1902_01064_amd.session import Session

pytestmark = pytest.mark.gpu


# one wave of all workers.  One XCD a record: 1, 7, 8, 9 and 17 records; 2 MB of rows (B = 128 x 4096, 64 x 8192) and one row or
# column more; 48 and 49 records of 16 column chunks (768 and more).
# Slices: from 7169 columns on where rows are over 2 MB (B = 73, 74), else from 11 265; up to 131 072; at least 8 columns a row;
# slices of 5 and 6 chunks, of one less where the last chunk has one column; 940 and 2256 chunks
@pytest.mark.parametrize("N,d,B", [(1, 1, 1), (7, 257, 3), (8, 1024, 64), (9, 4096, 128), (9, 4096, 129), (9, 4097, 100), (17, 1000, 200),
                                   (3, 512, 1024), (3, 512, 1000), (48, 4096, 5), (49, 4096, 5), (3, 8192, 64), (3, 8193, 64),
                                   (2, 7168, 74), (2, 7169, 73), (2, 7169, 74), (3, 11264, 40), (3, 11265, 40), (2, 131072, 16),
                                   (2, 131073, 16), (2, 8192, 1024), (2, 8191, 1024), (1, 11521, 3), (20, 12001, 50), (48, 12001, 17)])
@pytest.mark.parametrize("momentum", [0.0, 0.9])
def test_wave(N, d, B, momentum):
    _check_wave(N, d, B, momentum, 70)


# Data sets that do not fit the memory-side cache and hold more than two minibatches: rows of slices read past the caches, with 8 and
# 4 wavefronts a chunk and with chunks of 1024 columns; ends of rows of 1, 2 and 0 columns over a multiple of four
@pytest.mark.parametrize("N,d,B,rows", [(1, 131072, 16, 520), (2, 100001, 16, 340), (5, 131070, 20, 110)])
@pytest.mark.parametrize("momentum", [0.0, 0.9])
def test_wave_of_large_data(N, d, B, rows, momentum):
    assert rows > 2 * B and N * d * rows * 4 > 256 << 20
    _check_wave(N, d, B, momentum, rows)


# Many rows: one or two records on all XCDs, three on one each
@pytest.mark.parametrize("N,d,B", [(1, 1000, 200), (1, 1000, 201), (2, 513, 200), (2, 513, 201), (2, 512, 1024), (3, 510, 201)])
@pytest.mark.parametrize("momentum", [0.0, 0.9])
def test_wave_of_many_rows(N, d, B, momentum):
    _check_wave(N, d, B, momentum, 70)


# Waves at the number of rows up to which they go in slices, and beyond it
@pytest.mark.parametrize("N,d,B", [(4, 8001, 875), (4, 8001, 876), (35, 7170, 100), (36, 7171, 100), (12, 11266, 501)])
@pytest.mark.parametrize("momentum", [0.0, 0.9])
def test_wave_of_many_rows_in_slices(N, d, B, momentum):
    _check_wave(N, d, B, momentum, 70)


# Results finished in place: 96 MB of them and more, and with workgroups of 4096 columns; jobs end with 0, 2 and 1 columns over four
@pytest.mark.parametrize("N,d,B", [(64, 393216, 1), (64, 393218, 1), (140, 500001, 1), (3, 150001, 3)])
@pytest.mark.parametrize("momentum", [0.0, 0.9])
def test_wave_in_place(N, d, B, momentum):
    _check_wave(N, d, B, momentum, 5)


def _check_wave(N, d, B, momentum, rows):
    nb = [[]] if N == 1 else inputs.ring(N)
    c = dict(inputs.config(1, d=d, rows=rows, K=1), in_nbrs=nb, W=inputs.uniform_weights(nb), N=N, s=0, b=0, batch=B, loss=1, lam=0.25,
             lr=0.5, momentum=momentum, skip_on=False, mult=None, delay_kind=inputs.DELAY_NONE)
    ws = inputs.hidden_w(6, d, "cuda")
    data = [inputs.dense_svm_data(6, i, rows, d, ws, "cuda") for i in range(N)]
    p0 = torch.randn(N, d, generator=torch.Generator(device="cuda").manual_seed(4), device="cuda") / d ** 0.5
    print("XCDs", N, d, B, momentum, rows, flush=True)
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
            X, y, w = data[i][0][ids].double(), data[i][1][ids].double(), p0[i].double()
            coef = torch.from_numpy(sess.coef(e)).cuda().double()
            # the slope of a coefficient in its margin is at most 1 / 4 B; a sum of d products is off by (d + 1) 2^-24 of their magnitudes
            off = (d + 1) * 2.0 ** -24 * (X.abs() @ w.abs())
            want = y / (B * (1 + torch.exp(y * (X @ w))))
            assert bool(((coef - want).abs() <= (0.25 * off + 1e-6) / B).all())
            g, mag = 0.25 * w - coef @ X, 0.25 * w.abs() + coef.abs() @ X.abs()
            acc, size = torch.zeros_like(g), torch.zeros_like(g)
            for a in range(int(s.src_begin[e]), int(s.src_begin[e + 1])):
                x = float(s.src_weight[a]) * p0[int(s.src_worker[a])].double()
                acc, size = acc + x, size + x.abs()
            got = sess.slot(i, int(s.out_slot[e])).double()
            room = 2.0 ** -24 * (0.5 * (B + 4) * mag + 8 * size)        # B + 1 products, up to three sources and the step
            assert bool(((got - (acc - 0.5 * g)).abs() <= room).all())
    finally:
        sess.close()


# Jumps: their Reduce in the margins' launch (one row a workgroup, two, and two past the caches) against a launch of its own, which
# a profiled pass makes; the chunks of 1024 columns of a jump end with 1, 2 and 0 columns over a multiple of four
@pytest.mark.parametrize("d,B", [(12001, 8), (30002, 100), (131072, 128), (8001, 500)])
def test_jumps_beside_the_margins(d, B):
    nb = inputs.ring(16)
    mult = [1.0] * 16
    mult[3] = 4.0
    c = dict(inputs.config(1, d=d, rows=130, K=10), in_nbrs=nb, W=inputs.uniform_weights(nb), N=16, s=2, b=0, batch=B, loss=1, lam=0.25,
             skip_on=True, mult=mult, delay_kind=inputs.DELAY_NONE)
    ws = inputs.hidden_w(6, d, "cuda")
    data = [inputs.dense_svm_data(6, i, 130, d, ws, "cuda") for i in range(16)]
    p0 = torch.randn(16, d, generator=torch.Generator(device="cuda").manual_seed(5), device="cuda") / d ** 0.5
    got = []
    print("jumps", d, B, flush=True)
    for timed in (False, True):
        sess = Session(c)
        try:
            sess.set_dense([x for x, _ in data], [y for _, y in data])
            sess.set_params(p0)
            s = sess.simulate()
            with_both = {int(s.wave[e]) for e in range(s.n_records) if int(s.kind[e]) == hop.HOP_JUMP} & {
                int(s.wave[e]) for e in range(s.n_records) if int(s.kind[e]) == hop.HOP_STEP}
            assert with_both
            hop.hop_profile(sess.ctx, int(timed))
            sess.step()
            sess.sync()
            got.append(sess.arena[:16 * sess.D * sess.stride].clone())
        finally:
            sess.close()
    assert torch.equal(*got)
