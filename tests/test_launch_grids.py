"""Launches at the edges of a grid: more jobs than it has rows, and vectors of more rounds of chunks than it has layers."""
import numpy as np
import pytest
import torch

from paper_1902_01064_amd import hop, inputs

pytestmark = pytest.mark.gpu


# rows of a grid: 65535; pairs are not formed where every vector is read once
@pytest.mark.parametrize("n", [65535, 65536, 70001])
@pytest.mark.parametrize("momentum", [False, True])
def test_mix_of_many_jobs(n, momentum):
    d, stride, eta, mu = 5, 8, 0.5, 0.75
    gen = torch.Generator(device="cuda").manual_seed(n)
    src, g, vel = (torch.randn(n, stride, generator=gen, device="cuda") for _ in range(3))
    out, before = torch.zeros(n, stride, device="cuda"), vel.double()
    at = [t.data_ptr() for t in (out, g, src, vel)]
    jobs = [dict(out=at[0] + 4 * stride * i, g=at[1] + 4 * stride * i, eta=eta, src=[at[2] + 4 * stride * i], w=[1.0 / (1 + i % 7)])
            for i in range(n)]
    if momentum:
        for i, j in enumerate(jobs):
            j.update(vel=at[3] + 4 * stride * i, mu=mu)
    print("mix of", n, "jobs, momentum", momentum, flush=True)
    hop.hop_mix(jobs, d, torch.cuda.current_stream().cuda_stream)
    w = torch.tensor([float(np.float32(1.0 / (1 + k))) for k in range(7)], dtype=torch.float64, device="cuda")
    v = mu * before + g.double() if momentum else g.double()
    want = w[torch.arange(n, device="cuda") % 7][:, None] * src.double() - eta * v
    room = 4 * 2.0 ** -24 * (src.double().abs() + eta * (mu * before.abs() + g.double().abs()))    # three roundings of the terms
    assert bool(((out.double() - want).abs() <= room)[:, :d].all()) and bool((out[:, d:] == 0).all())
    if momentum:
        assert bool(((vel.double() - v).abs() <= room / eta)[:, :d].all()) and torch.equal(vel[:, d:].double(), before[:, d:])


# 65535 layers of 8 chunks of 2048 columns are not enough for the generator of a wave: parameters of zero become a step along the
# gradients that a call by itself, on a grid of one row, gives
@pytest.mark.parametrize("d", [65535 * 8 * 2048, 65535 * 8 * 2048 + 5])
def test_generator_of_very_long_vectors(d):
    from paper_1902_01064_amd.session import Session
    nb = inputs.ring(2)
    c = dict(inputs.config(4, d=d, K=1), in_nbrs=nb, W=inputs.uniform_weights(nb), N=2, s=1, b=0, skip_on=False, mult=None,
             delay_kind=inputs.DELAY_NONE, grad_ahead=1)
    pieces = list(range(0, d, 1 << 26)) + [d]              # every column, a few at a time
    print("generator of", d, "columns", flush=True)
    g = torch.empty((d + 3) // 4 * 4, device="cuda")
    sess = Session(c)
    try:
        hop.hop_set_grad_source(sess.ctx, hop.HOP_GRAD_SYNTH, 1e-3)
        sess.set_params(torch.zeros(d, device="cuda"))
        sess.simulate()
        hop.hop_profile(sess.ctx, 1)                       # a profiled pass goes wave by wave
        sess.step()
        sess.sync()
        lr = torch.tensor(c["lr"], dtype=torch.float32, device="cuda")
        for i, p in enumerate(sess.params()[0]):
            hop.hop_synth_grad(c["seed"], i, 0, 1e-3, g.data_ptr(), d, sess.stream)
            torch.cuda.synchronize()
            assert bool((g[:d] != 0).any())
            for lo, hi in zip(pieces, pieces[1:]):         # sums of zeros, then one product: exact
                assert torch.equal(p[lo:hi], -(lr * g[lo:hi]))
    finally:
        sess.close()
        torch.cuda.empty_cache()


# Waves whose jobs (two pairs; with velocities four records, three times their share) come to 32 MB and a little more, with 1, 2 and 3
# columns over a multiple of four: results stored for the L2s or past them, wave by wave, against the pass in one launch, bit for bit
@pytest.mark.parametrize("d,momentum", [(4194304, 0.0), (4194305, 0.0), (2097153, 0.0), (699050, 0.9), (699051, 0.9), (4099, 0.0), (4098, 0.9)])
@pytest.mark.parametrize("gradient", [hop.HOP_GRAD_ZERO, hop.HOP_GRAD_SYNTH])
def test_waves_that_stay_near(d, momentum, gradient):
    from paper_1902_01064_amd.session import Session
    nb = inputs.ring(4)
    c = dict(inputs.config(4, d=d, K=6), in_nbrs=nb, W=inputs.uniform_weights(nb), N=4, s=1, b=0, skip_on=False, mult=None,
             delay_kind=inputs.DELAY_NONE, grad_ahead=1, momentum=momentum)
    p0 = torch.randn(4, d, generator=torch.Generator(device="cuda").manual_seed(d % 89), device="cuda")
    got = []
    print("near", d, momentum, gradient, flush=True)
    for whole in (True, False):
        sess = Session(c)
        try:
            hop.hop_set_grad_source(sess.ctx, gradient, 1e-3 if gradient == hop.HOP_GRAD_SYNTH else 0.0)
            sess.set_params(p0)
            n = sess.simulate().n_waves
            for _ in range(2):
                for at in [(0, n)] if whole else [(w, w + 1) for w in range(n)]:
                    sess.step(*at)
            sess.sync()
            assert hop.hop_pass_path(sess.ctx, sess.sched) == hop.HOP_PASS_ONE_LAUNCH       # what the whole pass took
            got.append(sess.arena[:4 * sess.D * sess.stride].clone())
        finally:
            sess.close()
    assert torch.equal(*got)
