"""The dense SVM gradient where its kernels change path: column counts around a 256-column chunk, a wavefront's last lane
and a 16384-column segment with every remainder mod 4, minibatches around the 8 rows a wavefront takes at a time, 15, 16,
64 and 65 partial products per row, data sets, parameters and results at any multiple of 4 bytes when d is no multiple of
four."""
import numpy as np
import pytest
import torch

from oracle import arith, rng
from paper_1902_01064_amd import hop

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _at(host, shift):
    """Device copy that starts `shift` floats past a 256-byte boundary."""
    t = torch.zeros(host.numel() + 64 + shift, device=DEV)
    v = t[shift:shift + host.numel()]
    v.copy_(host.reshape(-1))
    return t, v


@pytest.mark.parametrize("loss", ["hinge", "log"])
@pytest.mark.parametrize("d,B,shift", [(1, 1, 1), (2, 9, 3), (3, 64, 2), (255, 8, 1), (256, 7, 0), (257, 65, 3), (1021, 1024, 1),
                                       (16383, 33, 2), (16385, 16, 1), (16390, 100, 0), (196612, 40, 0),
                                       (245758, 9, 2), (245761, 17, 1), (524288, 8, 0), (1048577, 5, 3), (1048580, 33, 0)])
def test_dense_gradient_at_the_edges(d, B, shift, loss):
    print("dense d=%d B=%d shift=%d %s" % (d, B, shift, loss), flush=True)
    gen = torch.Generator().manual_seed(d * 7 + B)
    rows = 40
    X = torch.randn(rows, d, generator=gen)
    y = torch.sign(torch.randn(rows, generator=gen))
    w = torch.randn(d, generator=gen) / np.sqrt(d)
    ids = rng.batch_rows(d, 0, 1, B, rows)
    keep, Xd = _at(X, shift)
    keep2, wd = _at(w, shift)
    gbuf = torch.full((d + 64 + shift,), 7.0, device=DEV)
    g = gbuf[shift:shift + d]
    yd, rd = y.to(DEV), torch.from_numpy(ids.astype(np.int32)).to(DEV)
    coef = torch.zeros(B, device=DEV)
    scratch = torch.empty(hop.hop_grad_scratch_floats(d, B), device=DEV)
    lam, st = 1e-3, torch.cuda.current_stream().cuda_stream
    hop.hop_svm_grad_dense(Xd.data_ptr(), yd.data_ptr(), wd.data_ptr(), rd.data_ptr(), B, d, lam, g.data_ptr(),
                           coef.data_ptr(), scratch.data_ptr(), st, 1 if loss == "log" else 0)
    torch.cuda.synchronize()
    got, cg = g.cpu().numpy().astype(np.float64), coef.cpu().numpy()
    Xn, yn, wn = X.numpy(), y.numpy(), w.numpy()
    ref, margins, act = arith.svm_subgradient_dense(Xn, yn, wn, ids, lam, loss=loss)
    if loss == "hinge":                                   # at a margin within rounding of 1 follow the kernel's side
        scale = np.abs(Xn[ids].astype(np.float64) * wn).sum(1)
        assert np.all(np.abs(1.0 - margins[act != (cg != 0)]) <= 1e-5 * (1.0 + scale[act != (cg != 0)]))
        ref, _, act = arith.svm_subgradient_dense(Xn, yn, wn, ids, lam, active=cg != 0)
    want_c, _ = arith.loss_coefficients(yn[ids].astype(np.float64), margins, B, loss, act)
    mag = lam * np.abs(wn) + np.abs(want_c) @ np.abs(Xn[ids].astype(np.float64))
    # an fp32 sum of B + 1 products is within (B + 3) 2^-24 of the sum of magnitudes; with the log loss a coefficient
    # carries its margin's error as well: the fp32 dot of d terms, at most d 2^-24 of its magnitudes
    slack = (B + 3) * 2.0 ** -24
    if loss == "log":
        slack += min(d, 4096) * 2.0 ** -24 * (1.0 + np.abs(Xn[ids].astype(np.float64) * wn).sum(1).max())
    assert np.all(np.abs(got - ref) <= slack * mag + 1e-30)
    assert (gbuf[:shift] == 7.0).all() and (gbuf[shift + d:] == 7.0).all()           # nothing written beside the result


@pytest.mark.parametrize("loss", ["hinge", "log"])
@pytest.mark.parametrize("d,B", [(1024, 8), (1021, 8), (4, 5), (3, 5), (258, 64), (4096, 100), (16390, 33)])
def test_samples_that_are_not_finite(d, B, loss):
    """The first sample of the minibatch has an infinite margin on the right side (hinge: one that is no number): it takes
    no part, and what it holds stays out of the gradient.  The second has an infinite margin on the wrong side: it takes
    part, in column 0 with an infinity."""
    print("not finite d=%d B=%d %s" % (d, B, loss), flush=True)
    gen = torch.Generator().manual_seed(d + B)
    X = torch.randn(B, d, generator=gen)
    y = torch.sign(torch.randn(B, generator=gen))
    w = 0.1 + torch.rand(d, generator=gen) / np.sqrt(d)
    y[0], y[1] = 1.0, 1.0
    X[0, d // 2], X[0, d - 1] = float("nan" if loss == "hinge" else "inf"), float("inf")
    X[1, 0] = float("-inf")                                       # active: -c * -inf = +inf in column 0
    ids = np.arange(B)
    Xd, yd, wd, rd = X.to(DEV), y.to(DEV), w.to(DEV), torch.from_numpy(ids.astype(np.int32)).to(DEV)
    g, coef = torch.empty(d, device=DEV), torch.zeros(B, device=DEV)
    scratch = torch.empty(hop.hop_grad_scratch_floats(d, B), device=DEV)
    hop.hop_svm_grad_dense(Xd.data_ptr(), yd.data_ptr(), wd.data_ptr(), rd.data_ptr(), B, d, 1e-3, g.data_ptr(),
                           coef.data_ptr(), scratch.data_ptr(), torch.cuda.current_stream().cuda_stream,
                           1 if loss == "log" else 0)
    torch.cuda.synchronize()
    cg, got = coef.cpu().numpy(), g.cpu().numpy().astype(np.float64)
    assert cg[0] == 0.0 and abs(cg[1] - 1.0 / B) <= 1e-7
    part = cg != 0
    ref = 1e-3 * w.numpy().astype(np.float64) - cg[part].astype(np.float64) @ X.numpy()[part].astype(np.float64)
    assert ref[0] == np.inf and got[0] == np.inf
    mag = 1e-3 * np.abs(w.numpy()) + np.abs(cg[part]) @ np.abs(X.numpy()[part].astype(np.float64))
    # an fp32 sum of B + 1 products is within (B + 3) 2^-24 of the sum of magnitudes
    assert np.all(np.abs(got[1:] - ref[1:]) <= (B + 3) * 2.0 ** -24 * mag[1:])


# a call of up to 2 MB keeps to one XCD
@pytest.mark.parametrize("loss", ["hinge", "log"])
@pytest.mark.parametrize("d,B", [(511, 1024), (513, 1024), (61, 769), (1024, 512), (1024, 513)])
def test_dense_gradient_of_many_rows(d, B, loss):
    test_dense_gradient_at_the_edges(d, B, 0, loss)


# the end of a vector: no column or one, two, three are left for the last thread, alone or beside others
@pytest.mark.parametrize("loss", ["hinge", "log"])
@pytest.mark.parametrize("d,B", [(4, 70), (5, 70), (6, 300), (7, 9), (1022, 300), (1023, 64), (16386, 100), (65538, 20), (65539, 128), (262147, 33)])
def test_dense_gradient_at_the_end_of_a_vector(d, B, loss):
    test_dense_gradient_at_the_edges(d, B, 0, loss)
