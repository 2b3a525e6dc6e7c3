"""A pass run as one launch, column by column: its program against the records one by one (on the CPU, under the
sanitizers), and the kernel against the same pass wave by wave, which takes every sum in the same order."""
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

from paper_1902_01064_amd import hop, inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"), reason="needs g++ and the HIP headers")
def test_program_gives_what_the_records_give(tmp_path):
    exe = str(tmp_path / "sweep_driver")
    csrc = os.path.join(ROOT, "paper_1902_01064_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-static-libasan", "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I",
                    os.path.join(ROOT, "include"), "-I", csrc, os.path.join(ROOT, "tests", "sweep_driver.cpp"),
                    os.path.join(csrc, "hop_api.cpp"), os.path.join(csrc, "hop_sim.cpp"), "-L/opt/rocm/lib", "-lamdhip64",
                    "-Wl,-rpath,/opt/rocm/lib", "-o", exe], check=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0:verify_asan_link_order=0")
    out = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=300)
    assert out.returncode == 0, out.stdout[-2000:] + out.stderr[-4000:]
    assert out.stdout.startswith("ok ")


# 1 column, one short of / exactly / one past a wavefront's 64, a ragged tail past the narrow-model limit; records of
# 1 to 14 sources (12 go through the kernel's chain); velocities; jumps; both approaches; a graph with too many values for the
# registers
@pytest.mark.gpu
@pytest.mark.parametrize("mode", ["zero", "synth", "external"])
@pytest.mark.parametrize("graph,over", [
    ("chords", dict(d=1)), ("chords", dict(d=63, momentum=0.9)), ("chords", dict(d=64)), ("chords", dict(d=65, serial=True)),
    ("chords", dict(d=66003, skip_on=True, mult=[3.0] + [1.0] * 31)), ("complete", dict(d=1028, momentum=0.5)),
    ("complete", dict(d=70000)), ("torus", dict(d=65540, K=4, momentum=0.9)),
])
def test_pass_equals_the_waves_bit_for_bit(mode, graph, over):
    nb = {"chords": lambda: inputs.ring_with_chords(32, 2, 7), "complete": lambda: inputs.complete(14),
          "torus": lambda: inputs.torus(9, 9)}[graph]()
    N = len(nb)
    if mode == "external":
        over = dict(over, d=(over["d"] + 3) // 4 * 4)        # what the entry point asks for with several workers
    c = dict(inputs.config(4, d=over["d"], K=8), in_nbrs=nb, W=inputs.uniform_weights(nb), N=N, s=2, b=1, skip_on=False,
             mult=None, delay_kind=inputs.DELAY_EXP1)
    c.update(over)
    print("sweep", mode, graph, over, flush=True)
    from paper_1902_01064_amd.session import Session
    p0 = torch.randn(N, c["d"], generator=torch.Generator().manual_seed(1))
    ext = (0.1 * torch.randn(N, c["d"], generator=torch.Generator().manual_seed(2))).cuda()
    got = {}
    for way in ("pass", "waves"):
        sess = Session(c)
        try:
            if mode == "synth":
                hop.hop_set_grad_source(sess.ctx, hop.HOP_GRAD_SYNTH, 1e-3)
            elif mode == "external":
                hop.hop_set_grad_source(sess.ctx, hop.HOP_GRAD_EXTERNAL, 0.0, ext.data_ptr())
            sess.arena.fill_(7.0)                             # what no record writes has to stay
            sess.set_params(p0)
            sched = sess.simulate()
            for _ in range(2):                                # the second pass starts from what the rings hold
                if way == "pass":
                    sess.step()
                else:
                    for w in range(sched.n_waves):
                        sess.step(w, w + 1)
            sess.sync()
            got[way] = sess.arena[:N * sess.D * sess.stride].cpu().numpy()
            # 81 workers with velocities would need 162 local slots; without gradients the velocities stay where they are
            refused = graph == "torus" and mode != "zero"
            assert hop.hop_pass_path(sess.ctx, sched) == (hop.HOP_PASS_WAVES if refused else hop.HOP_PASS_ONE_LAUNCH)
            if c.get("momentum"):
                got[way] = np.concatenate([got[way], sess.vel_snapshot().reshape(-1)])
        finally:
            sess.close()
    assert np.isfinite(got["waves"]).all() and np.array_equal(got["pass"], got["waves"])


@pytest.mark.gpu
def test_pass_keeps_the_sign_of_zero():
    """Parameters of -0: with a velocity a sum starts with a product, so every average is -0 again, whether the number of
    sources is odd or even."""
    nb = inputs.ring_with_chords(32, 2, 7)
    c = dict(inputs.config(4, d=130, K=8), in_nbrs=nb, W=inputs.uniform_weights(nb), N=32, s=2, b=1, skip_on=False, mult=None,
             delay_kind=inputs.DELAY_EXP1, momentum=0.9)
    from paper_1902_01064_amd.session import Session
    sess = Session(c)
    try:
        hop.hop_set_grad_source(sess.ctx, hop.HOP_GRAD_ZERO)
        sess.arena.fill_(-0.0)
        sess.set_params(torch.full((c["d"],), -0.0))
        sched = sess.simulate()
        sources = np.diff(sched.src_begin)
        assert (sources % 2 == 1).any() and (sources % 2 == 0).any()
        sess.step()
        sess.sync()
        assert np.array_equal(sess.ring_snapshot().view(np.uint32), np.full_like(sess.ring_snapshot(), -0.0).view(np.uint32))
    finally:
        sess.close()


# many records per wave of a narrow model are faster in waves, and so are synthetic gradients where records of many sources take
# several parts; without them such records are faster in one launch (15 iterations in lock-step, waves and one launch: 14 workers x
# 1024 columns 56.5 and 42.2 us, 24 x 65 536 267 and 110 us)
@pytest.mark.gpu
@pytest.mark.parametrize("nb,d,delay,mode,one", [
    (inputs.ring(4), 1024, "none", "zero", True), (inputs.torus(4, 4), 1000, "none", "zero", True),
    (inputs.torus(9, 9), 1024, "none", "zero", False), (inputs.torus(9, 9), 1 << 20, "none", "synth", True),
    (inputs.complete(14), 1024, "none", "zero", True), (inputs.complete(14), 1024, "exp1", "zero", True),
    (inputs.complete(24), 1024, "none", "synth", False), (inputs.complete(24), 65536, "none", "zero", True),
    (inputs.complete(14), 1 << 20, "none", "synth", True), (inputs.ring_with_chords(32, 2, 7), 300007, "exp1", "synth", True),
])
def test_which_way_a_pass_goes(nb, d, delay, mode, one):
    N = len(nb)
    c = dict(inputs.config(4, d=d, K=10), in_nbrs=nb, W=inputs.uniform_weights(nb), N=N, s=2, b=0, skip_on=False, mult=None,
             delay_kind=inputs.DELAY_EXP1 if delay == "exp1" else inputs.DELAY_NONE, grad_ahead=1)
    from paper_1902_01064_amd.session import Session
    sess = Session(c)
    try:
        hop.hop_set_grad_source(sess.ctx, hop.HOP_GRAD_SYNTH if mode == "synth" else hop.HOP_GRAD_ZERO, 1e-3)
        sess.set_params(torch.zeros(d))
        sched = sess.simulate()
        with pytest.raises(hop.HopError) as e:
            hop.hop_pass_path(sess.ctx, sched)
        assert e.value.code == hop.HOP_ERR_STATE
        sess.step(0, 1)
        assert hop.hop_pass_path(sess.ctx, sched) == (hop.HOP_PASS_ONE_LAUNCH if one else hop.HOP_PASS_WAVES)
        hop.hop_use_graph(sess.ctx, 1)
        assert hop.hop_pass_path(sess.ctx, sched) == (hop.HOP_PASS_ONE_LAUNCH if one else hop.HOP_PASS_GRAPH)
    finally:
        sess.close()
