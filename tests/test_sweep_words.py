"""What the whole-pass kernel reads (on the CPU, under the sanitizers), and the kernel where several wavefronts share a SIMD:
the same bits as the pass wave by wave, for every number of registers it is built with."""
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

from paper_1902_01064_amd import hop, inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"), reason="needs g++ and the HIP headers")
def test_words_give_what_the_records_give(tmp_path):
    exe = str(tmp_path / "sweep_words_driver")
    csrc = os.path.join(ROOT, "paper_1902_01064_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-static-libasan", "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I",
                    os.path.join(ROOT, "include"), "-I", csrc, os.path.join(ROOT, "tests", "sweep_words_driver.cpp"),
                    os.path.join(csrc, "hop_api.cpp"), os.path.join(csrc, "hop_sim.cpp"), "-L/opt/rocm/lib", "-lamdhip64",
                    "-Wl,-rpath,/opt/rocm/lib", "-o", exe], check=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0:verify_asan_link_order=0")
    out = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=300)
    assert out.returncode == 0, out.stdout[-2000:] + out.stderr[-4000:]
    assert out.stdout.startswith("ok ")


# up to 48, 80, 112 and 168 local slots; records of one source, of five and six (half of their words or all), of 14 and 16
# (two parts); ragged lengths of 800 to 32 000 wavefronts, so that all SIMDs hold several at different places of the program
@pytest.mark.gpu
@pytest.mark.parametrize("graph,d,mode,over", [
    ("ring", 2_000_003, "synth", dict(momentum=0.9, K=30)), ("ring", 51_203, "zero", dict(K=30)),
    ("double_ring", 1_000_001, "synth", dict(momentum=0.9, K=20)), ("double_ring", 400_004, "external", dict(momentum=0.9, K=20)),
    ("double_ring", 400_001, "zero", dict(momentum=0.9, K=20)), ("chords", 700_003, "synth", dict(K=10, skip_on=True)),
    ("chords", 300_004, "external", dict(K=10, serial=True)), ("chords", 700_003, "synth", dict(momentum=0.9, K=8)),
    ("torus", 500_003, "synth", dict(momentum=0.9, K=6)), ("complete", 800_002, "synth", dict(K=8)),
])
def test_pass_of_many_wavefronts_equals_the_waves(graph, d, mode, over):
    nb = {"ring": lambda: inputs.ring(4), "double_ring": lambda: inputs.double_ring(16), "torus": lambda: inputs.torus(8, 8),
          "chords": lambda: inputs.ring_with_chords(32, 2, 7), "complete": lambda: inputs.complete(16)}[graph]()
    N = len(nb)
    c = dict(inputs.config(4, d=d), in_nbrs=nb, W=inputs.uniform_weights(nb), N=N, s=3, b=1, skip_on=False, mult=None,
             delay_kind=inputs.DELAY_EXP1, grad_ahead=1)
    c.update(over)
    print("sweep words", graph, d, mode, over, flush=True)
    from paper_1902_01064_amd.session import Session
    gen = torch.Generator(device="cuda").manual_seed(3)
    p0 = torch.randn(N, d, generator=gen, device="cuda")
    ext = 0.1 * torch.randn(N, d, generator=gen, device="cuda")
    got = {}
    for way in ("pass", "waves"):
        sess = Session(c)
        try:
            if mode == "synth":
                hop.hop_set_grad_source(sess.ctx, hop.HOP_GRAD_SYNTH, 1e-3)
            elif mode == "external":
                hop.hop_set_grad_source(sess.ctx, hop.HOP_GRAD_EXTERNAL, 0.0, ext.data_ptr())
            sess.arena.fill_(7.0)
            sess.set_params(p0)
            sched = sess.simulate()
            for _ in range(2):
                if way == "pass":
                    sess.step()
                else:
                    for w in range(sched.n_waves):
                        sess.step(w, w + 1)
            sess.sync()
            assert hop.hop_pass_path(sess.ctx, sched) == hop.HOP_PASS_ONE_LAUNCH
            got[way] = [sess.arena[:N * sess.D * sess.stride].clone()]
            if c.get("momentum"):
                got[way].append(sess.arena[sess.arena.numel() - N * sess.stride:].clone())
        finally:
            sess.close()
    for a, b in zip(got["pass"], got["waves"]):
        assert bool(torch.isfinite(b).all()) and bool(torch.equal(a, b))
