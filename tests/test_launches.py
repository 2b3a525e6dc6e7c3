"""What a pass launches and the rules behind it, on the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"), reason="needs g++ and the HIP headers")


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("launches") / "launch_driver")
    csrc = os.path.join(ROOT, "paper_1902_01064_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-static-libasan",
                    "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", os.path.join(ROOT, "include"), "-I", csrc,
                    os.path.join(ROOT, "tests", "launch_driver.cpp"), os.path.join(csrc, "hop_api.cpp"),
                    os.path.join(csrc, "hop_sim.cpp"), "-o", exe], check=True)

    def run(*what):
        env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0:verify_asan_link_order=0")
        out = subprocess.run([exe] + [str(w) for w in what], capture_output=True, text=True, env=env, timeout=120)
        assert out.returncode == 0, out.stdout[-2000:] + out.stderr[-4000:]
        lines = [line.split() for line in out.stdout.splitlines()]
        return [(name, dict(a.split("=") for a in rest)) for name, *rest in lines]
    return run


# 4 workers x 16384 columns are 256 KB a row of each data set: 1024 rows of all of them are the memory-side cache's 256 MB; two
# minibatches of 600 rows are more than that
@pytest.mark.parametrize("rows,batch,again", [(1024, 64, 1), (1025, 64, 0), (1200, 600, 1), (1201, 600, 0)])
@pytest.mark.parametrize("momentum", [0.0, 0.9])
def test_rows_that_come_again(launches, rows, batch, again, momentum):
    got = [a["rows_again"] for name, a in launches("dense", 4, 16384, batch, rows, momentum) if name == "dense_grad"]
    assert got == [str(again)] * 2


# One XCD a record: 2 MB, 8192 columns, 768 chunks; one or two records of a wave only with up to 200 rows
@pytest.mark.parametrize("n,d,B,one,alone", [
    (1, 1024, 64, 1, 1), (1, 1024, 200, 1, 1), (2, 1024, 201, 0, 1), (1, 512, 1024, 0, 1), (3, 512, 1024, 1, 1),
    (4, 8192, 64, 1, 1), (4, 8193, 63, 0, 0), (4, 4096, 129, 0, 0), (48, 4096, 5, 1, 1), (49, 4096, 5, 0, 1)])
def test_one_xcd(launches, n, d, B, one, alone):
    (_, got), = launches("rules", n, d, B)
    assert (got["one_xcd"], got["one_xcd_alone"]) == (str(one), str(alone))


# Slices: of a pass by its rows, of a wave by how many of them it has, where a row is one segment of the other form
@pytest.mark.parametrize("n,d,B,of_pass,of_wave", [
    (35, 7169, 100, 1, 1), (36, 11264, 100, 1, 0), (4, 11264, 875, 1, 1), (4, 11264, 876, 1, 0), (60, 11265, 100, 1, 1), (61, 14336, 100, 1, 0),
    (61, 14337, 100, 1, 1), (1000, 131072, 1024, 1, 1), (1, 131073, 64, 0, 0), (1, 7168, 100, 0, 0), (2, 8191, 1024, 0, 0)])
def test_slices(launches, n, d, B, of_pass, of_wave):
    (_, got), = launches("rules", n, d, B)
    assert (got["slices"], got["wave_slices"]) == (str(of_pass), str(of_wave))


# Waves that stay in the L2s: by their jobs, so that the two pairs of a lock-step ring of four stay up to 64 MB of results
def test_waves_that_stay_near(launches):
    assert launches("external", 4, 4096, 0, 0, 0.0) == [("pair", dict(jobs="2"))] * 2
    assert launches("external", 4, 4096, 0, 0, 0.9) == [("mix", dict(jobs="4"))] * 2
    for n, d, near, with_velocity in [(2, 4194304, 1, 0), (2, 4194305, 0, 0), (4, 699050, 1, 1), (4, 699051, 1, 0), (1, 8388608, 1, 0), (1, 8388609, 0, 0)]:
        (_, got), = launches("rules", n, d, 1)
        assert (got["near"], got["near_velocity"]) == (str(near), str(with_velocity))


# Averages by themselves: a few jobs as an argument, more in memory; these stay in the L2s up to 16 MB and where no two records share a job
@pytest.mark.parametrize("n,d,sources,momentum,want", [
    (32, 1000, 5, 0.0, ("pair_args", dict(jobs="16"))), (34, 1000, 5, 0.0, ("pair_alone", dict(jobs="17", results="34", near="0"))),
    (16, 262144, 13, 0.0, ("pair_alone", dict(jobs="16", results="16", near="1"))),
    (16, 262145, 13, 0.0, ("pair_alone", dict(jobs="16", results="16", near="0"))), (34, 1000, 5, 0.9, ("mix", dict(jobs="34")))])
def test_stand_alone_averages(launches, n, d, sources, momentum, want):
    assert launches("average", n, d, sources, momentum) == [want]


# Results that the same wave's gradient reads next
@pytest.mark.parametrize("n,d,near", [(4, 1024, 1), (64, 393216, 1), (64, 393217, 0), (48, 524288, 1), (49, 524288, 0)])
def test_results_in_place(launches, n, d, near):
    (_, got), = launches("rules", n, d, 1)
    assert got["in_place"] == str(near)


# Sparse margins beside records that run singly: known by the results of the jobs, not by fewer jobs than gradients, as jumps pair up too
def test_single_records(launches):
    got = [tuple(int(a[k]) for k in ("jobs", "results", "gradients")) for name, a in launches("skipping", 4, 256, 4, 50, 0.0) if name == "pair_csr_margin"]
    assert all(jobs <= results <= 2 * jobs and gradients <= results for jobs, results, gradients in got)
    assert any(jobs == results for jobs, results, _ in got) and any(gradients <= jobs < results for jobs, results, gradients in got)


# Which way whole passes go: us in waves / in one launch on MI355X 96 / 178, 119 / 184, 282 / 198, 79 / 134, 227 / 131, 72 / 128, 40 / 8
@pytest.mark.parametrize("n,d,momentum,one", [(32, 4096, 0.9, 0), (32, 20000, 0.9, 0), (32, 65540, 0.9, 1), (24, 4096, 0.9, 0), (24, 4096, 0.0, 1),
                                              (24, 336, 0.0, 0), (4, 64, 0.0, 1)])
def test_way_of_whole_passes(launches, n, d, momentum, one):
    got = [name for name, _ in launches("complete", n, d, 0, 0, momentum)]
    assert got == (["sweep"] if one else ["mix" if momentum else "pair"] * 15)
