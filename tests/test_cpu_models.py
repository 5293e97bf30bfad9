"""The kernels' own index and mask arithmetic on the CPU (tests/cpu_models)."""
import os
import shutil
import subprocess

import pytest

from paper_2007_08501_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def hipcc():
    try:
        return build.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not installed")


@pytest.fixture(scope="module")
def edge_mask(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("edge") / "edge_mask_margin")
    subprocess.check_call([hipcc(), "-x", "hip", "--cuda-host-only", "-O2", "-std=c++17", "-ffp-contract=off",
                           os.path.join(ROOT, "tests", "cpu_models", "edge_mask_margin.hip"), "-o", exe])

    def run(trials, share):
        p = subprocess.run([exe, str(trials), str(share)], capture_output=True, text=True, timeout=300)
        assert p.returncode in (0, 1), p.stdout + p.stderr
        words = p.stdout.split()
        return {k: int(words[words.index(k) + 1]) for k in ("pixels", "kept", "lost")}, p.stdout

    return run


def test_edge_masks_lose_no_pixel_with_a_tenth_of_their_slack(edge_mask):
    n, out = edge_mask(2000000, 0.1)
    assert n["pixels"] > 50_000_000 and n["lost"] == 0, out


def test_edge_mask_check_sees_lost_pixels(edge_mask):
    # (a radius below the plain one by as much must lose some)
    n, out = edge_mask(100000, -0.1)
    assert n["lost"] > 100, out


def test_edge_masks_are_tight(edge_mask):
    # the whole slack keeps a few pixels more than must be kept, not many
    n, out = edge_mask(200000, 1.0)
    m, _ = edge_mask(200000, 0.0)
    assert n["lost"] == 0 and n["kept"] <= 1.1 * m["kept"], out


def test_tile_block_model(tmp_path):
    """The fine pass's LDS block: every offset inside it, every face tested
    once, every fragment written once; a block a few bytes smaller fails."""
    if shutil.which("g++") is None:
        pytest.skip("g++ not installed")
    exe = str(tmp_path / "tile_block_model")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                           "-fno-sanitize-recover=undefined",
                           os.path.join(ROOT, "tests", "cpu_models", "tile_block_model.cpp"), "-o", exe])

    def run(*args):
        return subprocess.run([exe, *args], capture_output=True, text=True, timeout=300,
                              env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))

    ok = run()
    assert ok.returncode == 0 and "ok: block of 6400 bytes" in ok.stdout, ok.stdout + ok.stderr
    short = run("6392")
    assert short.returncode == 1 and "FAILED: staged word" in short.stdout, short.stdout + short.stderr
    few = run(str(63 * 96))
    assert few.returncode == 1 and "FAILED: record place" in few.stdout, few.stdout + few.stderr
