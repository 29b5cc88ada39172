"""The rules that choose between kernels, built for the host (CPU only): their
edges, and that no launch of the scaling kernel reaches 2^32 work-items."""
import os
import shutil
import subprocess
import tempfile

import pytest

from test_k4_host import HIPCC, ROOT


@pytest.fixture(scope="module")
def ask():
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    d = tempfile.mkdtemp()
    exe = os.path.join(d, "routes_host_driver")
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17",
                           "-ffp-contract=off", "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_2606_29129_amd", "csrc"),
                           os.path.join(ROOT, "tests", "routes_host_driver.cpp"), "-o", exe],
                          stderr=subprocess.DEVNULL)

    def run(lines):
        out = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True,
                             check=True).stdout.split()
        assert len(out) == len(lines)
        return [x == "1" for x in out]

    yield run
    shutil.rmtree(d, ignore_errors=True)


def test_scaling_kernel_rule(ask):
    want = {
        "d 256 256 256 14": True, "d 128 128 2816 14": True, "d 128 128 2817 14": False,
        "d 752 8 4096 14": False, "d 760 8 4096 14": True, "d 4096 4096 4096 14": True,
        "d 4096 4096 4097 14": False, "d 64 4096 4096 14": False, "d 64 4096 3071 14": True,
        "d 256 4096 4096 14": False, "d 257 4096 4096 14": True, "d 64 10240 4096 14": True,
        "s 128 128 2304 7": True, "s 128 128 2305 7": False, "s 1000 16 3071 7": True,
        "s 1000 16 3072 7": False, "s 2048 16 4096 7": True,
        "z 64 3072 4096 14": False, "z 3072 64 4096 14": True, "z 64 1024 4096 14": True,
        "z 257 3072 4096 14": True, "c 128 128 4096 7": True, "c 64 6144 2500 7": False}
    assert dict(zip(want, ask(["k12 " + x for x in want]))) == want


def test_scaling_kernel_stays_within_a_launch(ask):
    """64 vectors to a block of 512 at short k: 2^29 rows would make 2^23
    blocks, 2^32 work-items; the separate kernels take those."""
    assert ask(["k12 d %d 1 1 2" % (1 << 28), "k12 d %d 1 1 2" % ((1 << 29) - 64),
                "k12 d %d 1 1 2" % (1 << 29), "k12 s %d 5 64 2" % (1 << 29),
                "k12 z %d 1 1 2" % (1 << 28)]) == [True, False, False, False, False]


def test_fused_kernel_rule(ask):
    want = {
        "d 12287 256 14": False, "d 12288 256 14": True, "d 12288 1024 2": True,
        "d 9215 64 14": False, "d 9216 64 14": True, "d 9216 65 14": False,
        "d 8192 2047 14": False, "d 8192 2048 14": True, "s 8192 4095 7": False,
        "s 8192 4096 7": True, "d 8192 2048 3": False, "d 8192 4096 3": True,
        "d 7167 100000 14": False, "d 7168 100000 14": True, "d 16384 65 14": True,
        "d 16385 1024 14": False, "d 18432 1023 14": False, "d 18432 1024 14": True,
        "d 24575 256 14": False, "d 24576 256 14": True, "d 65536 4096 14": True}
    assert dict(zip(want, ask(["fuse " + x for x in want]))) == want
