"""What the library plans for a batch, without a GPU: its source built for the host alone into tests/sanitize/plan_harness.cpp."""
import os
import subprocess

import pytest

from test_gpu_tile_crowded import ONE_PART

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("plan")
    exe = str(tmp / "plan_harness")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, "--offload-host-only", "-fuse-cuid=none", "-O1", "-std=c++17", "-pthread", "-o", exe, "-x", "hip",
                    os.path.join(ROOT, "tests", "sanitize", "plan_harness.cpp")], check=True, cwd=tmp, stdout=subprocess.PIPE, stderr=subprocess.PIPE)

    def plan(fmt, *rest):
        run = subprocess.run([exe, *map(str, (*fmt, *rest))], stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=60)
        assert run.returncode == 0, run.stderr
        return tuple(map(int, run.stdout.split()))
    return plan


@pytest.mark.parametrize("case", ONE_PART, ids=str)
def test_crowded_tokens_leave_one_part(harness, case):
    """The cases of the test of that name on the GPU, on 256 compute units."""
    even, crowded, _, _ = harness(*case)
    assert even > 1 and crowded == 1


def test_crowded_cases_run_every_kernel(harness):
    kernels = {(harness(*case)[3], case[0][0], case[1] > 0 and case[0][0] == 2) for case in ONE_PART}
    assert {k[0] for k in kernels} == {16, 32, 192}
    assert {(192, 2, False), (192, 2, True), (192, 3, False), (192, 4, False)} <= kernels


@pytest.mark.parametrize("case", [((4, 64), 0, 4096, 14336, 8, 2, 512, 0), ((3, 64), 0, 256, 2048, 8, 2, 512, 0), ((4, 64), 0, 256, 512, 16, 4, 1024, 0), ((4, 128), 0, 512, 1024, 4, 1, 60, 0)], ids=str)
def test_host_time_of_a_plan(harness, case):
    """Every queued step makes its plan anew.  The expected blocks of an expert, of 32 and of 128 tokens and at most 1024 in all, take a call each and
    one more: 33 and 9, however many parts are compared."""
    assert 0 < harness(*case)[2] <= 33 + 9


@pytest.mark.parametrize("case", [((4, 64), 0, 512, 11520, 1, 1, 60, 0), ((4, 128), 128, 256, 11648, 4, 3, 17, 0), ((4, 128), 128, 512, 7296, 2, 2, 48, 0),
                                  ((4, 64), 256, 704, 6336, 1, 1, 27, 0), ((3, 64), 0, 256, 2688, 2, 1, 49, 0), ((3, 64), 256, 384, 640, 1, 1, 107, 0)], ids=str)
def test_parts_of_narrow_layers(harness, case):
    """w2 of a few row blocks of a few experts leaves most compute units idle even in as many parts as there can be: it takes those, whichever kernel
    runs it.  (A launch of fewer blocks than compute units takes a round's time, not none.)"""
    sets = (case[3] // 64 + 3) // 4
    per = -(-sets // min(8, sets))
    assert harness(*case)[0] == -(-sets // per)


@pytest.mark.parametrize("case,tile", [(((4, 64), 0, 3136, 640, 1, 1, 252, 0), True), (((4, 64), 0, 2624, 576, 2, 2, 123, 0), True), (((4, 64), 256, 2688, 576, 1, 1, 87, 0), True),
                                       (((4, 64), 256, 4032, 512, 4, 2, 57, 0), True), (((4, 64), 128, 2688, 640, 8, 2, 102, 0), True), (((4, 64), 256, 2944, 704, 6, 4, 29, 0), True),
                                       (((4, 64), 128, 2944, 576, 2, 2, 17, 0), True), (((4, 64), 0, 1152, 1792, 2, 2, 116, 0), True),
                                       (((4, 64), 0, 1152, 1792, 8, 2, 96, 0), False), (((4, 64), 256, 640, 1088, 13, 2, 111, 0), False), (((4, 64), 0, 1024, 2048, 8, 2, 136, 0), True)], ids=str)
def test_kernels_of_small_layers(harness, case, tile):
    """4-bit layers up to 1024 x 2048: the tile kernels beyond one window of tokens, and with rows of more than 1024 where an expert has more than 32
    tokens on average, 16 with two-level metadata."""
    assert (harness(*case, 0)[3] > 0) == tile


@pytest.mark.parametrize("case", [((3, 64), 0, 1024, 6976, 13, 4, 1009, 0), ((4, 128), 0, 1280, 14336, 8, 2, 1008, 0), ((3, 64), 0, 1280, 7552, 8, 4, 587, 0)], ids=str)
def test_parts_fill_the_xcds(harness, case):
    """The large kernel's jobs of w2, row blocks times parts, go to eight XCDs in whole: as many parts as leave few of them short of one."""
    parts, _, _, kernel = harness(*case)
    jobs = -(-case[2] // 256) * parts
    assert kernel == 192 and jobs >= 0.8 * (-(-jobs // 8) * 8)


@pytest.mark.parametrize("sg,hidden,ffn,batch,tokens", [(0, 4096, 14336, 64, 32), (0, 4096, 14336, 96, 32), (128, 4096, 14336, 64, 32), (0, 4096, 8192, 72, 32), (128, 4096, 8192, 80, 32),
                                                        (128, 2048, 14336, 72, 32), (0, 4096, 14336, 200, 192), (128, 4096, 14336, 256, 192)])
def test_kernels_of_3bit_batches(harness, sg, hidden, ffn, batch, tokens):
    """w2 of large 3-bit layers, 8 experts, top 2: one or two tiles of an expert are the 32-token kernel's, more the large one's."""
    assert harness((3, 64), sg, hidden, ffn, 8, 2, batch, 0)[3] == tokens
