"""What a list of linears launches, asked of the built library on a machine without a GPU (tests/host_dispatch_driver.cpp):
the workspace that every launch of the matrix-core GEMM lays out against the one that the call asked for, and which
kernels serve which lists."""
import os
import random
import shutil
import subprocess

import pytest

from .helpers import ensure_built
from .midm_lists import EDGE_M, EDGES, LISTS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not found")


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    """ask(lists) -> for each list (bits, M, [(N, K, group size), ...]): the workspace asked for and the launches, each as
    (kernel, blocks, workspace of its items as a list of their own, items).  ask.variants: those of the medium-batch kernel that
    are compiled, ask.run: those that lists asked so far run, each as (mode, row blocks, column tiles of a wave, log2 of the K parts)."""
    exe = str(tmp_path_factory.mktemp("dispatch") / "host_dispatch_driver")
    r = subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-host-only", "-Wno-unused-command-line-argument", "-rdynamic",
                        "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2412_01034_amd", "csrc"), os.path.join(ROOT, "tests", "host_dispatch_driver.cpp"), "-o", exe, "-ldl"],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-4000:]
    lib = ensure_built().LIB_PATH

    def ask(lists):
        text = "\n".join("w%d %d %d " % (bits, M, len(shapes)) + " ".join("%d %d %d" % s for s in shapes) for bits, M, shapes in lists)
        r = subprocess.run([exe, lib], input=text + "\n", stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=300)
        assert r.returncode == 0, r.stderr[-4000:]
        out, lines = [], iter(r.stdout.splitlines())
        ask.variants = {tuple(int(n) for n in v.split(",")) for v in next(lines).split()[1:]}
        for bits, M, shapes in lists:
            word, status, need, n = next(lines).split()
            assert word == "list" and status == "0", (bits, M, shapes, status)
            launches = []
            for _ in range(int(n)):
                line, _, variants = next(lines).partition("|")
                kernel, blocks, own, *items = line.split()
                if variants:
                    mode, rb = kernel[len("midm_kernel<"):-1].split(",")
                    ask.run |= {(int(mode), int(rb), *(int(n) for n in v.split("."))) for v in variants.split()}
                launches.append((kernel, int(blocks), int(own), [int(i) for i in items]))
            out.append((int(need), launches))
        return out

    ask.run = set()
    return ask


def mixed_lists():
    """Lists in which several kernels take items: what one of them leaves is another's."""
    lists = [(4, 48, [(256, 256, 128)] * 4 + [(4096, 10880, 128)] * 8),   # 85 groups of 128: the GEMM's alone
             (8, 48, [(256, 256, 128)] * 3 + [(4096, 10880, 128)] * 6),
             (4, 24, [(512, 512, 64)] * 2 + [(4096, 11008, 256)] * 9)]
    rng = random.Random(5)
    for _ in range(400):
        bits = rng.choice((4, 4, 8))
        shapes = []
        while len(shapes) < rng.choice((3, 9, 12, 20, 40)):
            g = rng.choice((64, 128, 128, 128, 256) if bits == 4 else (64, 128, 128, 256))
            N, K = 16 * rng.randint(1, 400), g * rng.randint(1, 11008 // g)
            shapes += [(N, K, g)] * rng.randint(1, 6)
        lists.append((bits, rng.choice((5, 8, 16, 17, 24, 32, 33, 40, 48, 49, 64, 65, 130)), shapes))
    return lists


def test_gemm_launches_fit_the_workspace_asked_for(ask):
    lists = mixed_lists()
    gemm = beside = 0
    for (bits, M, shapes), (need, launches) in zip(lists, ask(lists)):
        for kernel, _, own, items in launches:
            if kernel == "gemm_prep_kernel":
                assert 1 <= len(items) <= 8
                assert own <= need, (bits, M, shapes, items)
                gemm += 1
                beside += any(k.startswith("midm") for k, *_ in launches)
    assert gemm > 300 and beside > 100   # the lists are of the kind meant


@pytest.mark.parametrize("bits,g,shapes", [(4, 64, [(152064, 3584)]), (4, 128, [(152064, 3584)]), (8, 128, [(152064, 3584)]), (8, 128, [(128256, 4096)]),
                                           (4, 64, [(140000, 512)]), (4, 64, [(22016, 4096), (4096, 11008)] * 8), (4, 128, [(1 << 21, 1024)])])
def test_medium_batch_kernel_has_one_block_per_unit_at_most(ask, bits, g, shapes):
    """Lists that its blocks (256 compute units) cannot serve in one round are other kernels': a second round costs as much as the first."""
    lists = [(bits, M, [(N, K, g) for N, K in shapes]) for M in (5, 8, 16, 17, 32, 33, 48, 64)]
    for (_, M, _), (_, launches) in zip(lists, ask(lists)):
        for kernel, blocks, _, _ in launches:
            assert not kernel.startswith("midm") or blocks <= 256, (M, kernel, blocks)


WIDE = [(10240, 8192), (8192, 8192), (57344, 8192), (8192, 28672)]   # 428 MB of nibbles


@pytest.mark.parametrize("bits,M,shapes,medium", [
    (4, 8, WIDE, False), (4, 10, WIDE, False), (4, 16, WIDE, True),       # saved passes against a slower stream
    (4, 7, [(4096, 4096)], False), (4, 16, [(4096, 11008)], True),
    (8, 48, [(8192, 28672)], False), (8, 48, [(22016, 4096)], True),      # against the matrix-core GEMM
    (4, 48, [(12288, 4096), (4096, 4096), (22016, 4096), (4096, 11008)], True), (4, 48, [(4096, 11008)], False),
])
def test_medium_batch_kernel_is_taken_where_it_was_faster(ask, bits, M, shapes, medium):
    [(_, launches)] = ask([(bits, M, [(N, K, 128) for N, K in shapes])])
    assert [k.startswith("midm") for k, *_ in launches] == ([True] if medium else [False] * len(launches)), launches


def test_lists_of_the_gpu_test_run_every_variant(ask):
    """Each is one launch of the medium-batch kernel, and no variant is compiled that none of them runs."""
    ask.run.clear()
    for (bits, M, shapes), (_, launches) in zip(LISTS, ask(LISTS)):
        assert [k.split("<")[0] for k, *_ in launches] == ["midm_kernel"], (bits, M, shapes, launches)
    assert ask.run == ask.variants


def test_edge_lists_of_the_gpu_test_reach_the_kernel_where_they_say(ask):
    lists = [(bits, M, shapes) for bits, shapes, _ in EDGES for M in EDGE_M]
    answers = iter(ask(lists))
    for bits, shapes, taken in EDGES:
        got = tuple(M for M in EDGE_M if any(k.startswith("midm") for k, *_ in next(answers)[1]))
        assert got == taken, (bits, shapes)
