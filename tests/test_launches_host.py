"""The kernel launches of the host code, without a GPU: the library runs in a
child process on a stand-in for the HIP runtime (hip_stub.c) that notes every
launch and refuses those of 2^32 threads or more, as HIP does.  Handles of any
size cost nothing there: device pointers are made up."""
from __future__ import annotations

import os
import subprocess
import sys

import pytest

from tests.conftest import ROOT

HEAD = """
import ctypes, sys
sys.path.insert(0, {root!r})
from paper_2106_04034_amd import gsgp
L, P = gsgp.lib(), ctypes.c_void_p
WS, DATA = 1 << 40, 1 << 44  # made-up device addresses
def handle(shapes, **settings):
    s = gsgp.Settings(**settings)
    runs = gsgp.run_descs([(*x, (DATA, DATA, DATA if x[1] else None, DATA if x[1] else None)) for x in shapes])
    cfg, h, size = s.c(), P(0), ctypes.c_size_t(0)
    gsgp.check(L.gsgp_workspace_size(ctypes.byref(cfg), runs, len(shapes), ctypes.byref(size)), "size")
    gsgp.check(L.gsgp_init(ctypes.byref(cfg), runs, len(shapes), P(WS), size.value, None, ctypes.byref(h)), "init")
    gsgp.check(L.gsgp_eval_population(h, None, None), "eval")
    return h
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("stub") / "libhip_stub.so")
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(ROOT, "tests", "hip_stub.c")])
    return so


@pytest.fixture
def launches(stub, tmp_path):
    """run(code, lineage) -> [(kernel, grid x, block x, device)] of the child."""
    def run(code, lineage=""):
        log = tmp_path / "log"
        env = dict(os.environ, LD_PRELOAD=stub, HIP_STUB_LOG=str(log))
        if lineage:
            env["HIP_STUB_LINEAGE"] = lineage
        out = subprocess.run([sys.executable, "-c", HEAD.format(root=ROOT) + code], env=env, cwd=ROOT,
                             capture_output=True, text=True, timeout=120)
        assert out.returncode == 0, out.stderr[-2000:]
        rows = [l.split() for l in log.read_text().splitlines()]
        return [(r[0], int(r[1]), int(r[4]), int(r[5])) for r in rows]
    return run


def test_semantics_of_more_than_2_to_32_values(launches):
    """8,192 individuals on 1,000,000 FP64 cases: every value has its thread."""
    got = launches("""
h = handle([(1_000_000, 0, 1)], pop_size=8192, pool_size=16, genome_len=15)
gsgp.check(L.gsgp_get_semantics(h, 0, 0, P(DATA)), "semantics")
""")
    threads = [g * b for k, g, b, _ in got if "k_fetch_semantics" in k]
    assert sum(threads) >= 8192 * 1_000_000 and max(threads) < 2**32


def test_more_than_2_to_26_genomes(launches):
    """17 pools of 2^22 trees: a wave a genome, over all runs."""
    got = launches("handle([(64, 0, 1)] * 17, pop_size=4, pool_size=1 << 22, genome_len=1, n_generations_max=1)")
    waves = [g * b // 64 for k, g, b, _ in got if "k_compile" in k]
    assert sum(waves) >= 17 * (4 + (1 << 22)) and max(waves) * 64 < 2**32


RECONSTRUCT = """
h = handle([(100_000, 0, 2)], pop_size=1024, pool_size=1024, genome_len=15, n_generations_max={gen})
gsgp.check(L.gsgp_generation(h, {gen}, None), "generation")
size = ctypes.c_size_t(0)
gsgp.check(L.gsgp_reconstruct_scratch_size(h, 0, {gen}, 0, {n}, ctypes.byref(size)), "size")
gsgp.check(L.gsgp_reconstruct(h, 0, {gen}, 0, P(DATA), {n}, P(DATA), P(DATA), size.value), "reconstruct")
"""


def test_programs_of_a_lineage_on_many_cases(launches):
    """1,500 programs on 6,000,000 cases: a wave a program and 128 cases."""
    got = launches(RECONSTRUCT.format(gen=9, n=6_000_000), "600 500 1000 5000")
    waves = [g * b // 64 for k, g, b, _ in got if "k_interpret_list" in k]
    assert sum(waves) >= 1500 * 6_000_000 // 128 and max(waves) * 64 < 2**32


def test_replay_of_a_small_lineage_on_many_cases(launches):
    """Three rows on 300,000,000 cases: a wave for four cases."""
    got = launches(RECONSTRUCT.format(gen=2, n=300_000_000), "3 3 4 5")
    blocks = [(g, g * b) for k, g, b, _ in got if "k_replay_lineage" in k]
    assert sum(g for g, _ in blocks) >= 300_000_000 // 4 and max(t for _, t in blocks) < 2**32


def test_every_launch_goes_to_the_handles_device(launches):
    """A handle of device 0 with device 1 current, on the NULL stream, which
    belongs to the current device."""
    got = launches("""
import numpy as np
h = handle([(5_000, 100, 2)], pop_size=1024, pool_size=64, genome_len=15, n_generations_max=60)
hip = ctypes.CDLL(None)
hip.hipSetDevice(1)
def call(name, *args):
    gsgp.check(getattr(L, name)(h, *args), name)
    d = ctypes.c_int(-1)
    hip.hipGetDevice(ctypes.byref(d))
    assert d.value == 1, name
out, i4 = np.zeros(1 << 20), np.zeros(4, np.int32)
p = P(out.ctypes.data)
call("gsgp_eval_population", None, None)
call("gsgp_time_eval", p)
call("gsgp_generation", 20, p)
rec = np.zeros((2, 1024), gsgp.RECORD_DTYPE)
call("gsgp_generation_replay", 2, P(rec.ctypes.data), None, p)
call("gsgp_time_stages", 2, p)
call("gsgp_set_launch", 2, 8, 1, 0)
call("gsgp_autotune", P(i4.ctypes.data))
call("gsgp_get_fitness", 0, p, p)
call("gsgp_get_semantics_rows", 0, 0, 0, 2, p)
call("gsgp_get_stats", 0, 0, 5, p)
size = ctypes.c_size_t(0)
call("gsgp_reconstruct_scratch_size", 0, 20, 0, 100, ctypes.byref(size))
call("gsgp_reconstruct", 0, 20, 0, P(DATA), 100, P(DATA), P(DATA), size.value)
call("gsgp_reconstruct_static", 0, 20, 0, P(DATA), 100, P(DATA))
blob = ctypes.create_string_buffer(1 << 28)
call("gsgp_checkpoint_save", blob, 1 << 28)
call("gsgp_checkpoint_load", blob, 1 << 28)
""", "3 3 4 5")
    assert len(got) > 30 and {k for k, _, _, device in got if device != 0} == set()
