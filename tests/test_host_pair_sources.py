"""The kernels that the library launches for a pass's collisions, on the CPU
under the workgroup emulator (tests/host_emu) with the address and undefined-
behaviour sanitizers, in forward, reverse and reshuffled thread and workgroup
order: the pairs drawn before the pass and the instance that takes them, the
instance that draws its pairs in chunks (each followed by the general instance
over the tiles it left) equal the general instance alone bit for bit, in passes
of both halves, of one half and in a collision call; the collision-heavy kernel
has one result in every order, the serial kernel's up to its fixed point."""
import os
import shutil
import struct
import subprocess

import numpy as np
import pytest

import oracle as O
from paper_2602_15130_amd import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
EMU = os.path.join(ROOT, "tests", "host_emu")
CSRC = os.path.join(ROOT, "paper_2602_15130_amd", "csrc")
FORWARD, REVERSE, SHUFFLE = ORDERS = 0, 1, 2
GENERAL, DRAWN, CHUNKS, HEAVY, SERIAL, DRAWN_BY_TILE = range(6)
DO_B, DO_A, COLLIDE_ONLY = 1, 2, 4


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("emu_pairs")
    src = d / "csrc"
    shutil.copytree(CSRC, src)
    # the launch's dynamic LDS is an array of the harness
    heavy = src / "pic_collide_heavy.hpp"
    heavy.write_text(heavy.read_text().replace("extern __shared__", "extern"))
    exe = str(d / "pair_sources")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g1", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-fno-omit-frame-pointer", "-I", EMU,
                    "-I", str(src), "-o", exe, os.path.join(EMU, "pair_sources.cpp")],
                   check=True, capture_output=True, text=True, timeout=600)
    return exe, d


_states = {}


def _oracle_state(prob, disc, steps):
    at = (id(prob), steps)
    if at not in _states:
        o = O.Sim(prob, disc, 5, 0)
        assert o.init() == 0 and o.step(steps) == 0
        cs = o.get(o.CELL_START).astype(np.int32)
        key = np.repeat(np.arange(len(cs) - 1, dtype=np.int32), np.diff(cs))
        _states[at] = b"".join(a.tobytes() for a in (
            o.get(o.V), cs, key, o.get(o.X), o.get(o.ID).astype(np.int32), o.get(o.E)))
    return _states[at]


def _run(harness, prob, disc, source, mode, order, precision=0, steps=1, lds_n=1920, split=1,
         scan=0):
    from paper_2602_15130_amd import pic as P
    exe, d = harness
    blob = bytes(P.make_problem(prob)) + bytes(P.make_disc(disc))
    blob += struct.pack("<QQqiiiiiiii", 5, 11, steps, precision, order, source, mode, lds_n, split,
                        scan, 0)
    blob += _oracle_state(prob, disc, steps)
    (d / "in.bin").write_bytes(blob)
    r = subprocess.run([exe, str(d / "in.bin"), str(d / "out.bin")], capture_output=True, text=True,
                       timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    raw = (d / "out.bin").read_bytes()
    n, nn = disc["np"], int(np.prod(disc["nc"]))
    state = np.frombuffer(raw, np.float64, 6 * n)
    at = state.nbytes
    cells = np.frombuffer(raw, np.int32, n + nn, at)
    at += cells.nbytes
    cnt = np.frombuffer(raw, np.uint64, 4, at)
    flags = np.frombuffer(raw, np.int32, 4, at + 32)
    left = np.frombuffer(raw, np.int32, 1, at + 48)[0]
    assert not flags.any()
    return {"state": state, "cells": cells, "accepted": int(cnt[0]), "left": int(left)}


def _cfg(nc, nbar, pairs, navg):
    n = int(np.prod(nc))
    prob = W.cfg_problem(two_way=True,
                         collisionality=pairs / (0.5 * (nbar - 0.9) * W.NU_MAX_T / W.T_CFG * 1e-3))
    return prob, {"nc": nc, "np": nbar * n + 3, "dt": 1e-3, "navg": navg, "cg_tol": 1e-12,
                  "cg_max_iter": 5000}


# mesh, particles per cell, pairs per outcome, outcomes
CASES = {"few": _cfg((4, 4, 4), 32, 0.06, 16),
         "many_outcomes": _cfg((3, 3, 4), 20, 0.02, 203),
         "ragged": _cfg((7, 5, 6), 3, 0.4, 6),       # N_avg no multiple of four, some empty cells
         "over_four": _cfg((4, 4, 4), 40, 4.2, 3),   # outcomes of more pairs than a list takes
         "overflow": _cfg((4, 3, 4), 32, 0.9, 20),   # lists that overflow
         "chunks": _cfg((3, 4, 3), 30, 2.0, 70),     # several chunks and blocks of items
         "over_96": _cfg((3, 3, 3), 110, 90.0, 2),   # outcomes over a chunk's most pairs
         "large_cells": _cfg((3, 3, 3), 350, 0.5, 3)}


def _same(a, b):
    return np.array_equal(a["state"], b["state"]) and np.array_equal(a["cells"], b["cells"]) and \
        a["accepted"] == b["accepted"]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("case", list(CASES))
def test_pair_sources_agree_in_every_order(harness, case, precision):
    prob, disc = CASES[case]
    halves = (DO_A, DO_B, COLLIDE_ONLY) if case in ("few", "ragged", "overflow") else (COLLIDE_ONLY,)
    for mode in (DO_B | DO_A, *halves):
        ref = _run(harness, prob, disc, GENERAL, mode, FORWARD, precision)
        assert ref["accepted"] > 0
        # the whole pass in several orders, the others in one
        whole = ORDERS if case == "few" else (REVERSE, SHUFFLE)
        for order in whole if mode == DO_B | DO_A else (SHUFFLE,):
            for source in (DRAWN, DRAWN_BY_TILE, CHUNKS):
                got = _run(harness, prob, disc, source, mode, order, precision)
                assert _same(got, ref), (mode, order, source)
                if case in ("large_cells", "over_96") or (case == "overflow" and source != CHUNKS):
                    assert got["left"] > 0
                if case in ("few", "many_outcomes") or (case == "chunks" and source == CHUNKS):
                    assert got["left"] == 0


def test_scanned_event_lists_change_no_bit(harness):
    """The mixed form's event lists (about 64 events a tile, sorted from 25 on)
    scanned instead (PIC_SORT_EVENTS=0, which the library reads)."""
    prob, disc = _cfg((4, 4, 4), 32, 1.0, 8)
    ref = _run(harness, prob, disc, GENERAL, DO_B | DO_A, SHUFFLE, 1)
    assert ref["accepted"] > 100
    assert _same(_run(harness, prob, disc, GENERAL, DO_B | DO_A, SHUFFLE, 1, scan=1), ref)
    from paper_2602_15130_amd import pic as P
    with open(P.LIB_PATH, "rb") as f:
        assert b"PIC_SORT_EVENTS" in f.read()


# mesh, particles per cell, pairs per outcome, outcomes; workgroups per cell, LDS particles
HEAVY_CASES = {"lanes": (_cfg((3, 3, 3), 60, 9.0, 24), 1, 128),
               "two_waves": (_cfg((3, 3, 3), 120, 80.0, 6), 1, 256),
               "one_wave": (_cfg((3, 3, 3), 120, 101.0, 5), 1, 256),
               "scratch": (_cfg((3, 3, 3), 330, 210.0, 3), 1, 640),
               "split": (_cfg((3, 3, 3), 100, 20.0, 24), 4, 256),
               "split_scratch": (_cfg((3, 3, 3), 330, 210.0, 4), 3, 640),
               "global_sums": (_cfg((3, 3, 3), 60, 9.0, 12), 1, 32),
               "split_global_sums": (_cfg((3, 3, 3), 60, 9.0, 24), 2, 32)}


@pytest.mark.parametrize("case", list(HEAVY_CASES))
def test_collision_heavy_kernel_in_every_order(harness, case):
    """<dv> within the fixed point's quantum (below 2^-45 of g_max here) times the
    pairs of a particle, and the rounding of the serial sums over N_avg."""
    (prob, disc), split, lds_n = HEAVY_CASES[case]
    ref = _run(harness, prob, disc, SERIAL, 0, FORWARD, steps=0)
    got = [_run(harness, prob, disc, HEAVY, 0, o, steps=0, split=split, lds_n=lds_n) for o in (REVERSE, SHUFFLE)]
    assert ref["accepted"] > 100
    for g in got:
        np.testing.assert_array_equal(g["state"], got[0]["state"])
        assert g["accepted"] == ref["accepted"]
    assert np.abs(got[0]["state"] - ref["state"]).max() <= 1e-13 * W.GMAX_CFG
