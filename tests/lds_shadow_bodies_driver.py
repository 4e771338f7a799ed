"""Runs kernels of the race-detection build (libspvar_shadow.so, loaded with SPVAR_LIBRARY=shadow)
against the oracle, bit for bit, and prints the detector's counts as one JSON line per phase:

* "exchange": tempering ladders split into groups of 4 slots and more, whose in-group swaps store
  words that also hold boundary slots' bytes (instance in LDS and in global memory, one and two
  chains, a ladder that is no multiple of four).

Run by tests/test_gpu_lds_shadow_bodies.py in a process of its own, with a phase's name."""
import json
import os
import sys

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import oracle  # noqa: E402
import paper_1706_07826_amd as spv  # noqa: E402
import spvar_inputs as si  # noqa: E402
from tests.lds_shadow_driver import say, with_env  # noqa: E402


def exchange(ctx):
    cube = si.cubic_lattice(4, "gauss", seed=9, scale_log2=10)
    P = spv.Problem.from_instance(cube)
    class_passes = 0
    for label, K, G, chains, big in (("quad_groups", 8, 2, 1, 0), ("quad_groups_two_chains", 16, 4, 2, 0),
                                     ("eight_slots", 32, 4, 1, 0), ("eight_slots_big", 32, 4, 2, 1),
                                     ("off_the_quads", 14, 2, 2, 0)):
        say(f"[shadow] exchange {label}: K={K} G={G} chains={chains}")
        betas = si.geometric_betas(0.2, 5.0, K)
        got = with_env({"SPVAR_PT_GROUPS": G, "SPVAR_PT_BIG": big},
                       lambda: spv.spv_pt_sample(ctx, P, betas, 2, chains, 120, 4))
        want = oracle.pt_sample(cube, betas, 2, chains, 120, seed=4)
        for key in ("final_spins", "final_E", "top_E", "top_count", "top_spins"):
            assert np.array_equal(got[key].cpu().numpy(), want[key]), (label, key)
        class_passes += 2 * G * 120 * cube.n_colours
    return dict(class_passes=class_passes)


def main():
    assert "race detection" in spv._lib.spv_version().decode(), spv._lib.spv_version()
    ctx = spv.Context(0)
    for phase in sys.argv[1:]:
        spv.spv_debug_lds_shadow(ctx, reset=True)
        extra = {"exchange": exchange}[phase](ctx)
        print(json.dumps(dict(phase=phase, **spv.spv_debug_lds_shadow(ctx, reset=True), **extra)), flush=True)


if __name__ == "__main__":
    main()
