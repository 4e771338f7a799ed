"""Runs kernels of the race-detection build (libspvar_shadow.so, loaded with SPVAR_LIBRARY=shadow)
against the oracle, bit for bit, and prints the detector's counts as one JSON line per phase:

* "exchange": tempering ladders split into groups of 4 slots and more, whose in-group swaps store
  words that also hold boundary slots' bytes (instance in LDS and in global memory, one and two
  chains, a ladder that is no multiple of four);
* "records_in_lds": the byte-parallel SA bodies with their records in LDS, one and two words per
  lane, in one launch and streamed (the held-sites body, which takes such problems by default, off);
* "held_sites": the held-sites SA body with one and several quads a workgroup, two to four colour
  classes, streamed, and in a batched launch.

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
from tests.lds_shadow_driver import sample_case, say, with_env  # noqa: E402
from tests.test_gpu_held import _layers  # noqa: E402


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


def records_in_lds(ctx):
    inst = si.chimera(4, seed=3)
    for words in (1, 2):
        for stream in (0, 8):
            sample_case(ctx, f"records_in_lds_w{words}", inst,
                        {"SPVAR_SA_HELD": 0, "SPVAR_SA_WPL": words, "SPVAR_SA_THREADS": 256,
                         "SPVAR_SA_STREAM": stream}, reads=300 if stream else 40)
            shape = spv.spv_sample_last_shape(ctx)
            assert shape["words_per_lane"] == words and (shape["chunks"] > 1) == (stream > 0)
    return {}


def held_sites(ctx):
    for name, inst, env, reads in (("chimera", si.chimera(4, seed=3), {}, 40),
                                   ("quads3", si.chimera(4, seed=3), {"SPVAR_SA_HELD": 3}, 50),
                                   ("streamed", si.chimera(4, seed=3), {"SPVAR_SA_STREAM": 8}, 300),
                                   ("three_classes", _layers([50, 50, 50], 2, 4, 3), {}, 40),
                                   ("four_classes", _layers([40, 40, 40, 40], 2, 4, 4), {}, 40)):
        sample_case(ctx, f"held_{name}", inst, env, reads=reads)
    insts = [_layers([40, 40], 3, 6, 5, 4), _layers([9, 8], 3, 6, 6, 4), _layers([129, 64], 3, 6, 7, 4)]
    reads, seeds, betas = [23, 400, 50], [5, 6, 7], si.linear_betas(0.05, 3.0, 25)
    say("[shadow] held_batch")
    sp, en = spv.spv_sample_batch(ctx, [spv.Problem.from_instance(i) for i in insts], betas, reads, seeds)
    assert spv.spv_batch_last_shape(ctx)["quads_per_item"] == 0
    for b, inst in enumerate(insts):
        oS, oE = oracle.sa_sample(inst, betas, reads=reads[b], seed=seeds[b])
        assert np.array_equal(sp[b].cpu().numpy(), oS) and np.array_equal(en[b].cpu().numpy(), oE), b
    return {}


def main():
    assert "race detection" in spv._lib.spv_version().decode(), spv._lib.spv_version()
    ctx = spv.Context(0)
    for phase in sys.argv[1:]:
        spv.spv_debug_lds_shadow(ctx, reset=True)
        extra = dict(exchange=exchange, records_in_lds=records_in_lds, held_sites=held_sites)[phase](ctx)
        print(json.dumps(dict(phase=phase, **spv.spv_debug_lds_shadow(ctx, reset=True), **extra)), flush=True)


if __name__ == "__main__":
    main()
