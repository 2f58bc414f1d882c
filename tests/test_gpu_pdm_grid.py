"""The draft module's projections under a cap on their workgroups (spd_set_pdm_grid): the same bits as without
one, whether a workgroup has several jobs (caps of 1 and 3), an uneven number of them (7), or one. Models on both
forms of the draft module's rows: matrix cores (the wide pipeline, widths that fill no tile) and vector GEMVs."""
import sys

import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

NARROW = synth.ModelShape("narrow", 3, 264, 2, 1, 64, 520, 777, "bf16", n_stages=3, pdm_layers=2)


@pytest.mark.parametrize("shape", [synth.WIDE, NARROW, synth.MID, synth.GQA8.with_(n_stages=5)], ids=lambda s: s.name)
def test_same_bits_under_any_grid(shape):
    from paper_2605_30852_amd.engine import DeviceWeights, Engine
    w = DeviceWeights(shape, 17)
    prompt = synth.prompt(shape, 5, 70)
    got = []
    for wgs in (0, 1, 3, 7, 4000):
        print(f"[{shape.name} grid {wgs}]", file=sys.stderr, flush=True)
        eng = Engine(w, max_tokens=200)
        eng.spd_set_debug(True)
        eng.spd_set_pdm_grid(wgs)
        first = eng.spd_prefill(prompt)
        log = eng.spd_run_steps(2 * shape.n_stages + 6, want_log=True)
        a = log[-2]["inflight"]
        got.append((first, log, eng.pdm_hidden()[:a], eng.pdm_logits(), eng.tokens()))
        eng.close()
    for first, log, hidden, logits, tokens in got[1:]:
        assert first == got[0][0] and log == got[0][1]
        assert np.array_equal(hidden, got[0][2]) and np.array_equal(logits, got[0][3])
        assert np.array_equal(tokens, got[0][4])
