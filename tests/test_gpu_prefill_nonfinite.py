"""A prompt token whose embedding is not finite (bf16 model): its own position and, past the first layer, the
later ones, which attend it, become NaN; the positions before it keep the keys and values they have with any other token there,
in every layer of the target and the draft module. Positions sit at the edges of the attention's 32-query
waves and 64-key tiles and of a workgroup's rows (128 at one query head per KV head, 32 at four, 16 at eight),
in a second chunk of rows, and at a prompt's last position.

Bound: the rows before the token may take the plain form of the attention instead of the matrix form, whose
sums run in another order: per position at most the 2e-2 to which the caches are held against the oracle."""
import sys

import numpy as np
import pytest

import synth
from tests.lockstep import REL_HIDDEN

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

G4 = synth.WIDE.with_(name="g4", n_layers=3, n_stages=2, pdm_layers=2)
CASES = [(synth.MHA, 200, 127), (synth.MHA, 200, 64), (synth.MHA, 97, 96), (G4, 130, 63), (G4, 200, 33),
         (synth.GQA8, 100, 17), (synth.MID, 45, 1), (synth.GQA8, 2113, 2100)]


@pytest.mark.parametrize("shape,P,at", CASES, ids=[f"{s.name}-{p}-{a}" for s, p, a in CASES])
def test_earlier_positions_keep_their_caches(shape, P, at):
    from paper_2605_30852_amd.engine import DeviceWeights, Engine
    w = DeviceWeights(shape, 5)
    prompt = np.random.RandomState(P + at).randint(2, shape.vocab, P).astype(np.int32)
    prompt[at] = 1
    got = []
    for bad in (False, True):
        w.t["embed"][1] = float("inf") if bad else 0.02
        w.t["embed"][1, ::2] = float("nan") if bad else -0.02
        print(f"[{shape.name} P={P} at={at} {'not finite' if bad else 'finite'}]", file=sys.stderr, flush=True)
        eng = Engine(w, max_tokens=P + 40, page_seed=3, ws_fill=0xFF)
        eng.spd_prefill(prompt)
        got.append([eng.kv(l, 0, P, pdm=pdm) for pdm, n in ((False, shape.n_layers), (True, shape.pdm_layers))
                    for l in range(n)])
        eng.close()
    for layer, (fine, bad) in enumerate(zip(*got)):
        for x, y in zip(fine, bad):
            x, y = (np.asarray(a, dtype=np.float64).reshape(P, -1) for a in (x, y))
            assert np.isfinite(y[:at]).all(), (layer, np.flatnonzero(~np.isfinite(y[:at]).all(1))[:5])
            assert np.isnan(y[at:at + 1] if layer == 0 else y[at:]).all(), (layer, at)
            err = np.linalg.norm(y[:at] - x[:at], axis=1) / np.linalg.norm(x[:at], axis=1)
            assert (err <= REL_HIDDEN).all(), (layer, int(np.argmax(err)), float(err.max()))
