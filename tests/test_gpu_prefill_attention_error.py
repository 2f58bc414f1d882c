"""The prefill attention's error against 64 bits over long prompts of flat scores, where sums carried through
the whole prompt would lose the most: they restart every few hundred keys.

A one-layer model is made so that nothing else rounds: embeddings of +-1 (the RMS is exactly 1), projections
with one weight a row (each key and value is one dyadic product, the keys rotated), no MLP, an output
projection and a head that copy. The stored keys and values are read back, so the 64-bit reference has the
kernel's own inputs; values of 1024 make the copied residual, the final norm and the logits cost no more than
some 6e-8 of the result.

Bound: 2e-7 relative (2-norm). Sums that restart every 256 keys measure 1.0e-7 to 1.7e-7 here, one accumulator 1.6e-7 at 300
keys and 6.3e-7 at 6000."""
import sys

import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _rotate(x, pos):
    half = x.shape[-1] // 2
    ang = pos * 10000.0 ** (-np.arange(half) / half)
    lo, hi = x[..., :half], x[..., half:]
    return np.concatenate([lo * np.cos(ang) - hi * np.sin(ang), hi * np.cos(ang) + lo * np.sin(ang)], -1)


@pytest.mark.parametrize("dh,hkv", [(64, 1), (128, 2)])
def test_long_flat_prompt(dh, hkv):
    from paper_2605_30852_amd.engine import DeviceWeights, Engine
    hq = 4 * hkv
    d = hq * dh
    sh = synth.ModelShape("flat", 1, d, hq, hkv, dh, 256, d + 8, "bf16", n_stages=1, pdm_layers=1, rms_eps=1e-30)
    rng = np.random.default_rng(dh)
    one_hot = lambda n, cols, v: np.eye(d, dtype=np.float32)[cols[:n]] * v  # noqa: E731
    pick = {k: rng.permutation(d) for k in ("q", "k", "v")}
    over = {"embed": rng.choice([-1.0, 1.0], (sh.vocab, d)), "lm_head": np.eye(sh.vocab, d),
            "layer.0.wq": one_hot(d, pick["q"], 0.5), "layer.0.wk": one_hot(hkv * dh, pick["k"], 0.5),
            "layer.0.wv": one_hot(hkv * dh, pick["v"], 1024.0), "layer.0.wo": np.eye(d), "layer.0.wd": np.zeros((d, 256))}
    for name in ("layer.0.attn_norm", "layer.0.mlp_norm", "final_norm"):
        over[name] = np.ones(d)
    w = DeviceWeights(sh, 3, overrides=over)
    worst = 0.0
    for P in (300, 1500, 6000):
        prompt = rng.integers(0, sh.vocab, P).astype(np.int32)
        print(f"[flat prompt dh={dh} P={P}]", file=sys.stderr, flush=True)
        eng = Engine(w, max_tokens=P + 40)
        eng.spd_set_debug(True)
        eng.spd_prefill(prompt)
        k, v = (np.asarray(a, dtype=np.float64).reshape(P, hkv, dh) for a in eng.kv(0, 0, P))
        x = over["embed"][prompt[-1]]
        q = _rotate((0.5 * x[pick["q"]]).reshape(hq, dh), P - 1)
        want = np.empty((hq, dh))
        for h in range(hq):
            s = k[:, h // 4] @ q[h] / np.sqrt(dh)
            p = np.exp(s - s.max())
            want[h] = p @ v[:, h // 4] / p.sum()
        want = want.reshape(-1) + x
        want /= np.sqrt((want * want).mean())
        got = eng.exit_logits()[:d].astype(np.float64)
        eng.close()
        err = np.linalg.norm(got - want) / np.linalg.norm(want)
        print(f"  relative error {err:.2e}", file=sys.stderr, flush=True)
        worst = max(worst, err)
    assert worst <= 2e-7, worst
