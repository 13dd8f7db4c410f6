"""p~ of the drawn token is the float32 nearest to the one that 64-bit sums give, whichever kernel weighs the
row's columns: short vocabularies, rows with few finite columns, rows at any element's address, vocabularies
of 2^18 columns and more.  The weights are 2^44 fixed point relative to the largest, each rounded once."""
import numpy as np
import pytest

import parity_util as P
from paper_2512_00719_amd import binding, synth

pytestmark = pytest.mark.gpu

LIST_CONTROLS = [dict(top_k=50, top_p=0.9), dict(top_k=900), dict(top_p=0.6), dict(min_p=0.02), dict(top_k=300, min_p=0.001), dict()]


def _params(controls, B, temperature):
    cols = {k: np.array([c.get(k, v) for c, _ in zip(controls * B, range(B))]) for k, v in dict(top_k=0, top_p=1.0, min_p=0.0).items()}
    return synth.make_params(B, temperature=temperature, top_k=cols["top_k"].astype(np.int32), top_p=cols["top_p"].astype(np.float32),
                             min_p=cols["min_p"].astype(np.float32))


def _errors(w, dev, dg_want, steps=4):
    """Checks ids and p~ of `steps` calls; returns the number of rows per diagnostics flag of dg_want."""
    seen = np.zeros(len(dg_want), int)
    for step in range(steps):
        ids, dg = P.run_gpu(w, step, dev=dev)
        want = P.run_oracle(w, step)
        P.compare(ids, dg, want, range(w.B))
        for r, o in enumerate(want):
            if int(ids[r]) != o.id or dg["flags"][r] & (binding.DIAG_GREEDY | binding.DIAG_ERROR):
                continue
            got = float(dg["p_chosen"][r])
            bad = [abs(got - p) - p * (1.001 * 2.0 ** -24 + o.n * 2.0 ** -45) - 2.0 ** -45 for p in (o.p_chosen, *o.alt_p)]
            assert min(bad) <= 0.0, (step, r, hex(int(dg["flags"][r])), got, o.p_chosen, abs(got - o.p_chosen) / o.p_chosen)
        for i, f in enumerate(dg_want):
            seen[i] += int(((dg["flags"] & f) > 0).sum())
    return seen


def _workload(name, z, dtype, params):
    B, V = z.shape
    return synth.Workload(name, B, V, dtype, synth.f32_to_bf16_bits(z) if dtype == "bf16" else z, params, np.zeros(B + 1, np.int64),
                          np.zeros(0, np.int32))


@pytest.mark.parametrize("kind,dtype,V", [("short", "f32", 700), ("short", "f32", 6000), ("short", "bf16", 3000), ("masked", "f32", 50_048),
                                          ("unaligned", "f32", 50_001), ("large", "f32", 270_000), ("aligned", "f32", 50_048)])
def test_listed_columns(kind, dtype, V):
    rng = np.random.default_rng(V)
    B = 24
    z = synth.zipf_profile_logits(B, V, 1.0, 1.0, rng, "f32", rng.permutation(V))
    if kind == "masked":
        keep = np.zeros(V, bool)
        keep[rng.choice(V, 1500, replace=False)] = True
        z[:, ~keep] = -np.inf
    controls = LIST_CONTROLS if kind == "short" else LIST_CONTROLS[:5] if kind == "masked" else LIST_CONTROLS[:2] + [dict(min_p=0.05)]
    w = _workload(f"weights-{kind}", z, dtype, _params(controls, B, np.resize([0.6, 0.8, 1.0], B).astype(np.float32)))
    wide, general = _errors(w, P.to_device(w), (binding.DIAG_WIDE, binding.DIAG_GENERAL))
    assert general <= 4 and (kind != "short" or wide == 0 or V < 8192)
