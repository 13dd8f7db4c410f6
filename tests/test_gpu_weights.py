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


def _errors(w, dev, dg_want, steps=4, check_s_k=False):
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
            if check_s_k and dg["flags"][r] & (binding.DIAG_WIDE | binding.DIAG_PATTERN) == binding.DIAG_WIDE and o.S_k_used:  # the mass of the row relative to its maximum
                assert abs(float(dg["s_k"][r]) - o.S_k) <= 1e-9 * o.S_k, (step, r, hex(int(dg["flags"][r])), float(dg["s_k"][r]) / o.S_k - 1.0)
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


@pytest.mark.parametrize("kind,dtype,V", [("unaligned", "f32", 50_001), ("unaligned", "bf16", 50_001), ("large", "f32", 270_000),
                                          ("large", "bf16", 270_000), ("high", "f32", 50_048), ("high", "f32", 270_000)])
@pytest.mark.parametrize("hot_set,history", [(False, False), (True, False), (True, True)])
def test_survivors_beyond_the_list(kind, dtype, V, hot_set, history):
    """Rows of the sliced kernels that the general kernel used to serve: a nucleus wider than the list, a min-p
    cut below it, top-k above it, and ("high") wide nuclei under a maximum that holds nearly all of the mass."""
    rng = np.random.default_rng(V + 3 * hot_set + history)
    B = 18
    z = (rng.standard_normal((B, V)) * rng.choice([0.3, 1.0], B)[:, None]).astype(np.float32)
    if kind == "high":
        z[np.arange(B), rng.integers(0, V, B)] = 16.5 + rng.random(B).astype(np.float32)
        params = _params([dict(top_p=0.9995), dict(top_p=0.9999), dict(top_p=0.9992, min_p=1e-9)], B, 1.0)
    else:
        params = _params([dict(top_p=0.9), dict(top_k=5000), dict(min_p=0.01), dict(top_p=0.95, min_p=0.001), dict(top_p=0.7), dict(top_k=20_000)], B,
                         np.resize([1.0, 0.8, 1.2], B).astype(np.float32))
    n = 200 if history else 0
    if history:
        params["rep_penalty"], params["freq_penalty"], params["n_prompt"] = 1.1, 0.2, 50
        params["rep_penalty"][4::6] = 0.9  # raises logits: no list
    w = synth.Workload(f"weights-{kind}", B, V, dtype, synth.f32_to_bf16_bits(z) if dtype == "bf16" else z, params,
                       np.arange(B + 1, dtype=np.int64) * n, rng.integers(0, V, B * n).astype(np.int32),
                       hot_ids=np.sort(rng.choice(V, V // 10, replace=False)).astype(np.int32) if hot_set else None)
    wide, general, pattern = _errors(w, P.to_device(w), (binding.DIAG_WIDE, binding.DIAG_GENERAL, binding.DIAG_PATTERN), steps=2, check_s_k=True)
    assert wide + pattern >= (B if kind != "high" else 4) and (general <= 6 or kind != "unaligned")


@pytest.mark.parametrize("dtype,V,offset", [("f32", 50_048, 0), ("bf16", 50_048, 0), ("f32", 50_001, 0), ("f32", 270_000, 0), ("f32", 8193, 3)])
@pytest.mark.parametrize("hot_set,history", [(False, False), (True, False), (True, True)])
def test_untruncated_rows_of_any_range(dtype, V, offset, hot_set, history):
    """Rows beyond the float32 weights' reach: a few columns hold much of the mass, one holds all but a trace, a spread
    of hundreds, masked columns.  Only a column more than 88 above the rest is the general kernel's."""
    rng = np.random.default_rng(V + 3 * hot_set + history)
    B = 20
    z = (rng.standard_normal((B, V)) * 0.7).astype(np.float32)
    z[0::5, rng.choice(V, 3, replace=False)] = 25.0 + rng.random(3).astype(np.float32)
    z[1::5, rng.integers(0, V)] = 120.0
    z[2::5] *= 60.0
    z[3::5] *= 60.0
    z[3::5, rng.permutation(V)[: V - 400]] = -np.inf
    z[4::5, rng.choice(V, 40, replace=False)] += 30.0
    params = _params([dict()], B, np.resize([1.0, 0.5, 1.3], B).astype(np.float32))
    n = 300 if history else 0
    if history:
        params["rep_penalty"], params["freq_penalty"], params["n_prompt"] = 1.1, 0.2, 50
    w = synth.Workload("weights-all", B, V, dtype, synth.f32_to_bf16_bits(z) if dtype == "bf16" else z, params, np.arange(B + 1, dtype=np.int64) * n,
                       rng.integers(0, V, B * n).astype(np.int32), hot_ids=np.sort(rng.choice(V, V // 10, replace=False)).astype(np.int32) if hot_set else None)
    dev = P.to_device(w)
    if offset:
        import torch
        buf = torch.zeros(B * V + 16, dtype=dev["logits"].dtype, device="cuda:0")
        buf[offset:offset + B * V] = dev["logits"].reshape(-1)
        dev["logits"] = buf[offset:offset + B * V].view(B, V)
    wide, general = _errors(w, dev, (binding.DIAG_WIDE, binding.DIAG_GENERAL))
    assert (general > 0 or dtype == "bf16") and general <= 4 * 4 and wide == 4 * B  # (bfloat16: the pattern counts carry any range)
