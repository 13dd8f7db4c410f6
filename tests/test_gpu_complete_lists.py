"""Rows whose candidate list holds every column that can be drawn, against the oracle: rows of which an
allow-list leaves a few finite columns, and vocabularies short enough to be listed whole.  Also nuclei
wider than the list under a row maximum far above its threshold."""
import numpy as np
import pytest

import parity_util as P
from paper_2512_00719_amd import binding, synth

pytestmark = pytest.mark.gpu

CONTROLS = [dict(), dict(top_k=50, top_p=0.9), dict(top_p=0.95), dict(top_k=1000), dict(temperature=0.0), dict(min_p=0.05),
            dict(top_k=1000, top_p=0.97, min_p=0.01), dict(top_k=3000, top_p=0.99), dict(top_p=0.0), dict(top_k=1),
            dict(top_p=0.999, rep_penalty=0.8), dict(rep_penalty=0.9), dict(top_k=20, pres_penalty=-0.2)]


def _params(rng, B, history):
    rows = [dict(CONTROLS[b % len(CONTROLS)]) for b in range(B)]
    base = dict(temperature=None, top_k=0, top_p=1.0, min_p=0.0, rep_penalty=1.1 if history else 1.0, freq_penalty=0.2 if history else 0.0,
                pres_penalty=0.1 if history else 0.0)
    cols = {k: [r.get(k, v if v is not None else float(rng.choice([0.6, 1.0, 1.3]))) for r in rows] for k, v in base.items()}
    return synth.make_params(B, n_prompt=30, **{k: np.array(v, np.int32 if k == "top_k" else np.float32) for k, v in cols.items()})


def _check(name, z, dtype, rng, history, hot_share=0.0, steps=(0, 1), id_pool=None):
    B, V = z.shape
    logits = synth.f32_to_bf16_bits(z) if dtype == "bf16" else z
    lens = rng.integers(1, min(900, 3 * V) + 1, B) if history else np.zeros(B, np.int64)
    hist_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    hist_ids = np.concatenate([rng.choice(id_pool[b] if id_pool is not None else V, int(n)) for b, n in enumerate(lens)]).astype(np.int32)
    hot = np.sort(rng.choice(V, max(1, int(V * hot_share)), replace=False)).astype(np.int32) if hot_share else None
    w = synth.Workload(name, B, V, dtype, logits, _params(rng, B, history), hist_ptr, hist_ids, hot_ids=hot)
    out = []
    for step in steps:
        ids, dg = P.run_gpu(w, step)
        P.compare(ids, dg, P.run_oracle(w, step), range(B))
        assert not (dg["flags"] & binding.DIAG_ERROR).any()
        out.append(dg)
    return out


@pytest.mark.parametrize("dtype,V", [("f32", 40_963), ("f32", 128_256), ("bf16", 128_256)])
@pytest.mark.parametrize("history,hot_share", [(False, 0.0), (True, 0.0), (True, 0.2)])
@pytest.mark.parametrize("allowed", [1, 3, 60, 700, 2000, 5000])
def test_rows_with_an_allow_list(dtype, V, history, hot_share, allowed):
    rng = np.random.default_rng(V + allowed + history)
    B = 26
    z = np.full((B, V), -np.inf, np.float32)
    pool = []
    for b in range(B):
        ids = rng.choice(V, allowed, replace=False)
        z[b, ids] = rng.standard_normal(allowed) * 2.0
        pool.append(np.concatenate([ids, rng.choice(V, 50)]))
    for dg in _check(f"allow-{allowed}", z, dtype, rng, history, hot_share, steps=(0,), id_pool=pool):
        if 60 <= allowed <= 2000 and dtype == "f32":
            # lists of one value in a bucket, rows that raise logits and bare top-k above the list stay the general kernel's
            assert ((dg["flags"] & binding.DIAG_GENERAL) > 0).sum() <= 10


@pytest.mark.parametrize("dtype,V", [("f32", 1), ("f32", 2), ("f32", 63), ("f32", 257), ("f32", 1023), ("f32", 1024), ("f32", 1025), ("f32", 3072),
                                     ("f32", 3073), ("f32", 6145), ("f32", 8191), ("f32", 8192), ("bf16", 5), ("bf16", 2047), ("bf16", 2049),
                                     ("bf16", 3073), ("bf16", 6144), ("bf16", 12_288), ("bf16", 12_289), ("bf16", 16_383), ("bf16", 16_384)])
@pytest.mark.parametrize("history", [False, True])
def test_short_vocabularies(dtype, V, history):
    rng = np.random.default_rng(V + history)
    z = (rng.standard_normal((39, V)) * 1.5).astype(np.float32)
    z[13:26, rng.permutation(V)[: V // 2]] = -np.inf
    z[26:, V - 1] = 25.0
    out = _check(f"short-{V}", z, dtype, rng, history, hot_share=0.2 if V > 100 and history else 0.0)
    untruncated = np.isin(np.arange(39) % len(CONTROLS), (0, 11))
    assert all((((dg["flags"] & binding.DIAG_WIDE) > 0)[untruncated] == (V > 1024)).all() for dg in out)
    if dtype == "f32" and 1023 <= V <= 3073:  # (rows with very many equal values may still be handed on)
        assert all(((dg["flags"] & binding.DIAG_GENERAL) > 0).sum() <= 4 for dg in out)


def test_more_short_rows_than_one_launch_takes():
    rng = np.random.default_rng(3)
    B, V = 4200, 513
    z = rng.standard_normal((B, V)).astype(np.float32)
    w = synth.Workload("short-many", B, V, "f32", z, _params(rng, B, False), np.zeros(B + 1, np.int64), np.zeros(0, np.int32))
    ids, dg = P.run_gpu(w, 0)
    rows = list(range(0, B, 101)) + [4095, 4096, 4199]
    P.compare(ids, dg, P.run_oracle(w, 0, rows=rows), rows)


@pytest.mark.parametrize("V", [128_256, 270_001])
def test_wide_nuclei_under_a_high_maximum(V):
    rng = np.random.default_rng(V)
    B = 12
    z = (rng.standard_normal((B, V)) * 0.3).astype(np.float32)
    z[np.arange(B), rng.integers(0, V, B)] = 15.5 + rng.random(B).astype(np.float32)   # holds nearly all of the mass ...
    params = synth.make_params(B, temperature=1.0, top_p=0.99)                         # ... and the nucleus wants more
    w = synth.Workload("high-max", B, V, "f32", z, params, np.zeros(B + 1, np.int64), np.zeros(0, np.int32))
    for step in (0, 1):
        ids, dg = P.run_gpu(w, step)
        P.compare(ids, dg, P.run_oracle(w, step), range(B))
        assert (dg["n_survivors"] > 5000).any()
        # (a cut inside the list, where a thousand columns share a few buckets, is the general kernel's)
        assert not (dg["flags"] & binding.DIAG_GENERAL)[dg["n_survivors"] > 2000].any()


@pytest.mark.parametrize("dtype,V", [("f32", 128_256), ("bf16", 200_000)])
@pytest.mark.parametrize("allowed", [1, 40, 2000, 20_000])
def test_min_p_on_masked_rows(dtype, V, allowed):
    """Few finite columns where the threshold is sampled (two tiles at the start of each sixteenth of a row), more than a
    list holds elsewhere; min-p leaves some of them, and its bound is the threshold."""
    rng = np.random.default_rng(V + allowed)
    B, T = 12, 1024 if dtype == "f32" else 2048
    col = np.arange(V)
    sampled = np.isin(col // T, [w * (V // T) // 16 + k for w in range(16) for k in (0, 1)])
    z = np.full((B, V), -np.inf, np.float32)
    for b in range(B):
        ids = np.concatenate([rng.choice(col[~sampled], allowed, replace=False), rng.choice(col[sampled], 20, replace=False)])
        z[b, ids] = rng.standard_normal(ids.size) * 2.0
    n = 30
    hist_ids = rng.integers(0, V, B * n).astype(np.int32)
    params = synth.make_params(B, temperature=np.resize([1.0, 0.7], B).astype(np.float32), min_p=np.resize([0.05, 0.2, 0.5], B).astype(np.float32),
                               top_p=np.resize([1.0, 1.0, 1.0, 0.9], B).astype(np.float32), rep_penalty=1.1, n_prompt=10)
    w = synth.Workload(f"min-p-{allowed}", B, V, dtype, synth.f32_to_bf16_bits(z) if dtype == "bf16" else z, params,
                       np.arange(B + 1, dtype=np.int64) * n, hist_ids)
    ids, dg = P.run_gpu(w, 0)
    P.compare(ids, dg, P.run_oracle(w, 0), range(B))
    assert not (dg["flags"] & binding.DIAG_GENERAL).any()


@pytest.mark.parametrize("dtype,V", [("f32", 1500), ("f32", 5865), ("f32", 8191), ("bf16", 7189), ("f32", 128_256)])
@pytest.mark.parametrize("values", [1, 3, 40])
@pytest.mark.parametrize("hot_share", [0.0, 0.3])
def test_cuts_among_many_ties(dtype, V, values, hot_share):
    """Lists whose columns share a few values: the bucket that holds a cut, or the draw's range of ids (an allow-list of
    neighbours), has more members than are resolved at once."""
    rng = np.random.default_rng(V + values)
    B = 26
    if V > 10_000:  # an allow-list of neighbouring ids
        z = np.full((B, V), -np.inf, np.float32)
        z[:, 70_000:73_000] = rng.integers(0, values, (B, 3000)) * np.float32(0.25)
    else:
        z = (rng.integers(0, values, (B, V)) * np.float32(0.25)).astype(np.float32)
        z[::2] += (rng.random((z[::2].shape[0], V)) < 0.01) * np.float32(3.0)
    pool = [np.arange(70_000, 73_000) if V > 10_000 else np.arange(V)] * B
    for history in (False, True):
        for dg in _check(f"ties-{values}", z, dtype, rng, history, hot_share, steps=(0,), id_pool=pool):
            handed = (dg["flags"] & binding.DIAG_GENERAL) > 0
            # (a sampled list whose threshold is one of the tied values certifies none of them)
            assert V > 10_000 or not handed.any(), np.flatnonzero(handed)


@pytest.mark.parametrize("dtype,V", [("f32", 900), ("f32", 6000), ("bf16", 7000), ("f32", 40_960), ("f32", 128_256), ("bf16", 128_256), ("f32", 270_001)])
@pytest.mark.parametrize("allowed,hot_share", [(1, 0.0), (50, 0.2), (700, 0.0)])
@pytest.mark.parametrize("history", [False, True])
def test_masks_of_the_types_lowest_value(dtype, V, allowed, hot_share, history):
    """Columns masked with the lowest finite value instead of -inf: finite logits without mass, which a temperature below
    one takes to -inf."""
    rng = np.random.default_rng(V + allowed)
    B = 26
    lowest = np.float32(np.finfo(np.float32).min) if dtype == "f32" else synth.bf16_bits_to_f32(np.array([0xFF7F], np.uint16))[0]
    z = np.full((B, V), lowest, np.float32)
    pool = []
    for b in range(B):
        ids = rng.choice(V, allowed, replace=False)
        z[b, ids] = rng.standard_normal(allowed) * 2.0
        pool.append(ids)
    _check(f"lowest-{allowed}", z, dtype, rng, history, hot_share, steps=(0,), id_pool=pool)
