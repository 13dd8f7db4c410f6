"""Penalties of listed columns, counted through a hash table of the list or a counter per column, against the oracle:
lists and histories on either side of the rule that chooses them, chains that wrap past the table's end, histories
longer than the registers hold, repeats, prompt splits inside the last round of ids, ids outside the vocabulary."""
import numpy as np
import pytest

import parity_util as P
from paper_2512_00719_amd import binding, synth

pytestmark = pytest.mark.gpu

CONTROLS = [dict(top_p=0.95), dict(top_k=20), dict(temperature=0.0), dict(top_k=200, top_p=0.99), dict(min_p=0.02), dict(top_p=0.999)]


def _place(ids):
    """Where the list's hash table looks for a column first (1024 places)."""
    return (np.asarray(ids, np.uint64) * 0x9E3779B1 & 0xFFFFFFFF) >> 22


def _check(V, dtype, n, nnz, crowded=False, beyond=0):
    B = 2 * len(CONTROLS)
    rng = np.random.default_rng(V + 7 * n + nnz)
    z = np.full((B, V), -np.inf, np.float32)
    every = np.arange(V)
    late = every[_place(every) >= 1020] if crowded else every  # (their chains run on from the table's start)
    hist = []
    for b in range(B):
        ids = rng.choice(late, n, replace=False)
        z[b, ids] = rng.standard_normal(n) * 2.0
        pool = np.concatenate([ids, rng.choice(late if crowded else V, n)])  # half of the history is listed, the rest is not
        h = rng.choice(pool, nnz - beyond)
        hist.append(np.concatenate([h, rng.choice([V, V + 5, 2 ** 31 - 1, -1, -2 ** 31], beyond)]).astype(np.int32))
    base = dict(temperature=1.0, top_k=0, top_p=1.0, min_p=0.0)
    cols = {k: np.resize(np.array([c.get(k, v) for c in CONTROLS], np.int32 if k == "top_k" else np.float32), B) for k, v in base.items()}
    n_prompt = np.resize(np.array([0, nnz // 2, max(nnz - 3 - beyond, 0), 1], np.int32), B)
    params = synth.make_params(B, rep_penalty=1.2, freq_penalty=0.05, pres_penalty=0.1, n_prompt=n_prompt, **cols)
    bits = synth.f32_to_bf16_bits(z) if dtype == "bf16" else z
    w = synth.Workload("listed", B, V, dtype, bits, params, np.arange(B + 1, dtype=np.int64) * nnz, np.concatenate(hist))
    valid = synth.Workload("valid", B, V, dtype, bits, params, np.arange(B + 1, dtype=np.int64) * (nnz - beyond),
                           np.concatenate([h[:nnz - beyond] for h in hist]))
    ids, dg = P.run_gpu(w, 0)
    assert not (dg["flags"] & binding.DIAG_ERROR).any()
    assert (((dg["flags"] & binding.DIAG_BAD_HISTORY_ID) > 0) == (beyond > 0)).all()
    P.compare(ids, dg, P.run_oracle(valid, 0), range(B))


@pytest.mark.parametrize("V,dtype", [(128_256, "f32"), (151_936, "bf16")])
@pytest.mark.parametrize("n", [1, 64, 191, 192, 193, 512])
@pytest.mark.parametrize("nnz", [5, 1024, 4097])
def test_the_rules_edges(V, dtype, n, nnz):
    _check(V, dtype, n, nnz)


@pytest.mark.parametrize("V,dtype,n", [(50_001, "f32", 192), (151_936, "bf16", 100), (128_256, "f32", 190), (6000, "f32", 3000), (3000, "bf16", 700)])
@pytest.mark.parametrize("nnz,beyond", [(8191, 0), (8192, 3), (8193, 1), (12_000, 40), (20_001, 9000)])
def test_long_histories(V, dtype, n, nnz, beyond):
    _check(V, dtype, n, nnz, beyond=beyond)


@pytest.mark.parametrize("V,dtype", [(128_256, "f32"), (151_936, "bf16")])
@pytest.mark.parametrize("n", [2, 60, 192])
def test_chains_past_the_tables_end(V, dtype, n):
    _check(V, dtype, n, 3000, crowded=True)


def test_one_id_as_often_as_counters_hold():
    """A history of one listed id: 16-bit counts of occurrences and of generated tokens side by side."""
    V, B, nnz = 50_001, 4, 50_000
    rng = np.random.default_rng(9)
    z = np.full((B, V), -np.inf, np.float32)
    hist = np.empty((B, nnz), np.int32)
    for b in range(B):
        ids = rng.choice(V, 50, replace=False)
        z[b, ids] = rng.standard_normal(50) * 2.0
        hist[b] = ids[0]
    params = synth.make_params(B, temperature=1.0, top_p=0.99, rep_penalty=1.1, freq_penalty=2.0 ** -14, n_prompt=np.array([0, 49_999, 50_000, 25_000], np.int32))
    w = synth.Workload("one-id", B, V, "f32", z, params, np.arange(B + 1, dtype=np.int64) * nnz, hist.ravel())
    ids, dg = P.run_gpu(w, 0)
    P.compare(ids, dg, P.run_oracle(w, 0), range(B))
